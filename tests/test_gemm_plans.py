"""The choice of kernel and K-slices for the products of a pass (host arithmetic of the library)."""
import os
import random

import pytest

import paper_2509_06980_amd as rl
from gemm_cases import DECODE, DECODE_ROWS, MANY_ROWS, MANY_ROWS_ORACLE, RESIDUAL, RESIDUAL_ROWS, small
from synthetic import SHAPES

PRODUCTS = ("qkv", "o", "gate_up", "down", "score_head", "logits_head")


@pytest.fixture(scope="module", autouse=True)
def lib():
    if not os.path.exists(rl.LIB_PATH):
        from paper_2509_06980_amd import build
        build.build()
    return rl.load_library()


def _dims(s):
    """product -> (N, K)"""
    return dict(qkv=(s.q_width + 2 * s.kv_width, s.hidden), o=(s.hidden, s.q_width), gate_up=(2 * s.intermediate, s.hidden),
                down=(s.hidden, s.intermediate), score_head=(s.vocab, s.hidden), logits_head=(s.vocab, s.hidden))


def test_plans_stay_within_what_kernels_and_buffers_take():
    rng = random.Random(5)
    taken = set()
    for _ in range(3000):
        nkv = rng.choice([1, 2, 3, 4, 8, 16, 32])
        s = SHAPES["small-d128"].replace(
            hidden=64 * rng.randint(1, 96), n_kv_heads=nkv, n_q_heads=nkv * rng.choice([1, 2, 4, 8]),
            intermediate=64 * rng.randint(1, 256), vocab=32 * rng.choice([1, 3, 128, 1000, 4748]))
        rows = int(round(2 ** rng.uniform(0, 13)))
        cap = max(rows, rng.choice([rows, 128, 1024, 8192]))
        cap += -cap % 128
        partial = max(cap, 8 * min(cap, 1024))            # rows of the partial-sum buffers
        for name, (kernel, width, slices, epilogue) in rl.debug_pass_plan(s, rows, cap).items():
            n, k = _dims(s)[name]
            taken.add((kernel, width, min(slices, 2), epilogue))
            assert 1 <= slices <= 8 and (slices == 1 or (epilogue == "store" and name != "logits_head"))
            assert slices * rows <= max(partial, rows)
            if epilogue in ("qkv", "add"):
                assert kernel in ("tile256", "wide128") and rows > 128 and slices == 1
                assert epilogue != "qkv" or width == 4                # a wave's 128 columns are a head
            if kernel == "decode":
                assert rows <= 128 and width in (2, 4, 5, 6)
                depth = 128 if width == 5 else 64
                assert k % depth == 0
                per = -(-(k // depth) // slices)
                assert (slices - 1) * per < k // depth                # no slice is empty
            elif kernel in ("tile256", "wide128"):
                assert rows > 128 and width in ((4, 5) if kernel == "tile256" else (4,))
                per = -(-(k // 32) // slices)
                assert (slices - 1) * per < k // 32
            else:
                assert kernel == "tile128"
    # every variant that the library holds is some size's choice
    for variant in [("decode", w, 1, e) for w in (2, 4, 5, 6) for e in ("store", "swiglu")] + \
            [("tile256", w, 1, e) for w in (4, 5) for e in ("add", "swiglu")] + [("tile256", 4, 1, e) for e in ("qkv", "logprob", "store")] + \
            [("wide128", 4, 1, e) for e in ("add", "swiglu", "qkv", "store")] + \
            [("tile128", 0, 1, e) for e in ("store", "swiglu", "logprob")] + \
            [(kernel, w, 2, "store") for kernel, w in (("decode", 2), ("decode", 4), ("tile256", 4), ("tile256", 5), ("wide128", 4), ("tile128", 0))]:
        assert variant in taken, variant


@pytest.mark.parametrize("heads,hidden,rows,fused", [
    ((32, 32), 4096, 300, True),                 # four K-slices of a wide projection: 80.5 us apart, 70.3 us in one
    ((32, 8), 4096, 3072, False),                # 160.7 us apart, 172.2 us in one
    ((32, 32), 4096, 1536, False),               # 168.6 / 173.0
    ((32, 8), 2560, 8192, True), ((32, 8), 2560, 587, False), ((16, 8), 1024, 2048, True), ((32, 8), 4096, 8192, True),
])
def test_projection_epilogue_follows_the_width(heads, hidden, rows, fused):
    s = SHAPES["small-d128"].replace(n_q_heads=heads[0], n_kv_heads=heads[1], hidden=hidden)
    assert (rl.debug_pass_plan(s, rows)["qkv"][3] == "qkv") == fused


@pytest.mark.parametrize("rows", [1, 64, 128, 129, 600, 8192])
def test_weights_beyond_a_buffer_descriptor_keep_64_bit_addresses(rows):
    # N x K bf16 weights of 0x7fff0000 bytes and more: loads with the LDS destination have 31-bit offsets
    base = SHAPES["qwen3-8b"]
    for over, name, change in ((True, "score_head", dict(vocab=262144)), (False, "score_head", dict(vocab=262016)),
                               (True, "gate_up", dict(intermediate=131072)), (False, "gate_up", dict(intermediate=131008)),
                               (True, "down", dict(intermediate=262144)), (False, "down", dict(intermediate=262016))):
        s = base.replace(**change)
        n, k = _dims(s)[name]
        assert (2 * n * k >= 0x7FFF0000) == over
        plan = rl.debug_pass_plan(s, rows)
        if over:
            assert plan[name][0] == "tile128"
            assert name != "score_head" or plan["logits_head"][0] == "tile128"
        elif rows == 8192:                                        # the limit decides, not the estimate
            assert plan[name][0] != "tile128"


def test_pass_plan_refuses_what_the_matrix_kernels_do_not_take():
    s = SHAPES["small-d128"]
    for bad, rows in ((s.replace(head_dim=64), 1), (s.replace(weight_dtype=0), 1), (s.replace(hidden=96), 1),
                      (s.replace(n_q_heads=6), 1), (s.replace(vocab=100), 1), (s, 0)):
        with pytest.raises(rl.RolloutError) as ei:
            rl.debug_pass_plan(bad, rows)
        assert ei.value.code == -1


@pytest.mark.parametrize("change,lens,sampled,takes", MANY_ROWS + MANY_ROWS_ORACLE)
def test_many_row_cases_reach_the_variants_that_they_are_there_for(change, lens, sampled, takes):
    rows = dict(append=sum(n - 1 for n in lens), recompute=sum(n + sampled - 1 for n in lens), score=sampled * len(lens))
    for part, products in takes.items():
        assert rows[part] <= 8192                                  # one pass
        plan = rl.debug_pass_plan(small(**change), rows[part])
        assert {name: plan[name] for name in products} == products


def test_decode_cases_reach_every_tile():
    seen = set()
    for change in DECODE:
        s = small(**change)
        for rows in DECODE_ROWS:
            inside = rl.debug_residual_plan(s, rows)               # O and down leave the plan there
            for name, (kernel, width, slices, epilogue) in rl.debug_pass_plan(s, rows).items():
                if kernel != "decode" or name in inside or name in ("score_head", "logits_head"):
                    continue
                n, k = _dims(s)[name]
                stages, tiles = k // (128 if width == 5 else 64), -(-n // (16 * width))
                seen |= {(width, epilogue, rows > 64), (width, epilogue, rows > 64, "ends inside" if n % (16 * width) else "whole"),
                         (width, epilogue, rows > 64, "unequal slices" if stages % slices else "equal slices")}
                if rows <= 64 and slices == 4 and -(-stages // 4) * (k // stages) >= 512:      # numbered by XCD
                    seen.add(("by XCD", width, "remainder" if tiles % 2 else "none"))
    for more in (False, True):                                     # one and two 16-row blocks a wave
        for width in (2, 4, 5, 6):
            assert (width, "store", more) in seen and (width, "swiglu", more) in seen
            assert (width, "store", more, "unequal slices") in seen
        for width in (5, 6):                                       # every width is a multiple of 64
            assert (width, "store", more, "ends inside") in seen and (width, "swiglu", more, "ends inside") in seen
    assert {("by XCD", 4, "none"), ("by XCD", 5, "remainder"), ("by XCD", 6, "remainder")} <= seen


def test_residual_products_tiles_and_bounds():
    reached, past_caches = {}, set()
    for change in RESIDUAL:
        s = small(**change)
        for rows in RESIDUAL_ROWS:
            for name, tile in rl.debug_residual_plan(s, rows).items():
                reached.setdefault((name, tile), set()).add(rows)
                n, k = _dims(s)[name]
                if rows <= 16 * tile[0] and 2 * n * k >= 24 << 20:
                    past_caches.add(tile)
    assert past_caches == {(1, 1), (1, 2), (2, 2)}
    for name in ("o", "down"):
        for tile in ((1, 1), (1, 2), (2, 2)):
            assert (name, tile) in reached, (name, tile)
        assert {1, 16} <= reached[name, (1, 1)] and {17, 33} & reached[name, (1, 2)] and 64 in reached[name, (2, 2)]
    rng = random.Random(6)
    for _ in range(2000):
        nkv = rng.choice([1, 2, 4, 8])
        s = SHAPES["small-d128"].replace(hidden=64 * rng.randint(1, 96), n_kv_heads=nkv, n_q_heads=nkv * rng.choice([1, 2, 4]),
                                         intermediate=64 * rng.randint(1, 256))
        rows = int(round(2 ** rng.uniform(0, 9)))
        plan, inside = rl.debug_pass_plan(s, rows), rl.debug_residual_plan(s, rows)
        assert not inside or rows <= 512
        assert "down" not in inside or plan["qkv"][3] == "store"      # the norm / RoPE kernel divides the rows
        if "o" in inside:             # gate-up divides them: the 128-column kernel, or the decode kernel where its ring
            kernel, width = plan["gate_up"][:2]                       # and 4 bytes per row and 16 columns fit 160 KB
            assert kernel in ("decode", "tile128")
            if kernel == "tile128":
                continue
            ring = (3 if width == 5 else 4) * (4 * (1 if rows <= 64 else 2) + width) * (4 if width == 5 else 2) * 1024
            assert ring + -(-rows // 16) * 16 * (s.hidden // 16) * 4 <= 160 * 1024
    for rows in (1, 16, 512):
        assert "down" not in rl.debug_residual_plan(SHAPES["qwen3-8b"].replace(intermediate=262144), rows)      # 31-bit offsets


@pytest.mark.parametrize("shape,rows,inside", [
    ((4096, 8, 2, 1024), 448, set()), ((4096, 8, 2, 1024), 131, {"o", "down"}),      # a layer without attention 97 us apart, 105 inside
    ((2048, 16, 8, 1536), 512, set()), ((2048, 16, 8, 1536), 192, {"o", "down"}),    # 80, 84
    ((2560, 8, 8, 1088), 512, set()), ((2560, 8, 8, 1088), 192, {"o", "down"}),      # 85, 90
    ((2560, 32, 8, 2048), 192, {"down"}),                                            # O of 4096: 46.2 with gate-up, 47.6
    ((1024, 16, 8, 3072), 512, {"o", "down"}), ((512, 8, 2, 1024), 512, {"o", "down"}),
])
def test_residual_products_of_more_than_128_rows_where_they_are_faster(shape, rows, inside):
    s = SHAPES["small-d128"].replace(**dict(zip(("hidden", "n_q_heads", "n_kv_heads", "intermediate"), shape)))
    assert set(rl.debug_residual_plan(s, rows)) == inside


def test_many_row_loads_stay_inside_their_buffers():
    # the scalar part of every load's offset, also of chunks behind a K-slice, strips behind the last and the second 128-row tile of
    # 256 rows that is not there: at every plan's rows, widths that end inside a tile, slices of odd and unequal length
    rng = random.Random(7)
    cases = [(587, 2560, 9728, "down"), (8192 - 100, 2560, 9728, "down"), (129, 32, 64, "o"), (385, 1056, 2112, "o")]
    cases += [(rng.randint(129, 1400), 32 * rng.randint(1, 40), 64 * rng.randint(1, 50), "o") for _ in range(60)]
    for rows, n, k, name in cases:
        for kernel, width in (("wide128", 4), ("tile256", 4), ("tile256", 5)):
            for slices in (1, 2, 3, 5, 8):
                if (slices - 1) * -(-(k // 32) // slices) < k // 32:          # no slice is empty
                    for epilogue in ("store", "add", "swiglu"):
                        stages, beyond_rows, beyond_weights = rl.debug_many_row_loads(rows, n, k, (kernel, width, slices, epilogue))
                        assert stages in (3, 4) and (beyond_rows, beyond_weights) == (0, 0), (rows, n, k, kernel, width, slices)


@pytest.mark.parametrize("rows,n,k,slices,epilogue,stages", [
    (587, 2560, 9728, 5, "store", 4), (587, 2560, 4096, 1, "add", 4),      # 250 workgroups of 61 chunks, 50 of 128: one to a CU
    (587, 2560, 9728, 8, "store", 3),                                      # 400 workgroups: two share one
    (587, 2560, 7616, 5, "store", 4), (587, 2560, 7488, 5, "store", 3),    # 48 and 47 chunks
    (300, 19456, 2560, 1, "swiglu", 4), (300, 6144, 2560, 1, "qkv", 3),    # the norm's epilogue has no room for a fourth
])
def test_stages_of_the_128_row_tiles(rows, n, k, slices, epilogue, stages):
    assert rl.debug_many_row_loads(rows, n, k, ("wide128", 4, slices, epilogue))[0] == stages


@pytest.mark.parametrize("bad", [(0, 32, 64, ("wide128", 4, 1, "store")), (200, 33, 64, ("wide128", 4, 1, "store")),
                                 (200, 32, 96, ("wide128", 4, 1, "store")), (200, 32, 64, ("decode", 4, 1, "store")),
                                 (200, 32, 64, ("wide128", 5, 1, "store")), (200, 32, 64, ("tile256", 4, 9, "store")),
                                 (200, 262144, 4096, ("tile256", 4, 1, "store"))])
def test_many_row_loads_refuse_what_the_kernel_does_not_take(bad):
    with pytest.raises(rl.RolloutError):
        rl.debug_many_row_loads(*bad)


def test_staging_of_several_decode_steps():
    # a call that fits without its page-table entries is taken; two groups wherever there are two regions, so that the host fills one
    # while the GPU works on the other; the entries cost no regions that two groups of eight would need
    rng = random.Random(8)
    seen = set()
    for _ in range(4000):
        T = int(round(2 ** rng.uniform(0, 15)))
        n, nkv, rows = rng.randint(1, T), rng.choice([0, 1, 2, 4, 8, 16]), rng.choice([0, 128, 2048, 16384])
        pages = int(n * rng.choice([0, 0.1, 1, 4, 64, 300]))
        cap = -(-max(rows or 8192, T) // 128) * 128
        room = 32 * cap + 3 * 65536
        region = 7 * n + 8 * (2 * n + (1024 // nkv + 3 * T + 64 if nkv else 0) + 8)
        ahead, regions, group = rl.debug_staging_plan(n, nkv, T, rows, pages)
        bare = min(room // region, 64)
        assert (regions >= 1) == (bare >= 1)
        assert regions * region + (0 if ahead else 3 * pages) <= room
        assert 1 <= group <= 8 and regions % group == 0
        if bare >= 2:
            assert regions >= 2 * group and regions > min(bare, 16) - group
        seen.add((ahead, min(regions, 2), min(group, 2)))
    assert seen == {(a, r, g) for a in (False, True) for r, g in ((1, 1), (2, 1), (2, 2))} | {(False, 0, 1), (True, 0, 1)}
    assert rl.debug_staging_plan(128, 8, 128, 0, 600) == (False, 56, 8)
