"""Edges of the kernels' size rules: each variant that a dispatch can take, at the sizes where it can go wrong."""
import numpy as np
import pytest

import paper_2509_06980_amd as rl
from crafted import FILLER, KEY, KINDS, QUERY, SELF, KeyBits, ManySmallWeights, Peaked, weight_sum
from gemm_cases import DECODE, DECODE_ROWS, MANY_ROWS, MANY_ROWS_ORACLE, RESIDUAL, RESIDUAL_ROWS, small
from oracle import OracleEngine
from oracle.bf16_error_model import forward_bf16_model
from oracle.decoder import forward_full
from oracle.sampler import sample_token
from synthetic import SHAPES, make_weight_blob

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,rows,T", [(1, 2, 1.0), (5, 3, 1.0), (4095, 2, 0.7), (4096, 1, 1.0), (4097, 3, 1.0), (4100, 300, 1.0), (4101, 3, 1.0),
                                      (8192, 4, 1.0), (8196, 4, 1.0), (12292, 400, 1.0), (12292, 3, 0.0), (16384, 5, 1.0), (16384, 3, 0.0),
                                      (16388, 5, 1.0), (20483, 300, 1.0), (20484, 300, 1.0), (20484, 300, 0.0), (40964, 260, 0.7),
                                      (1100000, 2, 1.0), (1100001, 1, 0.0)])
def test_sampler_segment_layouts(V, rows, T):
    # rows of whole 16-byte pieces (in one workgroup of 256, 512 or 1024 threads up to 4096, 8192, 16384 logits) and others (up
    # to 4096); in segments beyond: one or several segments (two of 6, three of 11) per workgroup, a last one with few logits,
    # more than 256 in a row; masked logits (minus infinity and the lowest float: weight 0, as -1e30 for the oracle)
    rng = np.random.default_rng(V + rows)
    z = (rng.standard_normal((rows, V)) * 2).astype(np.float32)
    ref = z.copy()
    if V > 4:
        z[-1, ::3], ref[-1, ::3] = -np.inf, -1e30
        z[0, 1::2], ref[0, 1::2] = -3.4e38, -1e30
    u = rng.integers(0, 2**32, rows, dtype=np.uint64).astype(np.uint32)
    u[0] = 2**32 - 1
    ids, lps = rl.sample_from_logits(z, T, u)
    for r in sorted({0, rows // 2, rows - 1}):
        tok, lp = sample_token(ref[r], T, int(u[r]))
        assert ids[r] == tok, (r, ids[r], tok)
        # float32 sums of up to V terms in a tree over 16 x 256 and the segments: well below 1e-5
        assert abs(lps[r] - lp) < 1e-5 * max(1.0, abs(lp))


@pytest.mark.parametrize("V,rows", [(16388, 8), (20483, 300), (151936, 128), (151937, 6), (300004, 40)])
def test_sampler_log_probs_sum_in_one_order(V, rows):
    # a token whose weight is all but a thousandth: its log-prob is minus the logarithm of a sum just above one, in which an fp32 step of
    # the sum shows 2000 times over.  One to eight segments per workgroup, more than 64 in a row, rows of whole 16-byte pieces and others
    rng = np.random.default_rng(V)
    z = rng.standard_normal((rows, V)).astype(np.float32)
    at = rng.integers(0, V, rows)
    z[np.arange(rows), at] = 8.0 + np.log(V / 2.7)
    sums = np.array([weight_sum(r, 1.0) for r in z[:40]])
    assert (sums != [weight_sum(r, 1.0, by_lane=True) for r in z[:40]]).any() and sums.max() < 1.004
    ids, lps = rl.sample_from_logits(z, 1.0, np.full(rows, 2**31, np.uint32))
    assert np.array_equal(ids, at)
    # an fp32 step of the sums is 2^-23; of a logarithm below 2^-8 it is 2^-32
    assert np.abs(lps[:40] + np.log(sums.astype(np.float64))).max() < 2.0 ** -29


@pytest.mark.parametrize("V", [5, 4100, 4101, 16384, 16388])
def test_sampler_rows_without_weight(V):
    # no logit is a number, one is infinite, none is finite, one is no number: the id is a token all the same
    nan, inf = np.float32("nan"), np.float32("inf")
    rng = np.random.default_rng(V)
    z = rng.standard_normal((4, V)).astype(np.float32)
    z[0], z[2] = nan, -inf
    z[1, V // 2] = inf
    z[3, 1] = nan
    u = rng.integers(0, 2**32, 4, dtype=np.uint64).astype(np.uint32)
    others = z[3].copy()
    others[1] = -1e30
    drawn, lps = rl.sample_from_logits(z, 1.0, u)
    assert drawn.tolist() == [0, 0, 0, sample_token(others, 1.0, int(u[3]))[0]] and np.isnan(lps).all()
    best, lps = rl.sample_from_logits(z, 0.0, u)
    assert best.tolist() == [0, V // 2, 0, int(others.argmax())] and np.isnan(lps).all()
    assert [sample_token(z[r], 1.0, int(u[r]))[0] for r in range(4)] == drawn.tolist()      # the oracle's rule
    assert [sample_token(z[r], 0.0, 0)[0] for r in range(4)] == best.tolist()


@pytest.mark.parametrize("V", [4100, 16388])         # a row in one workgroup, and in segments
@pytest.mark.parametrize("T", [1e-45, 1e-40, 4e-39, 1e-37])
def test_sampler_temperatures_next_to_zero(T, V):
    # log2(e) / T beyond fp32: the maximum has all the weight, two equal maxima half of it each
    z = np.random.default_rng(5).standard_normal((3, V)).astype(np.float32)
    z[1:, 7] = z[1:, V - 1] = 9.0
    ids, lps = rl.sample_from_logits(z, T, np.array([123, 2**31 - 1, 2**31], np.uint32))
    assert ids.tolist() == [int(z[0].argmax()), 7, V - 1]
    assert np.abs(lps - [0.0, -np.log(2.0), -np.log(2.0)]).max() < 1e-6


@pytest.mark.parametrize("name", ["small-d128", "tiny"])
def test_decode_of_logits_that_are_no_numbers(name):
    # the token that such a row yields is embedded by the next step, on the device within a call
    shape = SHAPES[name].replace(tie_embeddings=1)
    blob = make_weight_blob(shape, seed=8, weight_std=0.03)
    kw = dict(max_context=64, max_trajectories=4, kv_pool_pages=16)
    g = rl.RolloutEngine(blob, **kw)
    g.append_observation([0], [3, 4, 5], [3])
    z = g.debug_logits(0)
    assert g.decode_steps([0], 2, 1e-40, 1)[0][0, 0] == z.argmax()                     # the temperature alone had done it
    assert not np.isnan(g.recompute_logprobs([0], 1e-40)).any()
    g.close()
    if shape.weight_dtype == 1:                                                        # the final norm's gains
        blob.view(np.uint16)[-shape.hidden:] = 0x7FC0
    else:
        blob.view(np.uint32)[-shape.hidden:] = 0x7FC00000
    g = rl.RolloutEngine(blob, **kw)
    g.append_observation([0, 1], [3, 4, 5], [1, 2])
    for T in (1.0, 0.0):
        ids, lps = g.decode_steps([0, 1], 3, T, 1)
        assert (ids == 0).all() and np.isnan(lps).all()
        ids, lps = g.decode_step([0, 1], T, 2)
        assert (ids == 0).all() and np.isnan(lps).all()
    assert (g.traj_read(1)[0][2:] == 0).all() and np.isnan(g.debug_logits(0)).all()
    g.close()


@pytest.mark.parametrize("name", ["small-g1", "small-g2", "small-d128", "small-g8"])
@pytest.mark.parametrize("lens", [[15], [256, 250], [127, 128, 129], [700], [1023, 900, 800], [40, 1000]])
def test_decode_attention_cuts_and_merges(name, lens):
    # contexts around the sizes at which a row is cut into parts (1 to 8 parts, equal and ragged batches),
    # every number of lane groups that share a row's parts (G = 1, 2, 4, 8), against the shape-generic kernels
    shape = SHAPES[name]
    blob = make_weight_blob(shape, seed=3, weight_std=0.03, gain_std=0.1)
    kw = dict(max_context=1100, max_trajectories=4, kv_pool_pages=280)
    a, b = rl.RolloutEngine(blob, **kw), rl.RolloutEngine(blob, flags=rl.FLAG_GENERIC_KERNELS, **kw)
    rng = np.random.default_rng(sum(lens))
    toks = rng.integers(0, shape.vocab, sum(lens))
    ids = list(range(len(lens)))
    for e in (a, b):
        e.append_observation(ids, toks, lens)
    for step in range(2):
        forced = rng.integers(0, shape.vocab, len(lens))
        la, lb = (e.decode_step_forced(ids, 1.0, forced) for e in (a, b))
        assert np.abs(la - lb).max() < 3e-2          # two bf16 paths, the bound of the parity tests
    za, zb = a.debug_logits(ids[-1]), b.debug_logits(ids[-1])
    assert np.abs(za - zb).max() < 3e-2
    o = OracleEngine(blob, **kw)                         # the last trajectory, as it stands now
    o.append_observation(ids[-1:], a.traj_read(ids[-1])[0], [lens[-1] + 2])
    assert np.abs(za - o.debug_logits(ids[-1])).max() < 3e-2
    a.close(), b.close()


@pytest.mark.parametrize("heads", [(2, 2), (4, 2), (8, 2), (8, 1), (16, 1)])
def test_prefill_attention_items_and_page_pairs(heads):
    # chunks on top of cached contexts: items of one row to 4 * 32 / G rows and one more, first and last row around the edges of
    # pages and of the pairs of pages that a stage holds, waves without rows, groups of 1 to 16 heads (G), against the
    # shape-generic kernels (two bf16 paths, the bound of the parity tests)
    shape = SHAPES["small-d128"].replace(n_q_heads=heads[0], n_kv_heads=heads[1], hidden=256, intermediate=512, vocab=4096, n_layers=2)
    blob = make_weight_blob(shape, seed=4, weight_std=0.03, gain_std=0.1)
    rows = 4 * 32 * heads[1] // heads[0]
    contexts = [0, 1, 15, 16, 17, 31, 32, 33, 64, 100]
    chunks = [1, 2, rows // 4, rows // 4 + 1, rows - 1, rows, rows + 1, 2 * rows + 5, 33, 300]
    kw = dict(max_context=512, max_trajectories=10, kv_pool_pages=300)
    a, b = rl.RolloutEngine(blob, **kw), rl.RolloutEngine(blob, flags=rl.FLAG_GENERIC_KERNELS, **kw)
    rng = np.random.default_rng(heads[0])
    first, more, forced = (rng.integers(0, shape.vocab, n) for n in (sum(contexts), sum(chunks), len(chunks)))
    got = []
    for e in (a, b):
        e.append_observation(range(1, 10), first, contexts[1:])
        e.append_observation(range(10), more, chunks)
        e.decode_step_forced(range(10), 1.0, forced)
        got.append(np.stack([e.debug_logits(i) for i in range(10)]))
        e.close()
    assert np.abs(got[0] - got[1]).max() < 3e-2


@pytest.mark.parametrize("heads", [(2, 2), (2, 1)])
def test_softmax_denominator_is_the_sum_of_unrounded_weights(heads):
    # up to 600 weights that bf16 would round down by 0.375 % each, in decode rows and in appended rows.  With a rounded
    # denominator the log-probs are 0.0015 to 0.0079 too high; the roundings behind it average to less than a tenth of that.
    m = ManySmallWeights(heads, 600)
    e = rl.RolloutEngine(m.blob, max_context=640, max_trajectories=1, kv_pool_pages=40)
    e.append_observation([0], [1, 0], [2])
    exact = m.logprobs(601)
    off = (m.logprobs(601, m.rounded) - exact)[100:].mean()
    decoded = np.concatenate([e.decode_step_forced([0], 1.0, [0]) for _ in range(600)])
    appended = e.recompute_logprobs([0], 1.0)[2:]
    for got in (decoded, appended):
        assert abs((got - exact)[100:].mean()) < 0.1 * off
    e.close()


@pytest.mark.parametrize("kv8", [False, True])
@pytest.mark.parametrize("heads", [(2, 2), (4, 2), (8, 2), (8, 1), (16, 1)])
def test_norm_rope_and_cache_write_inside_the_decode_attention(heads, kv8):
    # positions first and last in their page and around it, rows in one part and in several (the last part writes the page), groups of
    # 1 to 8 heads and of 16 (not taken); the oracle and the bound of the 8-bit parity tests for both caches
    shape = SHAPES["small-d128"].replace(n_q_heads=heads[0], n_kv_heads=heads[1], hidden=256, intermediate=512, vocab=4096, n_layers=2)
    blob = make_weight_blob(shape, seed=8, weight_std=0.03, gain_std=0.1)
    lens = [1, 15, 16, 17, 31, 33, 64, 255, 256, 700]
    kw = dict(max_context=720, max_trajectories=len(lens), kv_pool_pages=120)
    g = rl.RolloutEngine(blob, flags=rl.FLAG_FP8_KV_CACHE if kv8 else 0, **kw)
    o = OracleEngine(blob, kv_cache_dtype="fp8_e4m3" if kv8 else None, **kw)
    rng = np.random.default_rng(heads[0])
    ids, toks = np.arange(len(lens)), rng.integers(0, shape.vocab, sum(lens))
    for e in (g, o):
        e.append_observation(ids, toks, lens)
    seen = [toks[:1], toks[-700:]]
    bound = 8.0 * max(float(np.sqrt(np.mean((forward_bf16_model(o.model, t) - forward_full(o.model, t)) ** 2))) for t in seen)
    for rows in (ids, ids[-1:], ids):
        forced = rng.integers(0, shape.vocab, len(rows))
        assert np.abs(g.decode_step_forced(rows, 1.0, forced) - o.decode_step_forced(rows, 1.0, forced)).max() < bound
    for i in ids:
        assert np.abs(g.debug_logits(i) - o.debug_logits(i)).max() < bound
    g.close()


@pytest.mark.parametrize("kv8", [False, True])
@pytest.mark.parametrize("heads", [(2, 2), (4, 2), (8, 2), (8, 1), (16, 1)])
def test_decode_rows_meet_their_own_key(heads, kv8):
    # every row looks for its own key and no earlier one has it: a part that reads its last page before the key and the value are there
    # moves the log-probs by 1 and more and the logits by 2 and more.  Rows in one part and in several, first and last in a page.
    # Bound: bf16 roundings of outputs and rows of logits of deviation 1, 2^-9 each, of 4096 logits the largest; measured 0.012.
    p = Peaked(heads, kv8)
    lens = [1, 15, 16, 17, 31, 33, 64, 255, 256, 700]
    g = rl.RolloutEngine(p.blob, flags=rl.FLAG_FP8_KV_CACHE if kv8 else 0, max_context=720, max_trajectories=len(lens), kv_pool_pages=120)
    seen = [[FILLER] * (n - 1) + [SELF(i)] for i, n in enumerate(lens)]
    g.append_observation(np.arange(len(lens)), np.concatenate(seen), lens)

    def without(t):                                  # its own key like all others
        return t[:-1] + [QUERY(t[-1] - SELF(0))]
    for step, rows in enumerate((range(len(lens)), [len(lens) - 1], range(len(lens)))):
        new = [SELF(j) for j in range(len(lens) + 6 * step, len(lens) + 6 * step + 6)]
        want, apart = (np.stack([p.logprobs(t(seen[i]))[new] for i in rows]) for t in (lambda t: t, without))
        pick = np.abs(want - apart).argmax(1)
        at = np.arange(len(rows))
        assert (np.abs(want - apart)[at, pick][[len(seen[i]) > 1 for i in rows]] > 0.5).all()
        got = g.decode_step_forced(list(rows), 1.0, [new[k] for k in pick])
        assert np.abs(got - want[at, pick]).max() < 0.05
        for i, k in zip(rows, pick):
            seen[i].append(new[k])
    for i, t in enumerate(seen):
        assert np.abs(g.debug_logits(i) - p.logits(t)).max() < 0.05
        assert np.abs(p.logits(without(t)) - p.logits(t)).max() > 1.0
    g.close()


@pytest.mark.parametrize("flags", [0, rl.FLAG_SHARED_PREFIX_ATTENTION])
@pytest.mark.parametrize("appended", [True, False])
def test_keys_are_rounded_as_written(flags, appended):
    # keys formed in a pass of appended rows and in decode rows, there inside the attention and by the kernel of their own.  A
    # sum of squares with the other square fused moves all weight to one of two tokens that share it: logits by 1 and more.
    k = KeyBits()
    e = rl.RolloutEngine(k.blob, flags=flags, max_context=64, max_trajectories=k.pairs, kv_pool_pages=k.pairs)
    ids = np.arange(k.pairs)
    toks = np.stack([[0, 0, 1 + 3 * i, 2 + 3 * i, 3 + 3 * i] for i in ids])
    if appended:
        e.append_observation(ids, toks.reshape(-1), [5] * k.pairs)
    else:
        e.append_observation(ids, toks[:, :2].reshape(-1), [2] * k.pairs)
        for j in range(2, 5):
            e.decode_step_forced(ids, 1.0, toks[:, j])
    for i in ids:
        want = k.logits(i)
        assert min(np.abs(k.logits(i, share) - want).max() for share in (0.0, 1.0)) > 1.0
        assert np.abs(e.debug_logits(i) - want).max() < 0.05            # bf16 roundings of logits of deviation 1
    e.close()


@pytest.mark.parametrize("kv8", [False, True])
@pytest.mark.parametrize("heads", [(2, 2), (8, 2), (8, 1)])
@pytest.mark.parametrize("change", [dict(hidden=256, intermediate=512), dict(hidden=2560, intermediate=640)])
def test_norm_and_rope_inside_and_outside_the_attention_have_the_same_bits(change, heads, kv8):
    # an engine that may read shared pages once leaves them to the kernel of their own; nothing else differs where no trajectory is
    # forked.  Rows divided by their rms and rows still to be divided (the second layer's, behind a down product with the norm inside)
    shape = SHAPES["small-d128"].replace(n_q_heads=heads[0], n_kv_heads=heads[1], vocab=4096, n_layers=2, **change)
    blob = make_weight_blob(shape, seed=8, weight_std=0.03, gain_std=0.1)
    lens = [1, 15, 16, 17, 31, 33, 64, 255, 256, 700]
    kw = dict(max_context=720, max_trajectories=len(lens), kv_pool_pages=120)
    kv = rl.FLAG_FP8_KV_CACHE if kv8 else 0
    a, b = rl.RolloutEngine(blob, flags=kv, **kw), rl.RolloutEngine(blob, flags=kv | rl.FLAG_SHARED_PREFIX_ATTENTION, **kw)
    rng = np.random.default_rng(heads[0])
    ids, toks = np.arange(len(lens)), rng.integers(0, shape.vocab, sum(lens))
    for e in (a, b):
        e.append_observation(ids, toks, lens)
    for _ in range(8):
        forced = rng.integers(0, shape.vocab, len(lens))
        assert np.array_equal(a.decode_step_forced(ids, 1.0, forced), b.decode_step_forced(ids, 1.0, forced))
    for i in ids:
        assert np.array_equal(a.debug_logits(i), b.debug_logits(i))
    a.close(), b.close()


def test_decode_attention_of_many_keys_leaves_the_norm_and_rope_outside():
    # 90 and 128 forks of 4000 tokens: 369 and 525 MB of keys and values, either side of the limit
    shape = SHAPES["small-g1"]
    blob = make_weight_blob(shape, seed=9, weight_std=0.03, gain_std=0.1)
    rng = np.random.default_rng(9)
    toks, forced = rng.integers(0, shape.vocab, 4000), rng.integers(0, shape.vocab, (2, 128))
    got = []
    for n in (90, 128):
        e = rl.RolloutEngine(blob, max_context=4016, max_trajectories=128, kv_pool_pages=520)
        e.append_observation([0], toks, [4000])
        e.fork(0, list(range(1, 128)))
        got.append([e.decode_step_forced(list(range(n)), 1.0, f[:n])[:90] for f in forced])
        e.close()
    assert np.abs(np.stack(got[0]) - np.stack(got[1])).max() < 3e-2          # two bf16 paths, the bound of the parity tests


@pytest.mark.parametrize("kv8", [False, True])
@pytest.mark.parametrize("n", [3900, 3970, 4090, 4150, 4220, 4290, 8200])
def test_decode_attention_waves_of_more_pages_than_lanes(n, kv8):
    # 128 rows are not cut: 61, 63, 64, 65, 66, 68 and 129 pages a wave, whose table entries are read 64 at a time.  Every row looks for
    # one key, which lies in one page: first and last of a wave, and around the entries at which the next 64 are read.  A wave that
    # takes another page for it moves the row's log-prob by 0.5 at least (all but the looked-for key weigh next to nothing).
    # 2^-9 roundings of logits of deviation 1: 0.05, as above.
    p = Peaked((2, 2), kv8)
    pages = (n + 2 + 15) // 16                       # of the second step's rows
    per = (pages + 3) // 4
    places = [(w, k) for w in range(4) for k in sorted({0, 57, 58, 59, 60, 61, 62, 63, 64, 65, 119, 120, 122, 123, 126, per - 1}) if k < per and w * per + k < pages - 1]
    rng = np.random.default_rng(n)
    toks = np.zeros(n, np.int64)
    used = min(KINDS, len(places))
    for j, x in enumerate(rng.permutation(len(places))[:used]):
        w, k = places[x]
        toks[(w * per + k) * 16 + rng.integers(0, 16)] = KEY(j)
    e = rl.RolloutEngine(p.blob, flags=rl.FLAG_FP8_KV_CACHE if kv8 else 0, max_context=n + 16, max_trajectories=128, kv_pool_pages=n // 16 + 270)
    e.append_observation([0], toks, [n])
    e.fork(0, list(range(1, 128)))
    kinds = np.arange(128) % used
    e.decode_step_forced(np.arange(128), 1.0, [QUERY(j) for j in kinds])
    want = np.stack([p.logprobs(np.append(toks, QUERY(j))) for j in range(used)])
    missed = np.stack([p.logprobs(np.append(np.where(toks == KEY(j), FILLER, toks), QUERY(j))) for j in range(used)])
    forced = np.abs(want - missed).argmax(1)
    assert np.abs(want - missed).max(1).min() > 0.5
    got = e.decode_step_forced(np.arange(128), 1.0, forced[kinds])
    assert np.abs(got - want[kinds, forced[kinds]]).max() < 0.05
    e.close()


@pytest.mark.parametrize("change", [dict(), dict(hidden=260, intermediate=700, vocab=4100), dict(hidden=250, head_dim=62, vocab=4090),
                                    dict(head_dim=68), dict(head_dim=128, n_q_heads=2), dict(n_kv_heads=4, head_dim=6)])
@pytest.mark.parametrize("lens", [[1], [16, 1], [65], [17, 64, 130], [2] * 17])
def test_fp32_products_and_attention_at_the_edges(change, lens):
    # one and several 16-row blocks, K and N that end inside a block, rows that are no whole 4-element
    # pieces (the tile kernel, the scalar attention reads), contexts around pages and groups of four pages
    shape = SHAPES["tiny"].replace(n_layers=1, **change)
    blob = make_weight_blob(shape, seed=4, weight_std=0.05, gain_std=0.1)
    kw = dict(max_context=160, max_trajectories=20, kv_pool_pages=80)
    o, g = OracleEngine(blob, **kw), rl.RolloutEngine(blob, **kw)
    rng = np.random.default_rng(sum(lens))
    ids = list(range(len(lens)))
    toks = rng.integers(0, shape.vocab, sum(lens))
    forced = rng.integers(0, shape.vocab, len(lens))
    for e in (o, g):
        e.append_observation(ids, toks, lens)
    lo, lg = (e.decode_step_forced(ids, 1.0, forced) for e in (o, g))
    assert np.abs(lo - lg).max() < 1e-4              # the fp32 bound of the parity tests
    for i in (ids[0], ids[-1]):
        assert np.abs(o.debug_logits(i) - g.debug_logits(i)).max() < 1e-4
    assert np.abs(o.recompute_logprobs(ids, 1.0) - g.recompute_logprobs(ids, 1.0)).max() < 1e-4
    g.close()


@pytest.mark.parametrize("kv8", [False, True])
@pytest.mark.parametrize("change,lens,sampled,takes", MANY_ROWS)
def test_many_row_products(change, lens, sampled, takes, kv8):
    # long trajectories and real widths against the shape-generic kernels (the 8-bit cache coarsely: its own oracle is below)
    shape = small(**change)
    blob = make_weight_blob(shape, seed=6, weight_std=0.02, gain_std=0.1)
    kw = dict(max_context=4096, max_trajectories=4, kv_pool_pages=520)
    a = rl.RolloutEngine(blob, flags=rl.FLAG_FP8_KV_CACHE if kv8 else 0, **kw)
    b = rl.RolloutEngine(blob, flags=rl.FLAG_GENERIC_KERNELS, **kw)
    rng = np.random.default_rng(sum(lens))
    ids = list(range(len(lens)))
    toks = rng.integers(0, shape.vocab, sum(lens))
    for e in (a, b):
        e.append_observation(ids, toks, lens)
    for _ in range(sampled):
        forced = rng.integers(0, shape.vocab, len(lens))
        for e in (a, b):
            e.decode_step_forced(ids, 1.0, forced)
    # two bf16 paths over one layer: the bound of the parity tests, on logits of standard deviation up to 1;
    # the 8-bit cache moves keys and values by up to 2^-4, attenuated by the average over the context
    tol = 3e-2 if not kv8 else 0.25
    za, zb = a.debug_logits(ids[-1]), b.debug_logits(ids[-1])
    assert np.abs(za - zb).max() < tol * max(1.0, float(zb.std()))
    ra, rb = a.recompute_logprobs(ids, 1.0), b.recompute_logprobs(ids, 1.0)
    assert np.abs(ra - rb).max() < tol
    assert np.array_equal(ra, a.recompute_logprobs(ids, 1.0))        # the same bits again
    a.close(), b.close()


@pytest.mark.parametrize("kv8", [False, True])
@pytest.mark.parametrize("change,lens,sampled,takes", MANY_ROWS_ORACLE)
def test_many_row_products_against_the_oracle(change, lens, sampled, takes, kv8):
    # every tile, K-slice and epilogue of the many-row products at widths that end inside a tile.  The bound of the 8-bit
    # parity tests for both caches: eight times the rms that bf16 arithmetic costs on the trajectory under test (the largest
    # of some thousand near-Gaussian differences lies at five to seven times it).  With short contexts a misplaced
    # part of a head is 2 to 60 times the bound (8- or 4-dim pieces of one head's keys or values swapped in the oracle).
    shape = small(**change)
    blob = make_weight_blob(shape, seed=6, weight_std=0.02, gain_std=0.1)
    kw = dict(max_context=max(lens) + sampled + 2, max_trajectories=len(lens), kv_pool_pages=sum((n + sampled + 16) // 16 for n in lens))
    g = rl.RolloutEngine(blob, flags=rl.FLAG_FP8_KV_CACHE if kv8 else 0, **kw)
    o = OracleEngine(blob, kv_cache_dtype="fp8_e4m3" if kv8 else None, **kw)
    rng = np.random.default_rng(sum(lens))
    ids, ends = np.arange(len(lens)), np.cumsum(lens)
    toks = [rng.integers(0, shape.vocab, n) for n in lens]
    rows = np.cumsum([n - 1 for n in lens])
    picked = sorted({int(np.searchsorted(rows, r, side="right")) for r in (0, 128, 256, rows[-1] // 2, rows[-1] - 1) if r < rows[-1]})
    g.append_observation(ids, np.concatenate(toks), lens)
    o.append_observation(picked, np.concatenate([toks[i] for i in picked]), [lens[i] for i in picked])
    bound = 8.0 * max(float(np.sqrt(np.mean((forward_bf16_model(o.model, toks[i]) - forward_full(o.model, toks[i])) ** 2))) for i in picked)
    for i in picked:
        assert np.abs(g.debug_logits(i) - o.debug_logits(i)).max() < bound
    for _ in range(sampled):
        forced = rng.integers(0, shape.vocab, len(lens))
        lg, lo = g.decode_step_forced(ids, 1.0, forced), o.decode_step_forced(picked, 1.0, forced[picked])
        assert np.abs(lg[picked] - lo).max() < bound
    rec, ref = g.recompute_logprobs(ids, 1.0), o.recompute_logprobs(picked, 1.0)
    start = ends - lens + sampled * ids
    assert np.abs(np.concatenate([rec[start[i]:start[i] + lens[i] + sampled] for i in picked]) - ref).max() < bound
    assert np.array_equal(rec, g.recompute_logprobs(ids, 1.0))        # the same bits again
    g.close()


@pytest.mark.parametrize("change", DECODE)
@pytest.mark.parametrize("rows", DECODE_ROWS)
def test_decode_products_row_counts(change, rows):
    # every row count at which the decode products change their tile, tiles of 32, 64, 80 and 96 columns, widths
    # that end inside the last two, depths that are no whole number of 128-k stages, K-slices of unequal length
    shape = small(**change)
    blob = make_weight_blob(shape, seed=7, weight_std=0.02, gain_std=0.1)
    kw = dict(max_context=32, max_trajectories=rows, kv_pool_pages=rows)
    a, b = rl.RolloutEngine(blob, **kw), rl.RolloutEngine(blob, flags=rl.FLAG_GENERIC_KERNELS, **kw)
    rng = np.random.default_rng(rows)
    ids = np.arange(rows, dtype=np.int32)
    toks = rng.integers(0, shape.vocab, 3 * rows)
    forced = rng.integers(0, shape.vocab, rows)
    for e in (a, b):
        e.append_observation(ids, toks, [3] * rows)
    la, lb = (e.decode_step_forced(ids, 1.0, forced) for e in (a, b))
    assert np.abs(la - lb).max() < 3e-2              # two bf16 paths over one layer, logits of deviation below 1.3
    o, picked = OracleEngine(blob, **kw), sorted({0, rows // 2, rows - 1})
    o.append_observation(picked, toks.reshape(rows, 3)[picked].reshape(-1), [3] * len(picked))
    assert np.abs(la[picked] - o.decode_step_forced(picked, 1.0, forced[picked])).max() < 3e-2
    a.close(), b.close()


@pytest.mark.parametrize("change", RESIDUAL)
@pytest.mark.parametrize("rows", RESIDUAL_ROWS)
def test_residual_add_and_norm_inside_the_products(change, rows):
    # two layers: gate-up and the next layer's QKV divide the rows by their rms, the last norm reads the stream itself;
    # the same trajectory twice in the batch has the same bits wherever its row lies
    shape = small(**change).replace(n_layers=2)
    blob = make_weight_blob(shape, seed=8, weight_std=0.02, gain_std=0.1)
    kw = dict(max_context=32, max_trajectories=rows, kv_pool_pages=rows)
    a, b = rl.RolloutEngine(blob, **kw), rl.RolloutEngine(blob, flags=rl.FLAG_GENERIC_KERNELS, **kw)
    rng = np.random.default_rng(rows)
    ids = np.arange(rows, dtype=np.int32)
    toks, forced = rng.integers(0, shape.vocab, (rows, 3)), rng.integers(0, shape.vocab, (2, rows))
    toks[-1], forced[:, -1] = toks[0], forced[:, 0]
    for e in (a, b):
        e.append_observation(ids, toks.reshape(-1), [3] * rows)
    o, picked = OracleEngine(blob, **kw), sorted({0, rows // 2, rows - 1})
    o.append_observation(picked, toks[picked].reshape(-1), [3] * len(picked))
    # logits of deviation below 1.3, as in the one-layer cases and their 3e-2: the layers' roundings are independent,
    # their energies add, and two layers have at most twice that of one and the head
    bound = 3e-2 * 2 ** 0.5
    for step in forced:
        la, lb = (e.decode_step_forced(ids, 1.0, step) for e in (a, b))
        assert la[0] == la[-1]
        assert np.abs(la - lb).max() < bound
        assert np.abs(la[picked] - o.decode_step_forced(picked, 1.0, step[picked])).max() < bound
    a.close(), b.close()


@pytest.mark.parametrize("hidden,head_dim,heads,intermediate", [
    (256, 64, (4, 2), 688), (256, 128, (2, 1), 324),     # norm, QKV, RoPE and cache write in one launch up to 64 rows
    (20, 64, (1, 1), 20),                                # one piece of four, waves without a step
    (516, 64, (3, 3), 260),                              # too wide for it: the norm inside the product, RoPE apart
    (256, 48, (4, 2), 100), (254, 64, (4, 2), 256)])     # another head_dim; rows that are no whole pieces: apart
@pytest.mark.parametrize("rows", [1, 16, 17, 64, 65])
def test_fp32_products_with_the_norm_inside(hidden, head_dim, heads, intermediate, rows):
    shape = SHAPES["tiny"].replace(hidden=hidden, head_dim=head_dim, n_q_heads=heads[0], n_kv_heads=heads[1],
                                   intermediate=intermediate, vocab=516)
    blob = make_weight_blob(shape, seed=9, weight_std=0.03, gain_std=0.1)
    kw = dict(max_context=32, max_trajectories=rows, kv_pool_pages=2 * rows)
    o, g = OracleEngine(blob, **kw), rl.RolloutEngine(blob, **kw)
    rng = np.random.default_rng(rows)
    ids, lens = np.arange(rows, dtype=np.int32), rng.integers(1, 9, rows)
    toks = rng.integers(0, shape.vocab, int(lens.sum()))
    for e in (o, g):
        e.append_observation(ids, toks, lens)
    for step in range(2):
        forced = rng.integers(0, shape.vocab, rows)
        a, b = (e.decode_step_forced(ids, 1.0, forced) for e in (o, g))
        assert np.abs(a - b).max() < 1e-4            # the fp32 bound of the whole suite
    k = rows // 2
    assert np.abs(o.debug_logits(k) - g.debug_logits(k)).max() < 1e-4
    assert np.abs(np.asarray(o.recompute_logprobs([k], 1.0)) - g.recompute_logprobs([k], 1.0)).max() < 1e-4
    g.close()


@pytest.mark.parametrize("n,steps", [(700, 20), (2000, 12), (2000, 330)])
def test_decode_steps_of_batches_that_leave_few_staging_regions(n, steps):
    # 28 regions (three groups of eight), eight (two groups of four, used again), and 42 000 page-table entries, more than a quarter of
    # the staging buffer (ahead on their own): the single steps' bits
    assert rl.debug_staging_plan(n, 0, n, 0, n * (steps // 16 + 1)) == {(700, 20): (False, 24, 8), (2000, 12): (False, 8, 4), (2000, 330): (True, 8, 4)}[n, steps]
    shape = SHAPES["tiny"].replace(n_layers=1, hidden=64, n_q_heads=1, n_kv_heads=1, intermediate=64, vocab=128)
    blob = make_weight_blob(shape, seed=5, weight_std=0.05)
    kw = dict(max_context=352, max_trajectories=n, kv_pool_pages=n * 22)
    a, b = rl.RolloutEngine(blob, **kw), rl.RolloutEngine(blob, **kw)
    ids = np.arange(n, dtype=np.int32)
    for e in (a, b):
        e.append_observation(ids, np.arange(n) % 128, np.ones(n, np.int32))
    single = [a.decode_step(ids, 1.0, 5) for _ in range(steps)]
    got_ids, got_lps = b.decode_steps(ids, steps, 1.0, 5)
    assert np.array_equal(got_ids, np.stack([x[0] for x in single])) and np.array_equal(got_lps, np.stack([x[1] for x in single]))
    assert a.n_free_pages() == b.n_free_pages()


def test_decode_steps_of_eight_thousand_trajectories():
    # parts of cut rows need room in every region: one fits the staging buffer, and only without the call's page-table entries
    shape = SHAPES["small-d128"].replace(n_layers=1, hidden=256, n_q_heads=8, n_kv_heads=8, intermediate=64, vocab=4096)
    blob = make_weight_blob(shape, seed=5, weight_std=0.05)
    n, steps = 8000, 64
    assert rl.debug_staging_plan(n, 8, n, 0, 4 * n) == (True, 1, 1) and rl.debug_staging_plan(n, 8, n) == (False, 1, 1)
    ids = np.arange(n, dtype=np.int32)
    got = []
    for several in (False, True):
        e = rl.RolloutEngine(blob, max_context=80, max_trajectories=n, kv_pool_pages=5 * n)
        e.append_observation(ids, np.arange(n) % 4096, np.ones(n, np.int32))
        r = e.decode_steps(ids, steps, 1.0, 5) if several else [np.stack(x) for x in zip(*[e.decode_step(ids, 1.0, 5) for _ in range(steps)])]
        got.append((*r, *e.decode_step(ids, 1.0, 6), e.n_free_pages()))
        e.close()
    assert all(np.array_equal(x, y) for x, y in zip(*got))


def test_decode_steps_that_do_not_fit_take_no_pages():
    # more trajectories than the staging buffer has room for, at the end of their pages: refused, and a single step goes on as if nothing had been
    shape = SHAPES["small-d128"].replace(n_layers=1, hidden=256, n_q_heads=8, n_kv_heads=8, intermediate=64, vocab=4096)
    n = 14000
    assert rl.debug_staging_plan(n, 8, n)[1] == 0
    e = rl.RolloutEngine(make_weight_blob(shape, seed=5, weight_std=0.05), max_context=64, max_trajectories=n, kv_pool_pages=2 * n)
    ids = np.arange(n, dtype=np.int32)
    e.append_observation([0, n - 1], np.arange(32), [16, 16])
    e.append_observation(ids[1:-1], np.ones(n - 2, np.int32), np.ones(n - 2, np.int32))
    before = e.n_free_pages(), e.traj_read(0)[3].tolist()
    with pytest.raises(rl.RolloutError):
        e.decode_steps(ids, 3, 1.0, 5)
    assert (e.n_free_pages(), e.traj_read(0)[3].tolist()) == before
    want = e.decode_step([n - 1], 1.0, 7), e.decode_step([0], 1.0, 7)
    assert e.n_free_pages() == before[0] - 2 and len(e.traj_read(0)[3]) == 2 and np.isfinite([w[1] for w in want]).all()
    e.close()
