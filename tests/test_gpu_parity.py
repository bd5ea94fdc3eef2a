"""GPU parity: the HIP path (through the C boundary) against the CPU oracle."""
import json
import os

import numpy as np
import pytest

import paper_2509_06980_amd as rl
from oracle import OracleEngine, RolloutError as OracleError
from oracle.sampler import sample_token, uniform_u32
from synthetic import SHAPES, make_weight_blob, make_workload
from synthetic.workloads import replay, uniform_turns, ragged_turns
from lockstep import run_lockstep, compare_records
from tolerances import check_against_rounding_model

pytestmark = pytest.mark.gpu

TOL_FP32 = 1e-4      # max abs error on logits / log-probs, fp32 mode
TOL_BF16 = 3e-2      # bf16 mode


def _pair(shape, blob, flags=0, **kw):
    kw.setdefault("max_context", 1024)
    kw.setdefault("max_trajectories", 16)
    kw.setdefault("kv_pool_pages", 256)
    okw = {k: v for k, v in kw.items() if k != "max_batch_rows"}
    return OracleEngine(blob, **okw), rl.RolloutEngine(blob, flags=flags, **kw)


# ---- sampler in isolation: identical logits + identical draws => identical ids -------------
@pytest.mark.parametrize("V", [4096, 151936, 1000])
@pytest.mark.parametrize("T", [1.0, 0.7, 0.0, 3.0])
def test_sampler_ids_bit_exact(V, T):
    rng = np.random.default_rng(V + int(T * 10))
    rows = 24
    z = (rng.standard_normal((rows, V)) * rng.choice([0.3, 1.0, 4.0], size=(rows, 1))).astype(np.float32)
    z[0] = 0.0                                   # uniform
    z[1, 7] = z[1, V - 3] = z[1].max() + 1.0     # tie for the arg-max
    z[2] = -50.0; z[2, 5] = 0.0; z[2, V // 2] = 0.0   # almost all weights exactly zero
    u = rng.integers(0, 2**32, rows, dtype=np.uint64).astype(np.uint32)
    u[3], u[4] = 0, 2**32 - 1
    ids, lps = rl.sample_from_logits(z, T, u)
    for r in range(rows):
        tok, lp = sample_token(z[r], T, int(u[r]))
        assert ids[r] == tok, (r, ids[r], tok)
        assert abs(lps[r] - lp) < TOL_FP32


def test_sampler_draws_match_oracle_stream():
    # inside a decode step the draw is u(seed, traj id, index of the new token)
    shape = SHAPES["tiny"].replace(n_layers=1)
    blob = make_weight_blob(shape, seed=5, weight_std=0.05, gain_std=0.1)
    o, g = _pair(shape, blob)
    toks = np.random.default_rng(0).integers(0, shape.vocab, 3 * 9)
    for e in (o, g):
        e.append_observation([4, 11, 7], toks, [9, 9, 9])
    for step in range(6):
        z = {t: g.debug_logits(t) for t in (4, 11, 7)}
        ids, lps = g.decode_step([4, 11, 7], 1.0, 77)
        for k, t in enumerate((4, 11, 7)):
            tok, lp = sample_token(z[t], 1.0, uniform_u32(77, t, 9 + step))
            assert ids[k] == tok and abs(lps[k] - lp) < TOL_FP32


@pytest.mark.parametrize("n_rows", [3, 40, 70, 131])
@pytest.mark.parametrize("vocab", [8192, 20512, 24608])
def test_mfma_decode_step_sampler_with_strip_maxima_is_bit_exact(n_rows, vocab):
    # bf16 MFMA path: above 16384 logits the lm-head epilogue hands the sampler per-strip maxima instead of a pass
    # over the logits (8192: a row in one workgroup, which takes its maximum itself; 24608: 24 MB of weights, which
    # up to 64 rows go past the caches).  Given the step's draws and its logits (rl_debug_logits: one row at a time; its
    # product may add up in another order, which moves the boundaries of a draw by some 1e-7 of the total weight), the
    # ids must be the oracle sampler's, for every instance of the lm-head kernel (1, 2, 4 row blocks; two row tiles).
    shape = SHAPES["small-d128"].replace(vocab=vocab)
    assert vocab * shape.hidden * 2 >= 24 << 20 or vocab != 24608
    blob = make_weight_blob(shape, seed=5, weight_std=0.05, gain_std=0.1)
    g = rl.RolloutEngine(blob, max_context=64, max_trajectories=n_rows, kv_pool_pages=n_rows * 4)
    rng = np.random.default_rng(n_rows)
    ids = np.arange(n_rows, dtype=np.int32) * 3 + 1
    lens = rng.integers(5, 30, n_rows)
    g.append_observation(ids, rng.integers(0, shape.vocab, int(lens.sum())), lens)
    probe = sorted(set([0, 1, n_rows // 2, n_rows - 1]))
    for step, T in enumerate([1.0, 0.7, 1.0, 0.0]):
        z = {k: g.debug_logits(int(ids[k])) for k in probe}
        out, lps = g.decode_step(ids, T, 77)
        for k in probe:
            tok, lp = sample_token(z[k], T, uniform_u32(77, int(ids[k]), int(lens[k]) + step))
            assert out[k] == tok and abs(lps[k] - lp) < TOL_FP32, (n_rows, step, k)


@pytest.mark.parametrize("name,flags,steps", [("tiny", 0, 40), ("tiny-bf16", 0, 21), ("small-d128", 0, 70),
                                              ("small-d128", 2, 37), ("small-d128", 4, 37), ("small-g8", 0, 19),
                                              ("tiny", 0, 1030)])
def test_decode_steps_equals_the_single_steps_bit_for_bit(name, flags, steps):
    # rl_decode_steps is n_steps single steps in one call (the sampled token feeds the next step on
    # the device, the host stages ahead): ids, log-probs, records, page indices and the free list
    # must be identical, also across page boundaries, more steps than staging regions (64), more
    # than one chunk of steps (1024), a forked group, and a following append + second call
    shape = SHAPES[name]
    blob = make_weight_blob(shape, seed=61, weight_std=0.05, gain_std=0.1)
    kw = dict(max_context=1400 if steps > 1000 else 256, max_trajectories=8,
              kv_pool_pages=8 * 90 if steps > 1000 else 8 * 18, flags=flags)
    a, b = rl.RolloutEngine(blob, **kw), rl.RolloutEngine(blob, **kw)
    rng = np.random.default_rng(steps)
    lens = [33, 5, 16, 47]
    toks = rng.integers(0, shape.vocab, sum(lens))
    ids = [3, 0, 9, 4, 12, 13]
    for e in (a, b):
        e.append_observation(ids[:4], toks, lens)
        e.fork(3, [12, 13])
    single = [a.decode_step(ids, 1.0, 5) for _ in range(steps)]
    multi_ids, multi_lps = b.decode_steps(ids, steps, 1.0, 5)
    assert multi_ids.shape == (steps, 6)
    assert np.array_equal(multi_ids, np.stack([x[0] for x in single]))
    assert np.array_equal(multi_lps, np.stack([x[1] for x in single]))
    obs = rng.integers(0, shape.vocab, 23)
    for e in (a, b):
        e.append_observation([9, 13], obs, [20, 3])
    s2 = [a.decode_step([13, 9, 0], 0.7 if k % 2 else 0.0, 8) for k in range(4)]
    m0 = b.decode_steps([13, 9, 0], 1, 0.0, 8)
    m1 = b.decode_steps([13, 9, 0], 1, 0.7, 8)
    m2 = b.decode_steps([13, 9, 0], 1, 0.0, 8)
    m3 = b.decode_steps([13, 9, 0], 1, 0.7, 8)
    for k, mm in enumerate((m0, m1, m2, m3)):
        assert np.array_equal(mm[0][0], s2[k][0]) and np.array_equal(mm[1][0], s2[k][1])
    for t in ids:
        ra, rb = a.traj_read(t), b.traj_read(t)
        assert all(np.array_equal(x, y) for x, y in zip(ra, rb)), t
    assert a.n_free_pages() == b.n_free_pages()
    assert np.array_equal(a.debug_logits(9), b.debug_logits(9))


def test_decode_steps_is_all_or_nothing():
    shape = SHAPES["tiny"].replace(n_layers=1)
    blob = make_weight_blob(shape, seed=4)
    g = rl.RolloutEngine(blob, max_context=48, max_trajectories=3, kv_pool_pages=4)
    g.append_observation([1, 2], np.arange(20), [17, 3])
    before = [g.traj_read(t) for t in (1, 2)]
    for args, code in [(([1, 2], 32, 1.0, 0), -6),        # trajectory 1 would reach 49 tokens
                       (([1, 2], 30, 1.0, 0), -5),        # 47 and 33 tokens need 3 + 3 pages, 4 exist
                       (([1, 7], 2, 1.0, 0), -2), (([1, 1], 2, 1.0, 0), -3),
                       (([1, 2], -1, 1.0, 0), -1), (([1, 2], 2, -1.0, 0), -1)]:
        with pytest.raises(rl.RolloutError) as ei:
            g.decode_steps(*args)
        assert ei.value.code == code, args
        for t, old in zip((1, 2), before):
            assert all(np.array_equal(x, y) for x, y in zip(g.traj_read(t), old))
        assert g.n_free_pages() == 1
    out, lps = g.decode_steps([1, 2], 0, 1.0, 0)
    assert out.shape == (0, 2) and g.n_free_pages() == 1
    out, lps = g.decode_steps([], 5, 1.0, 0)
    assert out.shape == (5, 0)
    out, lps = g.decode_steps([2, 1], 14, 1.0, 0)          # 17 + 31 tokens: exactly the 4 pages
    assert out.shape == (14, 2) and g.n_free_pages() == 0 and g.traj_info(1) == (31, 2)


# ---- cfg1: tiny fp32 decoder, free-running greedy rollout --------------------------------
def test_cfg1_fp32_free_running_matches_oracle_golden():
    shape = SHAPES["tiny"]
    blob = make_weight_blob(shape, seed=1)
    w = make_workload("cfg1", shape.vocab)
    g = rl.RolloutEngine(blob, max_context=128, max_trajectories=8, kv_pool_pages=64)
    out = replay(g, w)
    gold = json.load(open(os.path.join(os.path.dirname(__file__), "golden", "cfg1_oracle.json")))
    for t in range(4):
        assert out[t][0] == gold["ids"][str(t)]
        assert np.abs(np.array(out[t][1]) - np.array(gold["logprobs"][str(t)])).max() < TOL_FP32


def test_cfg1_fp32_lockstep_logits_and_state():
    shape = SHAPES["tiny"]
    blob = make_weight_blob(shape, seed=1, weight_std=0.05, gain_std=0.1)
    w = make_workload("cfg1", shape.vocab)
    o, g = _pair(shape, blob, max_context=128, kv_pool_pages=64)
    r = run_lockstep(o, g, w, check_logits_every=5, logit_rows=4)
    assert r["n_decoded"] == 192
    assert r["max_logp_err"] < TOL_FP32 and r["max_logit_err"] < TOL_FP32


# ---- bf16 paths --------------------------------------------------------------------------
def _bf16_workload(vocab):
    # 6 trajectories in 2 groups of 3 sharing a 45-token prompt, 2 turns of (7 decoded, 21 appended):
    # several pages, a ragged tail, a fork with a partial last page
    return uniform_turns("bf16-small", vocab, 6, 45, 2, 7, 21, 1.0, group_size=3, final_release=False)


@pytest.mark.parametrize("name,flags", [("tiny-bf16", 0), ("small-d128", 1), ("small-d128", 0),
                                        ("small-g2", 0), ("small-g1", 0), ("small-g8", 0)])
def test_bf16_lockstep(name, flags):
    shape = SHAPES[name]
    blob = make_weight_blob(shape, seed=2, weight_std=0.03, gain_std=0.1)
    o, g = _pair(shape, blob, flags=flags)
    r = run_lockstep(o, g, _bf16_workload(shape.vocab), check_logits_every=3, logit_rows=6)
    print(name, flags, r)
    assert r["max_logp_err"] < TOL_BF16 and r["max_logit_err"] < TOL_BF16, r
    rec = g.recompute_logprobs([0, 4], 1.0)
    ref = o.recompute_logprobs([0, 4], 1.0)
    assert rec.shape == ref.shape and np.abs(rec - ref).max() < TOL_BF16
    m = np.concatenate([o.traj_read(0)[1], o.traj_read(4)[1]])
    assert np.all(rec[m == 1] == 0.0)


@pytest.mark.parametrize("name,group,prompt", [("small-d128", 5, 200), ("small-g2", 3, 150),
                                               ("small-g1", 4, 133), ("small-g8", 5, 300)])
def test_shared_prefix_decode_attention(name, group, prompt):
    # forked groups whose shared prompt spans many pages: with the shared-prefix flag the decode
    # attention reads those pages once per block of 16/G members (blocks of several members, a lone
    # member, a prefix long enough to be cut into parts) and merges with each member's own pages
    shape = SHAPES[name]
    blob = make_weight_blob(shape, seed=5, weight_std=0.03, gain_std=0.1)
    w = uniform_turns("shared", shape.vocab, 2 * group, prompt, 2, 6, 19, 1.0, group_size=group,
                      final_release=False)
    kw = dict(max_context=512, max_trajectories=16, kv_pool_pages=400)
    o = OracleEngine(blob, **kw)
    g = rl.RolloutEngine(blob, flags=rl.FLAG_SHARED_PREFIX_ATTENTION, **kw)
    r = run_lockstep(o, g, w, check_logits_every=2, logit_rows=2 * group)
    print(name, r)
    assert r["max_logp_err"] < TOL_BF16 and r["max_logit_err"] < TOL_BF16, r
    # same calls without the flag: same integer state, log-probs within the bf16 tolerance
    p = rl.RolloutEngine(blob, **kw)
    for ev in w.events:
        if ev[0] == "append":
            p.append_observation(ev[1], ev[2], ev[3])
        elif ev[0] == "fork":
            p.fork(ev[1], ev[2])
        elif ev[0] == "decode":
            p.decode_step_forced(ev[1], ev[2], np.array([g.traj_read(int(t))[0][p.traj_info(int(t))[0]]
                                                         for t in ev[1]], np.int32))
    for t in range(2 * group):
        a, b = g.traj_read(t), p.traj_read(t)
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]) and np.array_equal(a[3], b[3])
        assert np.abs(a[2] - b[2]).max() < TOL_BF16


def _replay_fused(o, g, w):
    """Like run_lockstep, but an append event directly followed by a decode event goes to the GPU
    engine as ONE call (rl_decode_step_forced_with_appends); the oracle makes the two calls."""
    evs, i, max_lp, fused = w.events, 0, 0.0, 0
    live = set()
    while i < len(evs):
        ev = evs[i]
        if ev[0] == "append" and i + 1 < len(evs) and evs[i + 1][0] == "decode":
            dv = evs[i + 1]
            o.append_observation(ev[1], ev[2], ev[3])
            ids, lps = o.decode_step(dv[1], dv[2], dv[3])
            glp = g.decode_step_forced_with_appends(ev[1], ev[2], ev[3], dv[1], dv[2], ids)
            max_lp = max(max_lp, float(np.abs(glp - lps).max()))
            live.update(int(t) for t in ev[1])
            fused += 1
            i += 2
            continue
        if ev[0] == "append":
            o.append_observation(ev[1], ev[2], ev[3])
            g.append_observation(ev[1], ev[2], ev[3])
            live.update(int(t) for t in ev[1])
        elif ev[0] == "fork":
            o.fork(ev[1], ev[2])
            g.fork(ev[1], ev[2])
            live.update(int(t) for t in ev[2])
        elif ev[0] == "decode":
            ids, lps = o.decode_step(ev[1], ev[2], ev[3])
            glp = g.decode_step_forced(ev[1], ev[2], ids)
            max_lp = max(max_lp, float(np.abs(glp - lps).max()))
        elif ev[0] == "release":
            for t in ev[1]:
                compare_records(o, g, int(t))
            o.release(ev[1])
            g.release(ev[1])
            live.difference_update(int(t) for t in ev[1])
        assert o.n_free_pages() == g.n_free_pages()
        i += 1
    for t in sorted(live):
        compare_records(o, g, t)
    return max_lp, fused


@pytest.mark.parametrize("name,tol", [("tiny", TOL_FP32), ("tiny-bf16", TOL_BF16), ("small-d128", TOL_BF16),
                                      ("small-g2", TOL_BF16)])
def test_decode_step_with_appends_equals_the_two_calls(name, tol):
    # Update + Generate in one forward pass: appended rows ride behind the decode rows; trajectories
    # that get an observation decode in the same call.  Uniform turns (everybody appends, then
    # everybody decodes) and ragged turns (a few append while the others keep decoding).
    shape = SHAPES[name]
    blob = make_weight_blob(shape, seed=7, weight_std=0.03, gain_std=0.1)
    for w in (_bf16_workload(shape.vocab),
              ragged_turns("ragged", shape.vocab, 7, 19, (1, 4), (2, 9), (3, 37), 200, 1.0)):
        o, g = _pair(shape, blob)
        max_lp, fused = _replay_fused(o, g, w)
        print(name, w.name, max_lp, fused)
        assert fused >= 1 and max_lp < tol


def test_decode_step_with_appends_overflow_and_errors():
    shape = SHAPES["small-d128"]
    blob = make_weight_blob(shape, seed=7, weight_std=0.03, gain_std=0.1)
    # more appended rows than one pass holds: the append is prefilled on its own first
    o, g = _pair(shape, blob, max_context=1024, max_trajectories=4, kv_pool_pages=200, max_batch_rows=128)
    rng = np.random.default_rng(2)
    t0 = rng.integers(0, shape.vocab, 40)
    for e in (o, g):
        e.append_observation([0, 1], t0, [25, 15])
    big = rng.integers(0, shape.vocab, 300)
    o.append_observation([1], big, [300])
    ids, lps = o.decode_step([0, 1], 1.0, 4)
    glp = g.decode_step_forced_with_appends([1], big, [300], [0, 1], 1.0, ids)
    assert np.abs(glp - lps).max() < TOL_BF16
    for t in (0, 1):
        compare_records(o, g, t)
        assert np.abs(o.debug_logits(t) - g.debug_logits(t)).max() < TOL_BF16
    # append part valid, decode part invalid: the append takes effect, the error is the decode's
    more = rng.integers(0, shape.vocab, 9)
    with pytest.raises(rl.RolloutError) as ei:
        g.decode_step_with_appends([0], more, [9], [0, 77], 1.0, 4)
    assert ei.value.code == -2
    o.append_observation([0], more, [9])
    compare_records(o, g, 0)
    assert np.abs(o.debug_logits(0) - g.debug_logits(0)).max() < TOL_BF16
    # append part invalid: nothing changes
    with pytest.raises(rl.RolloutError) as ei:
        g.decode_step_with_appends([0], [shape.vocab], [1], [0], 1.0, 4)
    assert ei.value.code == -4
    compare_records(o, g, 0)
    # empty append list = plain decode step; empty decode list = plain append
    top2 = [np.sort(o.debug_logits(t))[-2:] for t in (0, 1)]
    ids, lps = o.decode_step([0, 1], 0.0, 4)
    gi, gl = g.decode_step_with_appends([], [], [], [0, 1], 0.0, 4)
    for k in range(2):
        # the arg-max is decided by the logits: it must agree wherever the oracle's two best logits
        # are further apart than both sides' errors can bridge, and then the log-probs must agree too
        if top2[k][1] - top2[k][0] > 2 * TOL_BF16:
            assert gi[k] == ids[k]
        if gi[k] == ids[k]:
            assert abs(gl[k] - lps[k]) < TOL_BF16
    assert any(top2[k][1] - top2[k][0] > 2 * TOL_BF16 for k in range(2))
    g2 = rl.RolloutEngine(blob, max_context=256, max_trajectories=4, kv_pool_pages=64)
    o2 = OracleEngine(blob, max_context=256, max_trajectories=4, kv_pool_pages=64)
    o2.append_observation([3], t0, [40])
    out = g2.decode_step_with_appends([3], t0, [40], [], 1.0, 4)
    assert len(out[0]) == 0
    compare_records(o2, g2, 3)
    assert np.abs(o2.debug_logits(3) - g2.debug_logits(3)).max() < TOL_BF16


@pytest.mark.parametrize("name,flags,rows,seed", [("small-d128", 0, 128, 1), ("small-d128", 2, 0, 2),
                                                 ("small-g2", 2, 256, 3), ("tiny", 0, 0, 4),
                                                 ("tiny-bf16", 0, 128, 5), ("small-d128", 4, 128, 6),
                                                 ("small-g8", 6, 0, 7)])
def test_random_call_sequences(name, flags, rows, seed):
    # random interleavings of every entry point (append, decode, Update+Generate in one pass, fork,
    # release, log-prob recompute) on both engines: integer state identical after every call,
    # log-probs / logits within tolerance.  Small row budgets force multi-pass prefill and the
    # fallback of the mixed pass; flag 2 = shared-prefix decode attention, flag 4 = 8-bit cache
    # (oracle with the same cache rule; tolerance from the error model's figure for these shapes).
    shape = SHAPES[name]
    tol = TOL_FP32 if shape.weight_dtype == 0 else TOL_BF16
    if flags & 4:
        tol = 8.0 * 0.018
    blob = make_weight_blob(shape, seed=20 + seed, weight_std=0.03, gain_std=0.1)
    max_ctx, max_traj = 448, 8
    kw = dict(max_context=max_ctx, max_trajectories=max_traj, kv_pool_pages=max_traj * (max_ctx // 16 + 1))
    o = OracleEngine(blob, kv_cache_dtype="fp8_e4m3" if flags & 4 else None, **kw)
    g = rl.RolloutEngine(blob, flags=flags, max_batch_rows=rows, **kw)
    rng = np.random.default_rng(seed)
    length, next_id = {}, 0

    def pick(ids, lo=1, hi=4):
        ids = list(ids)
        k = int(rng.integers(lo, min(hi, len(ids)) + 1))
        return [int(x) for x in rng.choice(ids, size=k, replace=False)]

    def draw_append():
        cand = [t for t in length if length[t] < max_ctx - 80]
        ids = pick(cand, 1, 3) if cand and rng.random() < 0.7 else []
        nonlocal next_id
        if len(length) + 1 <= max_traj and (not ids or rng.random() < 0.4):
            ids.append(next_id)
            next_id += 1
        lens = [int(rng.integers(0, 70)) if t in length else int(rng.integers(1, 150)) for t in ids]
        toks = rng.integers(0, shape.vocab, sum(lens))
        return ids, toks, lens

    worst = 0.0
    for step in range(70):
        live = [t for t in length if length[t] > 0]
        op = rng.choice(["append", "decode", "mixed", "fork", "release", "recompute", "logits"],
                        p=[0.2, 0.3, 0.2, 0.1, 0.06, 0.07, 0.07])
        if op == "append" or not live:
            ids, toks, lens = draw_append()
            if not ids:
                continue
            o.append_observation(ids, toks, lens)
            g.append_observation(ids, toks, lens)
            for t, n in zip(ids, lens):
                length[t] = length.get(t, 0) + n
        elif op == "decode":
            ids = [t for t in pick(live) if length[t] < max_ctx - 4]
            for _ in range(int(rng.integers(1, 4))):
                if not ids:
                    break
                T = float(rng.choice([1.0, 0.7, 0.0]))
                tok, lps = o.decode_step(ids, T, 9)
                glp = g.decode_step_forced(ids, T, tok)
                worst = max(worst, float(np.abs(glp - lps).max()))
                for t in ids:
                    length[t] += 1
        elif op == "mixed":
            ids, toks, lens = draw_append()
            for t, n in zip(ids, lens):
                length[t] = length.get(t, 0) + n
            dec = [t for t in length if 0 < length[t] < max_ctx - 4]
            dec = pick(dec) if dec else []
            o.append_observation(ids, toks, lens)
            tok, lps = o.decode_step(dec, 1.0, 9)
            glp = g.decode_step_forced_with_appends(ids, toks, lens, dec, 1.0, tok)
            if len(dec):
                worst = max(worst, float(np.abs(glp - lps).max()))
            for t in dec:
                length[t] += 1
        elif op == "fork" and len(length) + 2 <= max_traj:
            src = pick(live, 1, 1)[0]
            dst = [next_id, next_id + 1][:int(rng.integers(1, 3))]
            next_id += len(dst)
            o.fork(src, dst)
            g.fork(src, dst)
            for d in dst:
                length[d] = length[src]
        elif op == "release":
            ids = pick(list(length), 1, 2)
            for t in ids:
                compare_records(o, g, t)
            o.release(ids)
            g.release(ids)
            for t in ids:
                del length[t]
        elif op == "recompute":
            ids = pick(live, 1, 3)
            T = float(rng.choice([1.0, 0.5]))
            a, b = o.recompute_logprobs(ids, T), g.recompute_logprobs(ids, T)
            assert a.shape == b.shape
            worst = max(worst, float(np.abs(a - b).max()))
        elif op == "logits":
            t = pick(live, 1, 1)[0]
            worst = max(worst, float(np.abs(o.debug_logits(t) - g.debug_logits(t)).max()))
        assert o.n_free_pages() == g.n_free_pages(), (step, op)
        assert worst < tol, (step, op, worst)
    for t in length:
        compare_records(o, g, t)
    print(name, flags, rows, "worst", worst, "live", len(length))


def test_mfma_long_context_split_attention_and_chunked_prefill():
    # context long enough that decode attention is split over several workgroups, appended with a
    # row budget that forces several prefill passes and splits a trajectory across passes
    shape = SHAPES["small-d128"]
    blob = make_weight_blob(shape, seed=3, weight_std=0.03, gain_std=0.1)
    o, g = _pair(shape, blob, max_context=2048, max_trajectories=4, kv_pool_pages=200, max_batch_rows=384)
    rng = np.random.default_rng(1)
    lens = [1700, 523]      # 107 pages against 33: the planner cuts the long context into parts
    toks = rng.integers(0, shape.vocab, sum(lens))
    for e in (o, g):
        e.append_observation([0, 1], toks, lens)
    for step in range(3):
        for t in (0, 1):
            assert np.abs(o.debug_logits(t) - g.debug_logits(t)).max() < TOL_BF16
        ids, lps = o.decode_step([0, 1], 1.0, 5)
        glp = g.decode_step_forced([0, 1], 1.0, ids)
        assert np.abs(glp - lps).max() < TOL_BF16
    for t in (0, 1):
        compare_records(o, g, t)


@pytest.mark.parametrize("name", ["small-d128", "small-g1", "small-g2", "small-g8"])
def test_chunked_prefill_page_pair_stage_and_item_edges(name):
    # the prefill kernel consumes pages in pairs from LDS stages of four pages, in items of
    # 4 waves x 2 blocks x 16/G rows: append lengths and starting positions chosen so that contexts
    # end on odd and even page counts, on and next to stage boundaries (64 tokens), items are
    # ragged (1 row, one row more or less than a block / an item) and later chunks start at
    # positions that are not page aligned, on top of keys cached by earlier chunks
    shape = SHAPES[name]
    blob = make_weight_blob(shape, seed=11, weight_std=0.03, gain_std=0.1)
    o, g = _pair(shape, blob, max_context=512, max_trajectories=8, kv_pool_pages=256)
    rng = np.random.default_rng(4)
    traj = [0, 1, 2, 3, 4, 5]
    rounds = [[1, 15, 17, 33, 64, 65], [63, 1, 47, 31, 1, 130], [2, 97, 16, 129, 66, 3]]
    for lens in rounds:
        toks = rng.integers(0, shape.vocab, sum(lens))
        for e in (o, g):
            e.append_observation(traj, toks, lens)
        worst = max(float(np.abs(o.debug_logits(t) - g.debug_logits(t)).max()) for t in traj)
        assert worst < TOL_BF16, (name, lens, worst)
        ids, lps = o.decode_step(traj, 1.0, 9)
        glp = g.decode_step_forced(traj, 1.0, ids)
        assert np.abs(glp - lps).max() < TOL_BF16
    for t in traj:
        compare_records(o, g, t)
    # the masked log-prob pass walks the same contexts in one teacher-forced prefill
    ro, rg = o.recompute_logprobs(traj, 1.0), g.recompute_logprobs(traj, 1.0)
    assert np.abs(np.asarray(ro) - np.asarray(rg)).max() < TOL_BF16


def test_ragged_workload_integer_state_bit_exact():
    # cfg4 shape of workload (ragged turns, shrinking batch) at reduced lengths, tiny fp32 model
    shape = SHAPES["tiny"].replace(n_layers=1)
    blob = make_weight_blob(shape, seed=4, weight_std=0.05, gain_std=0.1)
    w = ragged_turns("ragged", shape.vocab, 12, 20, (1, 4), (2, 12), (3, 40), 160, 1.0)
    o, g = _pair(shape, blob, max_context=160, max_trajectories=12, kv_pool_pages=100)
    r = run_lockstep(o, g, w, check_logits_every=7)
    assert r["max_logp_err"] < TOL_FP32 and r["max_logit_err"] < TOL_FP32
    assert g.n_free_pages() == 100


def test_error_codes_and_all_or_nothing():
    shape = SHAPES["tiny"].replace(n_layers=1)
    blob = make_weight_blob(shape, seed=4)
    kw = dict(max_context=48, max_trajectories=3, kv_pool_pages=4)
    o, g = OracleEngine(blob, **kw), rl.RolloutEngine(blob, **kw)
    for e in (o, g):
        e.append_observation([1], [1, 2, 3], [3])
    cases = [
        lambda e: e.append_observation([1, 1], [1, 2], [1, 1]),
        lambda e: e.append_observation([1], [4096], [1]),
        lambda e: e.append_observation([-4], [1], [1]),
        lambda e: e.append_observation([1], [5] * 46, [46]),
        lambda e: e.append_observation([2, 3], [5] * 64, [32, 32]),
        lambda e: e.append_observation([2, 3, 4], [5] * 3, [1, 1, 1]),
        lambda e: e.decode_step([7], 1.0, 0),
        lambda e: e.decode_step([1, 1], 1.0, 0),
        lambda e: e.decode_step([1], -1.0, 0),
        lambda e: e.release([1, 8]),
        lambda e: e.fork(8, [2]),
        lambda e: e.fork(1, [1]),
        lambda e: e.traj_read(8),
        lambda e: e.decode_step_forced([1], 1.0, [4096]),
    ]
    for fn in cases:
        with pytest.raises(OracleError) as eo:
            fn(o)
        with pytest.raises(rl.RolloutError) as eg:
            fn(g)
        assert eo.value.code == eg.value.code
        compare_records(o, g, 1)
        assert o.n_free_pages() == g.n_free_pages() == 3
    for e in (o, g):
        e.append_observation([2], [], [0])
    with pytest.raises(rl.RolloutError) as eg:
        g.decode_step([2], 1.0, 0)
    assert eg.value.code == -7
    assert g.traj_info(2) == (0, 0)


def test_batch_composition_does_not_change_ids():
    # draws are keyed by (trajectory, position): a trajectory decoded alone or inside a batch, in any
    # order, yields the same ids (fp32 mode, deterministic kernels)
    shape = SHAPES["tiny"].replace(n_layers=1)
    blob = make_weight_blob(shape, seed=6, weight_std=0.05, gain_std=0.1)
    rng = np.random.default_rng(2)
    prompts = {i: rng.integers(0, shape.vocab, 5 + 4 * i) for i in range(4)}
    kw = dict(max_context=64, max_trajectories=4, kv_pool_pages=16)
    solo = {}
    for i, p in prompts.items():
        g = rl.RolloutEngine(blob, **kw)
        g.append_observation([i], p, [len(p)])
        solo[i] = [g.decode_step([i], 1.0, 9)[0][0] for _ in range(4)]
    g = rl.RolloutEngine(blob, **kw)
    order = [2, 0, 3, 1]
    g.append_observation(order, np.concatenate([prompts[i] for i in order]), [len(prompts[i]) for i in order])
    for s in range(4):
        ids, _ = g.decode_step(order, 1.0, 9)
        assert [int(x) for x in ids] == [solo[i][s] for i in order]


@pytest.mark.parametrize("kv", [None, "fp8_e4m3"])
def test_full_size_cfg3_launch_configuration_sampled_trajectory(kv):
    """Qwen3-4B shape, 128 trajectories in 16 forked groups (the launch configuration bench.py
    times: same batch rows, GEMM split plan and attention grid), contexts short enough that the
    oracle can follow ONE trajectory (a forked group member) token by token.  The oracle samples
    that trajectory's ids; the GPU is teacher-forced with them (other rows get seeded ids)."""
    shape = SHAPES["qwen3-4b"]
    blob = make_weight_blob(shape, seed=1)
    n_traj, group, prompt, obs = 128, 8, 80, 24
    check = 9                                       # member 1 of group 1
    g = rl.RolloutEngine(blob, max_context=256, max_trajectories=n_traj, kv_pool_pages=n_traj * 10,
                         flags=rl.FLAG_FP8_KV_CACHE if kv else 0)      # kv: the 8-bit cache variant
    o = OracleEngine(blob, max_context=256, max_trajectories=2, kv_pool_pages=32, kv_cache_dtype=kv)
    rng = np.random.default_rng(2)
    leaders = np.arange(0, n_traj, group, dtype=np.int32)
    prompts = rng.integers(0, shape.vocab, (len(leaders), prompt), dtype=np.int32)
    g.append_observation(leaders, prompts.reshape(-1), np.full(len(leaders), prompt, np.int32))
    for L in leaders:
        g.fork(int(L), np.arange(L + 1, L + group, dtype=np.int32))
    o.append_observation([check], prompts[check // group], [prompt])
    ids = np.arange(n_traj, dtype=np.int32)
    dlp = []
    chunk = None
    for turn in range(2):
        for step in range(3):
            tok, lp = o.decode_step([check], 1.0, 3)
            forced = rng.integers(0, shape.vocab, n_traj, dtype=np.int32)
            forced[check] = tok[0]
            if chunk is not None:
                # first step after the observation: Update + Generate in one pass (3200 rows)
                glp = g.decode_step_forced_with_appends(ids, chunk.reshape(-1), np.full(n_traj, obs, np.int32),
                                                        ids, 1.0, forced)
                chunk = None
            else:
                glp = g.decode_step_forced(ids, 1.0, forced)
            dlp.append(float(glp[check]) - float(lp[0]))
        if turn == 0:
            chunk = rng.integers(0, shape.vocab, (n_traj, obs), dtype=np.int32)
            o.append_observation([check], chunk[check], [obs])
    zo, zg = o.debug_logits(check), g.debug_logits(check)
    # At this depth and width bf16 rounding of activations and cached keys / values alone moves the
    # logits by more than the 3e-2 absolute bound (which the small shapes above meet): measure what
    # the arithmetic type costs on this very trajectory and hold the GPU to that (tests/tolerances.py)
    from oracle.bf16_error_model import forward_bf16_model
    zm = forward_bf16_model(o.model, o.traj_read(check)[0])[-1]
    fig = check_against_rounding_model(zg, zo, zm, dlp, f"4B shape, cache {kv}")
    print("full-size:", fig, "logit std", float(zo.std()))
    # masked log-prob pass at the full vocabulary (log-softmax reduced in the lm-head epilogue)
    ro, rg = o.recompute_logprobs([check], 1.0), g.recompute_logprobs([check], 1.0)
    assert ro.shape == rg.shape and np.count_nonzero(rg) == 6
    assert np.abs(ro - rg).max() < fig["dlogp_bound"]
    # the recomputed values against the log-probs the decode steps returned: two GPU schedules, each
    # within the bound of the oracle, so their difference has sqrt(2) times the spread
    gen = g.traj_read(check)[2]
    sampled = g.traj_read(check)[1] == 0
    assert np.abs(rg - gen)[sampled].max() < np.sqrt(2.0) * fig["dlogp_bound"]
    to, mo, _, po = o.traj_read(check)
    tg, mg, _, pg = g.traj_read(check)
    assert np.array_equal(to, tg) and np.array_equal(mo, mg)
    # group 1's trajectories took their pages in call order: 5 shared prompt pages, then own pages
    assert list(pg[:4]) == list(g.traj_read(8)[3][:4])
    g.close()


def test_bf16_path_is_bit_reproducible_and_empty_calls_are_noops():
    # split-K partial sums and context parts are combined in a fixed order: two engines fed the same
    # calls return bit-identical ids, log-probs and logits
    shape = SHAPES["small-d128"]
    blob = make_weight_blob(shape, seed=8, weight_std=0.03, gain_std=0.1)
    rng = np.random.default_rng(3)
    toks = rng.integers(0, shape.vocab, 300 + 77)
    runs = []
    for _ in range(2):
        g = rl.RolloutEngine(blob, max_context=512, max_trajectories=4, kv_pool_pages=80)
        g.append_observation([], [], [])
        g.append_observation([5, 6], toks, [300, 77])
        out = [g.decode_step([5, 6], 1.0, 11) for _ in range(5)]
        ids0, lps0 = g.decode_step([], 1.0, 11)
        assert len(ids0) == 0 and len(lps0) == 0
        g.release([])
        runs.append((np.concatenate([o[0] for o in out]), np.concatenate([o[1] for o in out]),
                     g.debug_logits(5), g.recompute_logprobs([6, 5], 1.0)))
        g.close()
    for a, b in zip(*runs):
        assert np.array_equal(a, b)


def test_recompute_over_several_lm_head_passes():
    # more rows than one lm-head pass holds: the recompute walks the rows in blocks
    shape = SHAPES["small-d128"]
    blob = make_weight_blob(shape, seed=9, weight_std=0.03, gain_std=0.1)
    o, g = _pair(shape, blob, max_context=512, max_trajectories=4, kv_pool_pages=80)
    rng = np.random.default_rng(4)
    lens = [230, 190]
    toks = rng.integers(0, shape.vocab, sum(lens))
    for e in (o, g):
        e.append_observation([0, 1], toks, lens)
    for _ in range(3):
        ids, _ = o.decode_step([0, 1], 1.0, 2)
        g.decode_step_forced([0, 1], 1.0, ids)
    ref, rec = o.recompute_logprobs([0, 1], 1.0), g.recompute_logprobs([0, 1], 1.0)
    assert rec.shape == ref.shape == (sum(lens) + 6,)
    assert np.abs(rec - ref).max() < TOL_BF16
    assert np.count_nonzero(rec) == 6 and np.count_nonzero(ref) == 6


def test_fused_logprob_pass_many_sampled_rows_and_temperature():
    # the masked log-prob pass gathers the rows whose target was sampled, runs the lm-head with the
    # log-softmax reduced in its epilogue and never stores logits: > 128 sampled rows (several row
    # tiles, ragged tail), interleaved with appended chunks, at a temperature other than 1
    shape = SHAPES["small-d128"]
    blob = make_weight_blob(shape, seed=12, weight_std=0.03, gain_std=0.1)
    o, g = _pair(shape, blob, max_context=512, max_trajectories=4, kv_pool_pages=100)
    rng = np.random.default_rng(6)
    toks0 = rng.integers(0, shape.vocab, 50)
    obs = rng.integers(0, shape.vocab, 2 * 19)
    for e in (o, g):
        e.append_observation([3, 1], toks0, [33, 17])
    for turn in range(2):
        for _ in range(37):
            ids, lps = o.decode_step([3, 1], 0.7, 21)
            glp = g.decode_step_forced([3, 1], 0.7, ids)
            assert np.abs(glp - lps).max() < TOL_BF16
        if turn == 0:
            for e in (o, g):
                e.append_observation([3, 1], obs, [19, 19])
    ref, rec = o.recompute_logprobs([1, 3], 0.7), g.recompute_logprobs([1, 3], 0.7)
    assert rec.shape == ref.shape == (50 + 38 + 4 * 37,)
    assert np.abs(rec - ref).max() < TOL_BF16
    mask = np.concatenate([o.traj_read(1)[1], o.traj_read(3)[1]])
    assert np.count_nonzero(mask == 0) == 148 and np.all(rec[mask == 1] == 0.0)
    # the recomputed values are the log-probs reported at generation time
    gen = np.concatenate([g.traj_read(1)[2], g.traj_read(3)[2]])
    assert np.abs(rec - gen)[mask == 0].max() < TOL_BF16
    # greedy convention: temperature 0 reports the T = 1 distribution
    assert np.array_equal(g.recompute_logprobs([1, 3], 0.0), g.recompute_logprobs([1, 3], 1.0))


def test_full_size_cfg2_shape_sampled_trajectories():
    """Qwen3-0.6B shape (GQA group 2, 28 layers), 64 trajectories as in cfg2: two trajectories are
    followed by the oracle, teacher-forcing the GPU with the oracle's ids."""
    shape = SHAPES["qwen3-0.6b"]
    blob = make_weight_blob(shape, seed=1)
    n_traj, prompt, obs = 64, 40, 12
    checks = [3, 41]
    g = rl.RolloutEngine(blob, max_context=128, max_trajectories=n_traj, kv_pool_pages=n_traj * 9)
    o = OracleEngine(blob, max_context=128, max_trajectories=2, kv_pool_pages=32)
    rng = np.random.default_rng(5)
    ids = np.arange(n_traj, dtype=np.int32)
    prompts = rng.integers(0, shape.vocab, (n_traj, prompt), dtype=np.int32)
    g.append_observation(ids, prompts.reshape(-1), np.full(n_traj, prompt, np.int32))
    o.append_observation(checks, prompts[checks].reshape(-1), [prompt, prompt])
    dlp = []
    for turn in range(2):
        for step in range(3):
            tok, lp = o.decode_step(checks, 1.0, 3)
            forced = rng.integers(0, shape.vocab, n_traj, dtype=np.int32)
            forced[checks] = tok
            glp = g.decode_step_forced(ids, 1.0, forced)
            dlp += list(glp[checks] - lp)
        if turn == 0:
            chunk = rng.integers(0, shape.vocab, (n_traj, obs), dtype=np.int32)
            g.append_observation(ids, chunk.reshape(-1), np.full(n_traj, obs, np.int32))
            o.append_observation(checks, chunk[checks].reshape(-1), [obs, obs])
    from oracle.bf16_error_model import forward_bf16_model
    zo, zg = o.debug_logits(checks[0]), g.debug_logits(checks[0])
    zm = forward_bf16_model(o.model, o.traj_read(checks[0])[0])[-1]
    fig = check_against_rounding_model(zg, zo, zm, dlp, "0.6B shape")
    print("cfg2 shape:", fig)
    for c in checks:      # (page indices differ: the oracle holds only the two checked trajectories)
        to, mo = o.traj_read(c)[:2]
        tg, mg = g.traj_read(c)[:2]
        assert np.array_equal(to, tg) and np.array_equal(mo, mg)
    g.close()


# ---- masked GRPO objective over the cached trajectories -------------------------------------
def _grpo_rollout(o, g, shape, n_groups, G, prompt, turns, seed):
    """Same multi-turn group rollout on both engines (ids taken from the oracle)."""
    rng = np.random.default_rng(seed)
    ids = []
    for q in range(n_groups):
        first = q * G
        toks = rng.integers(0, shape.vocab, prompt + q)
        for e in (o, g):
            e.append_observation([first], toks, [len(toks)])
            if G > 1:
                e.fork(first, list(range(first + 1, first + G)))
        ids += list(range(first, first + G))
    for turn, (n_gen, n_obs) in enumerate(turns):
        act = [i for i in ids if (i + turn) % 3 != 0 or turn == 0]     # some trajectories stop early
        for _ in range(n_gen):
            tok, _ = o.decode_step(act, 1.0, 17)
            g.decode_step_forced(act, 1.0, tok)
        if n_obs:
            lens = [n_obs + (i % 3) for i in act]
            obs = rng.integers(0, shape.vocab, sum(lens))
            for e in (o, g):
                e.append_observation(act, obs, lens)
    return ids


@pytest.mark.parametrize("name,flags,tol,rows,ddof", [
    ("tiny", 0, TOL_FP32, 0, 0), ("tiny-bf16", 0, TOL_BF16, 0, 1), ("small-d128", 0, TOL_BF16, 0, 0),
    ("small-d128", 0, TOL_BF16, 128, 1), ("small-d128", 1, TOL_BF16, 128, 0)])
def test_grpo_objective_matches_oracle(name, flags, tol, rows, ddof):
    shape = SHAPES[name]
    blob = make_weight_blob(shape, seed=14, weight_std=0.03, gain_std=0.1)
    kw = dict(max_context=512, max_trajectories=16, kv_pool_pages=200)
    if rows:
        kw["max_batch_rows"] = rows        # trajectories then span several blocks of the pass
    o, g = _pair(shape, blob, flags=flags, **kw)
    G = 4
    ids = _grpo_rollout(o, g, shape, 3, G, 37, [(9, 11), (6, 20), (12, 0)], seed=8)
    rng = np.random.default_rng(3)
    rewards = rng.random(len(ids)).astype(np.float32)
    rewards[4:8] = 0.5                                       # a group with equal rewards: advantages 0
    base = o.recompute_logprobs(ids, 1.0)
    old = (base + rng.normal(0, 0.3, base.size)).astype(np.float32)     # off-policy: clipping is active
    ref = (base + rng.normal(0, 0.2, base.size)).astype(np.float32)
    for kwargs in (dict(), dict(old_logprobs=old), dict(old_logprobs=old, ref_logprobs=ref)):
        beta = 0.04 if "ref_logprobs" in kwargs else 0.0
        want = o.grpo_objective(ids, G, rewards, 1.0, 0.2, beta, std_ddof=ddof, **kwargs)
        got = g.grpo_objective(ids, G, rewards, 1.0, 0.2, beta, std_ddof=ddof, **kwargs)
        assert got["n_tokens"] == want["n_tokens"] > 0
        assert np.abs(got["advantages"] - want["advantages"]).max() < 1e-12
        assert np.all(got["advantages"][4:8] == 0.0)
        # an error d of a log-prob changes its ratio by a factor e^d and its k3 by about |e^(ref-new) - 1| d
        o_old = old if "old_logprobs" in kwargs else np.concatenate([o.traj_read(i)[2] for i in ids])
        mask = np.concatenate([o.traj_read(i)[1] for i in ids]) == 0
        rho_max = float(np.exp(base - o_old)[mask].max())
        k_max = float(np.abs(np.expm1(ref - base))[mask].max()) if beta else 0.0
        bound = (np.exp(tol) - 1.0) * (np.abs(want["advantages"]).max() * rho_max + beta * (k_max + 1.0)) + 1e-9
        assert abs(got["objective"] - want["objective"]) < bound, (kwargs.keys(), got, want, bound)
        assert abs(got["kl"] - want["kl"]) < (np.exp(tol) - 1.0) * (k_max + 1.0) + 1e-12
        if not kwargs:
            assert abs(got["objective"]) < bound      # on-policy: mean of group-normalised advantages
        again = g.grpo_objective(ids, G, rewards, 1.0, 0.2, beta, std_ddof=ddof, **kwargs)
        assert again["objective"] == got["objective"] and again["kl"] == got["kl"]     # fixed summation order
    # no state change: the cache still decodes like the oracle's
    tok, lp = o.decode_step(ids[:3], 1.0, 5)
    assert np.abs(g.decode_step_forced(ids[:3], 1.0, tok) - lp).max() < tol


def test_grpo_objective_errors():
    shape = SHAPES["tiny"]
    blob = make_weight_blob(shape, seed=14)
    g = rl.RolloutEngine(blob, max_context=64, max_trajectories=8, kv_pool_pages=32)
    g.append_observation([0, 1, 2, 3], np.arange(12), [3, 3, 3, 3])
    g.decode_step([0, 1, 2, 3], 1.0, 1)
    ok = g.grpo_objective([0, 1, 2, 3], 2, [1, 0, 0, 1], 1.0, 0.2, 0.0)
    assert ok["n_tokens"] == 4 and np.allclose(ok["advantages"], [1, -1, -1, 1], atol=1e-5)
    for bad, code in [(dict(traj_ids=[0, 1, 2], rewards=[1, 0, 0]), -1),
                      (dict(traj_ids=[0, 1, 2, 9]), -2),
                      (dict(traj_ids=[0, 1, 1, 2]), -3),
                      (dict(rewards=[1, 0, np.nan, 1]), -1),
                      (dict(clip_eps=-0.1), -1), (dict(beta=-1.0), -1),
                      (dict(group_size=1, std_ddof=1), -1), (dict(std_ddof=2), -1),
                      (dict(temperature=-1.0), -1)]:
        a = dict(traj_ids=[0, 1, 2, 3], group_size=2, rewards=[1, 0, 0, 1], temperature=1.0, clip_eps=0.2, beta=0.0)
        a.update(bad)
        with pytest.raises(rl.RolloutError) as ei:
            g.grpo_objective(**a)
        assert ei.value.code == code, bad
    # trajectories without sampled tokens contribute nothing
    g.append_observation([5, 6], np.arange(8), [4, 4])
    out = g.grpo_objective([5, 6], 2, [1, 0], 1.0, 0.2, 0.0)
    assert out["objective"] == 0.0 and out["n_tokens"] == 0


# ---- 8-bit (E4M3) key / value cache variant --------------------------------------------------
def _fp8_pair(shape, blob, **kw):
    kw.setdefault("max_context", 1024)
    kw.setdefault("max_trajectories", 16)
    kw.setdefault("kv_pool_pages", 256)
    okw = {k: v for k, v in kw.items() if k != "max_batch_rows"}
    return (OracleEngine(blob, kv_cache_dtype="fp8_e4m3", **okw),
            rl.RolloutEngine(blob, flags=rl.FLAG_FP8_KV_CACHE, **kw))


def _fp8_model_rms(o, traj):
    """What the arithmetic type costs on this trajectory under the 8-bit cache: rms distance of the
    logits between the oracle (codes chosen from exact keys / values) and the bf16 error model with
    the same cache rule (codes chosen from bf16-perturbed ones: near a rounding boundary the code
    flips, a full E4M3 step on that element)."""
    from oracle.bf16_error_model import forward_bf16_model
    from oracle.decoder import forward_full
    toks = o.traj_read(traj)[0]
    d = forward_bf16_model(o.model, toks) - forward_full(o.model, toks)
    return float(np.sqrt((d ** 2).mean()))


@pytest.mark.parametrize("name", ["small-d128", "small-g2", "small-g1", "small-g8"])
def test_fp8_kv_cache_lockstep(name):
    shape = SHAPES[name]
    blob = make_weight_blob(shape, seed=2, weight_std=0.03, gain_std=0.1)
    o, g = _fp8_pair(shape, blob)
    r = run_lockstep(o, g, _bf16_workload(shape.vocab), check_logits_every=3, logit_rows=6)
    rms = _fp8_model_rms(o, 0)
    print(name, r, "model rms", rms)
    # the oracle with the cache rule is the reference; the bound is what bf16 arithmetic in front of
    # the 8-bit rounding costs (several times the plain bf16 bound), measured by the error model
    assert r["max_logit_err"] < 8.0 * rms and r["max_logp_err"] < 8.0 * rms, (r, rms)
    rec, ref = g.recompute_logprobs([0, 4], 1.0), o.recompute_logprobs([0, 4], 1.0)
    assert rec.shape == ref.shape and np.abs(rec - ref).max() < 8.0 * rms
    # the variant really is a different contract: it is further from the unquantised oracle
    # than the bf16 bound, and the unquantised GPU path is further from this oracle
    o2, g2 = _pair(shape, blob)
    run_lockstep(o2, g2, _bf16_workload(shape.vocab))
    z8, zb = o.debug_logits(0), o2.debug_logits(0)
    assert np.abs(z8 - zb).max() > TOL_BF16
    assert np.abs(g.debug_logits(0) - z8).max() < np.abs(g2.debug_logits(0) - z8).max()


def test_fp8_kv_cache_long_context_split_attention_chunked_prefill_and_mixed_pass():
    shape = SHAPES["small-d128"]
    blob = make_weight_blob(shape, seed=3, weight_std=0.03, gain_std=0.1)
    o, g = _fp8_pair(shape, blob, max_context=2048, max_trajectories=4, kv_pool_pages=200, max_batch_rows=384)
    rng = np.random.default_rng(1)
    lens = [1700, 523]      # 107 pages against 33: the planner cuts the long context into parts
    toks = rng.integers(0, shape.vocab, sum(lens))
    for e in (o, g):
        e.append_observation([0, 1], toks, lens)
        e.fork(1, [2])
    rms = _fp8_model_rms(o, 1)
    for step in range(3):
        for t in (0, 1, 2):
            assert np.abs(o.debug_logits(t) - g.debug_logits(t)).max() < 8.0 * rms
        ids, lps = o.decode_step([0, 1, 2], 1.0, 5)
        glp = g.decode_step_forced([0, 1, 2], 1.0, ids)
        assert np.abs(glp - lps).max() < 8.0 * rms
    # Update + Generate in one pass
    obs = rng.integers(0, shape.vocab, 40)
    o.append_observation([2, 0], obs, [25, 15])
    ids, lps = o.decode_step([0, 1, 2], 1.0, 5)
    glp = g.decode_step_forced_with_appends([2, 0], obs, [25, 15], [0, 1, 2], 1.0, ids)
    assert np.abs(glp - lps).max() < 8.0 * rms
    for t in (0, 1, 2):
        compare_records(o, g, t)
    # the objective pass reads the same cache
    out = g.grpo_objective([0, 1, 2], 3, [1.0, 0.0, 0.5], 1.0, 0.2, 0.0)
    want = o.grpo_objective([0, 1, 2], 3, [1.0, 0.0, 0.5], 1.0, 0.2, 0.0)
    assert out["n_tokens"] == want["n_tokens"] and abs(out["objective"] - want["objective"]) < 8.0 * rms * 2


def test_fp8_kv_cache_needs_the_mfma_path():
    for name, flags in [("tiny", rl.FLAG_FP8_KV_CACHE), ("tiny-bf16", rl.FLAG_FP8_KV_CACHE),
                        ("small-d128", rl.FLAG_FP8_KV_CACHE | rl.FLAG_GENERIC_KERNELS)]:
        shape = SHAPES[name]
        with pytest.raises(rl.RolloutError) as ei:
            rl.RolloutEngine(make_weight_blob(shape, seed=1), flags=flags, max_context=64,
                             max_trajectories=2, kv_pool_pages=8)
        assert ei.value.code == -1


def test_fp8_kv_cache_is_bit_reproducible():
    shape = SHAPES["small-d128"]
    blob = make_weight_blob(shape, seed=5, weight_std=0.03, gain_std=0.1)
    w = _bf16_workload(shape.vocab)
    runs = []
    for _ in range(2):
        g = rl.RolloutEngine(blob, flags=rl.FLAG_FP8_KV_CACHE, max_context=1024, max_trajectories=16,
                             kv_pool_pages=256)
        rec = replay(g, w)
        runs.append((rec, [g.traj_read(t) for t in range(6)]))
        g.close()
    assert runs[0][0].keys() == runs[1][0].keys() and len(runs[0][0]) == 6
    for t in runs[0][0]:
        assert runs[0][0][t] == runs[1][0][t]
    for a, b in zip(runs[0][1], runs[1][1]):
        assert all(np.array_equal(x, y) for x, y in zip(a, b))
