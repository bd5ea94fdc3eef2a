"""Timed cases of the rollout engine: what one pass of each is, its inputs and its exact result.

Every case goes through the public entry points of `paper_2509_06980_amd`.  The models have the layer
dimensions of the repository's shapes with fewer layers (a pass of a decoder is the same layer over and
over), random weights and tied embeddings; token ids are uniform.  Decode steps are teacher-forced, so
that log-probs can be compared whatever the rounding of the logits does to a draw.

Kinds of work:
  logits   one sequence, next-token logits (rl_debug_logits): the smallest call, one row
  decode   `steps` decode steps of a batch over cached contexts; the contexts grow from pass to pass
  mixed    one decode step of a batch with the first chunks of newly arrived requests riding along
  append   prompts (or observations on top of a cached context) prefilled, one token each, release
  score    log-probs of whole cached trajectories recomputed (observation tokens masked out)
  sample   the sampler alone on device buffers
  rollout  the whole multi-turn loop of the fp32 shape, greedy
"""
import math
import random
import struct
import weakref

import numpy as np
import torch

import paper_2509_06980_amd as rl
from synthetic import SHAPES

MODELS = ("tiny", "small-d128", "qwen3-0.6b", "qwen3-4b", "qwen3-8b")
GROW = 1024        # tokens a decode state can grow by before its contexts are built again
HELD = 4           # states of one case that fit the page pool at once


def listed():
    return [
        # the fp32 shape's whole loop: 4 prompts, 3 turns of 16 greedy tokens and 8 observation tokens
        dict(name="rollout-fp32", kind="rollout", model="tiny", layers=2, batch=4, context=32, turns=3, steps=16, tokens=8),
        # one interactive sequence: latency of a one-row pass, logits out
        dict(name="logits-0.6b", kind="logits", model="qwen3-0.6b", layers=4, batch=1, context=777, cache8=False),
        # small-model rollout, 64 trajectories in the middle of their second turn
        dict(name="decode-0.6b-64", kind="decode", model="qwen3-0.6b", layers=8, batch=64, context=640, longest=640, group=1, steps=4, cache8=False),
        # the headline rollout in its third turn: 128 trajectories, groups of 8 on a 512-token prompt
        dict(name="decode-4b-128", kind="decode", model="qwen3-4b", layers=8, batch=128, context=2048, longest=2048, group=8, steps=2, cache8=False),
        # the same batch later on, with the 8-bit cache
        dict(name="decode-4b-128-fp8", kind="decode", model="qwen3-4b", layers=8, batch=128, context=3000, longest=3000, group=8, steps=2, cache8=True),
        # what is left of a batch of ragged trajectories while the others wait for their tools
        dict(name="decode-4b-ragged-37", kind="decode", model="qwen3-4b", layers=8, batch=37, context=300, longest=7000, group=1, steps=4, cache8=False),
        # few long conversations on the larger shape
        dict(name="decode-8b-6-long", kind="decode", model="qwen3-8b", layers=4, batch=6, context=6000, longest=8000, group=1, steps=16, cache8=False),
        # continuous batching: 48 trajectories decode while 3 requests of about 200 tokens arrive
        dict(name="mixed-4b-48", kind="mixed", model="qwen3-4b", layers=8, batch=48, context=1000, longest=1000, group=1, arrivals=3, tokens=201, cache8=False),
        # start of a rollout: 16 prompts of 512 tokens
        dict(name="prompts-4b", kind="append", model="qwen3-4b", layers=8, batch=16, context=0, tokens=512, longest=512, cache8=False),
        # tool results come back: about 500 observation tokens on top of contexts of 3000
        dict(name="observe-4b", kind="append", model="qwen3-4b", layers=8, batch=12, context=3000, tokens=333, longest=800, cache8=False),
        # log-probs of finished trajectories for the policy update
        dict(name="score-4b", kind="score", model="qwen3-4b", layers=8, batch=12, context=500, longest=1500, steps=64, turns=3, cache8=False),
        # the sampler at the size of a decode step
        dict(name="sample-128", kind="sample", rows=128, vocab=151936, temperature=1.0),
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["logits", "decode", "decode", "decode", "mixed", "append", "append", "score", "sample", "rollout"])
    if kind == "sample":
        return dict(kind=kind, rows=log(1, 256), vocab=rng.choice([4096, 8192, 151936, log(3000, 151000)]),
                    temperature=rng.choice([1.0, 0.0, round(rng.uniform(0.3, 1.5), 3)]))
    if kind == "rollout":
        return dict(kind=kind, model="tiny", layers=2, batch=log(1, 12), context=log(8, 120), turns=rng.randint(1, 4), steps=log(2, 24), tokens=log(1, 30))
    model, layers = rng.choice([("small-d128", 3), ("qwen3-0.6b", 4), ("qwen3-0.6b", 8), ("qwen3-4b", 8), ("qwen3-8b", 4)])
    small = model == "small-d128"
    cache8 = rng.random() < 0.25
    if kind == "logits":
        return dict(kind=kind, model=model, layers=min(layers, 4), batch=1, context=log(2, 400 if small else 6000), cache8=False)
    if kind == "decode":
        batch = log(1, 150)
        context = log(16, min(6000, 200000 // batch))
        longest = rng.choice([context, context, min(8000, 2 * context)])
        group = rng.choice([1, 1, 8]) if batch % 8 == 0 else 1
        return dict(kind=kind, model=model, layers=layers, batch=batch, context=context, longest=longest, group=group,
                    steps=max(2, min(16, 96 // batch)), cache8=cache8)
    if kind == "mixed":
        context = log(16, 2000)
        return dict(kind=kind, model=model, layers=layers, batch=log(8, 100), context=context, longest=context + log(1, 500), group=1,
                    arrivals=rng.randint(1, 5), tokens=log(20, 400), cache8=cache8)
    if kind == "append":
        batch, tokens = log(1, 24), log(30, 600)
        return dict(kind=kind, model=model, layers=layers, batch=batch, context=rng.choice([0, log(20, 3000)]), tokens=tokens,
                    longest=tokens + rng.randint(0, tokens), cache8=cache8)
    context = log(60, 1000)
    return dict(kind=kind, model=model, layers=layers, batch=log(2, 12), context=context, longest=context + rng.randint(0, 500),
                steps=log(4, 64), turns=rng.randint(1, 3), cache8=cache8)


# ---- sizes that follow from a case alone --------------------------------------------------------

def _shape(case):
    return SHAPES[case["model"]].replace(n_layers=case["layers"], tie_embeddings=1)


def _spread(lo, hi, n, salt):
    """n lengths from lo to hi, the same ones for every seed."""
    r = random.Random(salt * 1000003 + n)
    got = [lo + int(round((hi - lo) * r.random())) for _ in range(n)]
    if n > 1:
        got[0], got[-1] = lo, hi
    return got


def _contexts(case):
    return _spread(case["context"], case.get("longest", case["context"]), case["batch"], 1)


def _chunks(case):
    """Lengths of the chunks that an append or mixed case prefills."""
    if case["kind"] == "mixed":
        return _spread(max(1, case["tokens"] // 2), case["tokens"] + case["tokens"] // 2, case["arrivals"], 2)
    return _spread(case["tokens"], case["longest"], case["batch"], 2)


def _prompt(case):
    """Tokens that the members of a group share."""
    return min(512, case["context"] // 2) if case.get("group", 1) > 1 else 0


def _turns(case):
    """Score: [(sampled, appended), ...] of every trajectory after its prompt; contexts are whole lengths."""
    return [(case["steps"], max(1, (n - case["turns"] * case["steps"]) // (case["turns"] + 1))) for n in _contexts(case)]


# ---- inputs, in numpy and torch -------------------------------------------------------------------

_kept = {}         # the model that the last case used: blob and engine, as a serving process keeps them


def _weights(shape):
    """The flat weights in blob order (a tensor on the GPU) and [(name, dims)]."""
    s = shape
    qw, kw = s.q_width, s.kv_width
    table = [("embed", (s.vocab, s.hidden))]
    for l in range(s.n_layers):
        table += [("g_in%d" % l, (s.hidden,)), ("w_q%d" % l, (qw, s.hidden)), ("w_k%d" % l, (kw, s.hidden)), ("w_v%d" % l, (kw, s.hidden)),
                  ("g_q%d" % l, (s.head_dim,)), ("g_k%d" % l, (s.head_dim,)), ("w_o%d" % l, (s.hidden, qw)), ("g_post%d" % l, (s.hidden,)),
                  ("w_gate%d" % l, (s.intermediate, s.hidden)), ("w_up%d" % l, (s.intermediate, s.hidden)),
                  ("w_down%d" % l, (s.hidden, s.intermediate))]
    table.append(("g_final", (s.hidden,)))
    gen = torch.Generator(device="cuda").manual_seed(1)
    dtype = torch.bfloat16 if s.weight_dtype == 1 else torch.float32
    std = 0.02 if s.hidden >= 1024 else 0.03
    flat = torch.empty(sum(math.prod(d) for _, d in table), dtype=dtype, device="cuda")
    off, at = 0, {}
    for name, dims in table:
        n = math.prod(dims)
        x = torch.randn(n, generator=gen, device="cuda")
        flat[off:off + n] = (1 + 0.1 * x if name.startswith("g_") else std * x).to(dtype)
        at[name] = (off, dims)
        off += n
    return flat, at


def _blob(shape):
    s = shape
    flat, _ = _weights(s)
    head = b"RLW1" + struct.pack("<I7i2f3i", 1, s.n_layers, s.hidden, s.n_q_heads, s.n_kv_heads, s.head_dim, s.intermediate, s.vocab,
                                 s.rms_eps, s.rope_theta, s.qk_norm, s.tie_embeddings, s.weight_dtype)
    raw = flat.view(torch.uint8).cpu().numpy()
    blob = np.zeros(64 + raw.size, np.uint8)
    blob[:len(head)] = np.frombuffer(head, np.uint8)
    blob[64:] = raw
    return blob


def _engine(case):
    shape = _shape(case)
    if _kept.get("shape") != shape:
        _drop_engine()
        _kept.update(shape=shape, blob=_blob(shape))
        torch.cuda.empty_cache()
    longest = max(_contexts(case))
    extra = max(_chunks(case)) + 1 if case["kind"] in ("append", "mixed") else 0
    grow = GROW if case["kind"] in ("decode", "mixed") else 0
    if case["kind"] == "rollout":
        extra = case["turns"] * (case["steps"] + case["tokens"])
    if case["kind"] == "append":
        longest = case["context"]
    if case["kind"] == "score":
        longest = max(o + case["turns"] * (g + o) for g, o in _turns(case))
    room = longest + extra + grow + 16
    n = case["batch"] * (2 if case["kind"] == "append" else 1) + case.get("arrivals", 0)
    config = (room, HELD * n, HELD * (n * (room // 16 + 2)), rl.FLAG_FP8_KV_CACHE if case.get("cache8") else 0)
    if _kept.get("config") != config:
        _drop_engine()
        _kept["config"] = config
        _kept["engine"] = rl.RolloutEngine(_kept["blob"], max_context=config[0], max_trajectories=config[1], kv_pool_pages=config[2],
                                           flags=config[3])
        _kept["next"] = 0
    return _kept["engine"]


def _drop_engine():
    engine = _kept.pop("engine", None)
    _kept.pop("config", None)
    if engine is not None:
        engine.close()


def _ids(n):
    first = _kept["next"]
    _kept["next"] = (first + n) % (1 << 30)
    return np.arange(first, first + n, dtype=np.int32)


class _State:
    """The trajectories of one state; they are released when the state is let go."""

    def __init__(self, engine, ids):
        self.engine, self.ids, self.live = engine, ids, set()
        weakref.finalize(self, _State._let_go, engine, self.live)

    @staticmethod
    def _let_go(engine, live):
        if getattr(engine, "_h", None) and live:
            engine.release(sorted(live))


def _tokens(case, seed):
    """Every token a pass can need, from the seed: {name: [array per trajectory]}."""
    rng = np.random.default_rng([int(seed), 2])
    v = _shape(case).vocab

    def some(n):
        return rng.integers(0, v, size=n, dtype=np.int32)

    kind = case["kind"]
    got = {}
    if kind == "score":
        plan = _turns(case)
        got["prompt"] = [some(o) for _, o in plan]
        got["turns"] = [[(some(g), some(o)) for _ in range(case["turns"])] for g, o in plan]
        return got
    if kind == "rollout":
        got["prompt"] = [some(case["context"]) for _ in range(case["batch"])]
        got["observed"] = [[some(case["tokens"]) for _ in range(case["batch"])] for _ in range(case["turns"])]
        return got
    shared = _prompt(case)
    group = case.get("group", 1)
    got["shared"] = [some(shared) for _ in range(case["batch"] // group)] if shared else []
    got["own"] = [some(n - shared) for n in _contexts(case)] if kind != "append" else [some(case["context"]) for _ in range(case["batch"])]
    if kind in ("append", "mixed"):
        got["chunk"] = [some(n) for n in _chunks(case)]
    rows = case["batch"] + (case["arrivals"] if kind == "mixed" else 0)
    got["forced"] = some(rows * GROW).reshape(GROW, rows)
    return got


def prepare(case, seed):
    if case["kind"] == "sample":
        gen = torch.Generator(device="cuda").manual_seed(int(seed))
        z = torch.randn(case["rows"], case["vocab"], generator=gen, device="cuda") * 1.5
        u = torch.randint(0, 1 << 32, (case["rows"],), generator=gen, device="cuda", dtype=torch.int64)
        u = torch.where(u >= 1 << 31, u - (1 << 32), u).to(torch.int32)
        return dict(case=case, logits=z, u32=u, ids=torch.zeros(case["rows"], dtype=torch.int32, device="cuda"),
                    lps=torch.zeros(case["rows"], dtype=torch.float32, device="cuda"))
    engine = _engine(case)
    tokens = _tokens(case, seed)
    kind, n = case["kind"], case["batch"]
    state = _State(engine, _ids(n * (2 if kind == "append" else 1) + case.get("arrivals", 0)))
    state.case, state.tokens = case, tokens
    if kind == "rollout":
        return state
    if kind == "score":
        ids = state.ids
        engine.append_observation(ids, np.concatenate(tokens["prompt"]), [len(t) for t in tokens["prompt"]])
        state.live.update(int(i) for i in ids)
        for turn in range(case["turns"]):
            for k in range(case["steps"]):
                engine.decode_step_forced(ids, 1.0, [t[turn][0][k] for t in tokens["turns"]])
            engine.append_observation(ids, np.concatenate([t[turn][1] for t in tokens["turns"]]), [len(t[turn][1]) for t in tokens["turns"]])
        return state
    _fill(state)
    return state


def _fill(state):
    """The cached contexts that a decode, mixed, logits or append case starts from."""
    case, tokens, engine = state.case, state.tokens, state.engine
    ids = state.ids[:case["batch"]]
    group = case.get("group", 1)
    if tokens["shared"]:
        leaders = ids[::group]
        engine.append_observation(leaders, np.concatenate(tokens["shared"]), [len(t) for t in tokens["shared"]])
        for g in leaders:
            engine.fork(int(g), np.arange(g + 1, g + group, dtype=np.int32))
    own = [len(t) for t in tokens["own"]]
    if sum(own):
        engine.append_observation(ids, np.concatenate(tokens["own"]), own)
    if tokens["shared"] or sum(own):
        state.live.update(int(i) for i in ids)
    state.at = 0


def run(state):
    if isinstance(state, dict):
        case = state["case"]
        rl.sample_device_logits(state["logits"].data_ptr(), case["rows"], case["vocab"], case["temperature"], state["u32"].data_ptr(),
                                state["ids"].data_ptr(), state["lps"].data_ptr(), torch.cuda.current_stream().cuda_stream)
        return {"ids": state["ids"], "logprobs": state["lps"]}
    case, engine, tokens, n = state.case, state.engine, state.tokens, state.case["batch"]
    kind = case["kind"]
    ids = state.ids[:n]
    if kind == "logits":
        return engine.debug_logits(int(ids[0]))
    if kind == "score":
        return engine.recompute_logprobs(ids, 1.0)
    if kind == "decode":
        if state.at + case["steps"] > GROW:        # the batch is over: the next one starts
            engine.release(ids)
            _fill(state)
        out = [engine.decode_step_forced(ids, 1.0, tokens["forced"][state.at + k]) for k in range(case["steps"])]
        state.at += case["steps"]
        return np.stack(out)
    if kind == "mixed":
        if state.at + 1 > GROW:
            engine.release(ids)
            _fill(state)
        new = state.ids[n:]
        out = engine.decode_step_forced_with_appends(new, np.concatenate(tokens["chunk"]), [len(t) for t in tokens["chunk"]], state.ids, 1.0,
                                                     tokens["forced"][state.at])
        engine.release(new)
        state.at += 1
        return out
    if kind == "append":
        target = state.ids[n:]
        if case["context"]:
            for a, b in zip(ids, target):
                engine.fork(int(a), [int(b)])
        engine.append_observation(target, np.concatenate(tokens["chunk"]), [len(t) for t in tokens["chunk"]])
        out = engine.decode_step_forced(target, 1.0, tokens["forced"][0])
        engine.release(target)
        return out
    # rollout: the whole loop, greedy
    engine.append_observation(ids, np.concatenate(tokens["prompt"]), [case["context"]] * n)
    got = []
    for turn in range(case["turns"]):
        got.append(engine.decode_steps(ids, case["steps"], 0.0, 3))
        engine.append_observation(ids, np.concatenate(tokens["observed"][turn]), [case["tokens"]] * n)
    engine.release(ids)
    return {"ids": np.stack([g[0] for g in got]), "logprobs": np.stack([g[1] for g in got])}


# ---- what a pass cannot do without ---------------------------------------------------------------

def work(case):
    kind = case["kind"]
    if kind == "sample":
        return {"bytes": case["rows"] * (case["vocab"] * 4.0 + 12), "flops": 20.0 * case["rows"] * case["vocab"]}
    s = _shape(case)
    el = 2.0 if s.weight_dtype == 1 else 4.0
    per_layer = s.linear_params() / s.n_layers
    linear, head = s.linear_params(), s.vocab * s.hidden
    kvtok = 2 * s.kv_width * s.n_layers * (1.0 if case.get("cache8") else el)     # keys + values of a token
    attn = 4.0 * s.q_width * s.n_layers                                          # flops per (row, key)

    def rows(contexts, shared=0.0):      # one decode step over these contexts
        m = len(contexts)
        return ((linear + head) * el + (sum(contexts) - shared) * kvtok + m * kvtok,
                2.0 * m * (linear + head) + attn * sum(contexts))

    def prefill(chunks, base):           # chunks on top of cached contexts: read once, written once
        keys = sum(b * c + c * (c + 1) / 2 for c, b in zip(chunks, base))
        return linear * el + sum(base) * kvtok + sum(chunks) * kvtok, 2.0 * sum(chunks) * linear + attn * keys

    if kind == "rollout":
        b = f = 0.0
        n, ctx = case["batch"], case["context"]
        parts = [prefill([ctx] * n, [0] * n)]
        for _ in range(case["turns"]):
            parts += [rows([ctx + k + 1] * n) for k in range(case["steps"])]
            ctx += case["steps"]
            parts.append(prefill([case["tokens"]] * n, [ctx] * n))
            ctx += case["tokens"]
        for x, y in parts:
            b, f = b + x, f + y
        return {"bytes": b, "flops": f}
    if kind == "score":
        lens = [o + case["turns"] * (g + o) for g, o in _turns(case)]
        b, f = prefill(lens, [0] * len(lens))
        picked = case["batch"] * case["turns"] * case["steps"]
        return {"bytes": b + head * el + 4.0 * sum(lens), "flops": f + 2.0 * picked * head}
    ctx = _contexts(case)
    if kind == "append":
        base = [case["context"]] * case["batch"]
        b, f = prefill(_chunks(case), base)
        b2, f2 = rows([c + x for c, x in zip(base, _chunks(case))])
        return {"bytes": b + b2, "flops": f + f2}
    shared = 0.0
    if case.get("group", 1) > 1:
        shared = (case["batch"] - case["batch"] // case["group"]) * float(_prompt(case))
    b, f = rows(ctx, shared)
    if kind == "mixed":
        chunks = _chunks(case)
        b += 2 * sum(chunks) * kvtok
        f += 2.0 * sum(chunks) * per_layer * s.n_layers + 2.0 * len(chunks) * head + attn * sum(c * (c + 1) / 2 for c in chunks)
        return {"bytes": b, "flops": f}
    steps = case.get("steps", 1)
    return {"bytes": steps * b + (4.0 * s.vocab if kind == "logits" else 0.0), "flops": steps * f}


def tolerance(case):
    """About four times the distance to exact() that the path shows."""
    kind = case["kind"]
    if kind == "sample":       # integer weights: the ids are the same; float sums of the log-prob in another order
        return {"rel": 1e-6, "max": 4e-6, "differ": 0.0}
    if kind == "rollout":      # fp32: sums in another order (1.2e-7 seen)
        return {"rel": 1e-6, "max": 1e-5, "differ": 0.01}
    if kind == "logits":       # bf16 activations and cache; logits of standard deviation 1 (7.5e-3 seen)
        return {"rel": 0.03, "max": 0.2}
    # log-probs around -12 whose logits carry the bf16 error (1.3e-3 seen), or that of single E4M3 codes (3.8e-3 seen)
    return {"rel": 1.5e-2, "max": 8e-2} if case.get("cache8") else {"rel": 5e-3, "max": 2.5e-2}


# ---- the exact result: plain torch in float64 ------------------------------------------------------

class _Exact:
    """The decoder in float64 on the weights' stored values, one trajectory (or shared prompt) at a time."""

    def __init__(self, case):
        self.s, self.cache8 = _shape(case), bool(case.get("cache8"))
        self.flat, self.at = _weights(self.s)

    def w(self, name):
        off, dims = self.at[name]
        return self.flat[off:off + math.prod(dims)].double().view(dims)

    def norm(self, x, g):
        return x / torch.sqrt((x * x).mean(-1, keepdim=True) + float(np.float32(self.s.rms_eps))) * g

    def rope(self, x, pos):
        half = self.s.head_dim // 2
        inv = float(np.float32(self.s.rope_theta)) ** (-torch.arange(half, dtype=torch.float64, device=x.device) * 2.0 / self.s.head_dim)
        a = pos.double()[:, None] * inv[None, :]
        c, n = torch.cos(a)[:, None, :], torch.sin(a)[:, None, :]
        u, v = x[..., :half], x[..., half:]
        return torch.cat([u * c - v * n, v * c + u * n], -1)

    def attend(self, q, k, v, base):
        """q [T, nq, d] at positions base + t over k, v [S, nkv, d]."""
        s, g = self.s, self.s.n_q_heads // self.s.n_kv_heads
        out = torch.empty_like(q)
        kt, vt = k.permute(1, 2, 0).contiguous(), v.permute(1, 0, 2).contiguous()
        for a in range(0, q.shape[0], 1024):
            qa = q[a:a + 1024]
            t = qa.shape[0]
            keys = base + a + t
            qh = qa.view(t, s.n_kv_heads, g, -1).permute(1, 2, 0, 3).reshape(s.n_kv_heads, g * t, -1).contiguous()
            z = torch.bmm(qh, kt[:, :, :keys].contiguous()) / math.sqrt(s.head_dim)
            hidden = torch.arange(keys, device=q.device)[None, :] > (base + a + torch.arange(t, device=q.device))[:, None]
            z.view(s.n_kv_heads, g, t, keys).masked_fill_(hidden, -math.inf)
            o = torch.bmm(torch.softmax(z, -1), vt[:, :keys].contiguous())
            out[a:a + 1024] = o.view(s.n_kv_heads, g, t, -1).permute(2, 0, 1, 3).reshape(t, s.n_q_heads, -1)
        return out

    def forward(self, pieces):
        """pieces: [(tokens, parent or None)]; a piece continues its parent's whole context.  -> [residual rows] per piece."""
        s = self.s
        h = [self.w_rows(t) for t, _ in pieces]
        base = []
        for t, p in pieces:
            base.append(0 if p is None else base[p] + len(pieces[p][0]))
        for l in range(s.n_layers):
            wq, wk, wv, wo = (self.w(n + str(l)) for n in ("w_q", "w_k", "w_v", "w_o"))
            wg, wu, wd = (self.w(n + str(l)) for n in ("w_gate", "w_up", "w_down"))
            keep = []
            for i, (t, p) in enumerate(pieces):
                n = len(t)
                a = self.norm(h[i], self.w("g_in%d" % l))
                q, k, v = ((a @ w.T).view(n, -1, s.head_dim) for w in (wq, wk, wv))
                pos = base[i] + torch.arange(n, device=a.device)
                if s.qk_norm:
                    q, k = self.norm(q, self.w("g_q%d" % l)), self.norm(k, self.w("g_k%d" % l))
                q, k = self.rope(q, pos), self.rope(k, pos)
                if self.cache8:
                    k, v = (x.clamp(-448, 448).to(torch.float32).to(torch.float8_e4m3fn).double() for x in (k, v))
                if p is not None:
                    k, v = torch.cat([keep[p][0], k]), torch.cat([keep[p][1], v])
                keep.append((k, v) if any(q_ == i for _, q_ in pieces) else None)
                h[i] = h[i] + self.attend(q, k, v, base[i]).reshape(n, -1) @ wo.T
                b = self.norm(h[i], self.w("g_post%d" % l))
                h[i] = h[i] + (torch.nn.functional.silu(b @ wg.T) * (b @ wu.T)) @ wd.T
        return h

    def w_rows(self, tokens):
        off, dims = self.at["embed"]
        return self.flat[off:off + math.prod(dims)].view(dims)[torch.as_tensor(np.asarray(tokens), dtype=torch.int64, device="cuda")].double()

    def logits(self, rows):
        return self.norm(rows, self.w("g_final")) @ self.w("embed").T

    def logprobs(self, rows, targets):
        lm, f, out = self.w("embed").T, self.norm(rows, self.w("g_final")), []
        t = torch.as_tensor(np.asarray(targets), dtype=torch.int64, device="cuda")
        for a in range(0, len(t), 512):
            z = f[a:a + 512] @ lm
            out.append(z.gather(1, t[a:a + 512, None])[:, 0] - torch.logsumexp(z, 1))
        return torch.cat(out).cpu().numpy()


def _exact_sample(case, seed):
    """The integer inverse-CDF law on the float32 logits; the log-prob in float64."""
    st = prepare(case, seed)
    z, temp = st["logits"], case["temperature"]
    m = z.max(1, keepdim=True).values
    if temp == 0.0:
        ids = (z == m).int().argmax(1)
        t64 = 1.0
    else:
        c = torch.tensor(np.float32(1.4426950408889634 / float(np.float32(temp))), device="cuda")
        t = (z - m) * c
        n = torch.floor(t)
        r = t - n
        p = torch.full_like(r, float.fromhex("0x1.b4d1e4p-13"))
        for k in ("0x1.4ca4ccp-10", "0x1.3c4a8ap-7", "0x1.c69f6ap-5", "0x1.ebfc40p-3", "0x1.62e430p-1", "0x1.0p0"):
            p = p * r
            p = p + float.fromhex(k)
        w = torch.floor(p.double() * torch.exp2(n.double()) * 4294967296.0)
        w = torch.where(n < -40, torch.zeros_like(w), w).to(torch.int64)
        total = w.sum(1).cpu().numpy()
        target = [(int(a) * (int(b) & 0xffffffff)) >> 32 for a, b in zip(total, st["u32"].cpu().numpy())]
        ids = (w.cumsum(1) <= torch.tensor(target, device="cuda")[:, None]).sum(1)
        t64 = float(np.float32(temp))
    y = z.double() / t64
    lp = y.gather(1, ids.long()[:, None])[:, 0] - torch.logsumexp(y, 1)
    return {"ids": ids.to(torch.int32).cpu().numpy(), "logprobs": lp.cpu().numpy()}


def exact(case, seed):
    kind, n = case["kind"], case.get("batch", 0)
    if kind == "sample":
        return _exact_sample(case, seed)
    if kind in ("decode", "mixed", "append") and n * max(_contexts(case) + [case["context"]]) > 600000:
        return None
    tokens = _tokens(case, seed)
    x = _Exact(case)
    cat = np.concatenate
    if kind == "logits":
        return x.logits(x.forward([(tokens["own"][0], None)])[0][-1:])[0].cpu().numpy()
    if kind == "score":
        out = []
        for p, turns in zip(tokens["prompt"], tokens["turns"]):
            seq = cat([p] + [y for t in turns for y in t])
            sampled = cat([np.zeros(len(p), bool)] + [np.full(len(y), k == 0) for t in turns for k, y in enumerate(t)])
            at = np.nonzero(sampled)[0]
            lp = np.zeros(len(seq))
            lp[at] = x.logprobs(x.forward([(seq[:-1], None)])[0][torch.as_tensor(at - 1, device="cuda")], seq[at])
            out.append(lp)
        return cat(out)
    if kind == "rollout":
        ids = np.zeros((case["turns"], case["steps"], n), np.int32)
        lps = np.zeros((case["turns"], case["steps"], n))
        for i in range(n):
            seq = tokens["prompt"][i]
            for turn in range(case["turns"]):
                for k in range(case["steps"]):
                    z = x.logits(x.forward([(seq, None)])[0][-1:])[0]
                    ids[turn, k, i] = int(z.argmax())
                    lps[turn, k, i] = float(z.max() - torch.logsumexp(z, 0))
                    seq = cat([seq, ids[turn, k, i:i + 1]])
                seq = cat([seq, tokens["observed"][turn][i]])
        return {"ids": ids, "logprobs": lps}
    steps = case.get("steps", 1) if kind == "decode" else 1
    group = case.get("group", 1)
    forced = tokens["forced"][:steps]
    pieces = [(t, None) for t in tokens["shared"]]
    tails = list(tokens["own"]) + (tokens["chunk"] if kind == "mixed" else [])
    if kind == "append":
        tails = [cat([a, b]) for a, b in zip(tokens["own"], tokens["chunk"])]
    for i, t in enumerate(tails):
        pieces.append((cat([t, forced[:-1, i]]), i // group if tokens["shared"] else None))
    h = x.forward(pieces)[len(tokens["shared"]):]
    lp = x.logprobs(torch.cat([r[-steps:] for r in h]), forced.T.reshape(-1)).reshape(len(tails), steps).T
    return lp if kind == "decode" else lp[0]
