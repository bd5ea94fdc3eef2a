"""Weights under which one key, one page or one rounding decides the logits, and sums in the kernels' order (test helper).

All models have one layer, an MLP of zeros and a RoPE base so large that the upper half of a head's dim pairs do not rotate.
"""
import numpy as np

from oracle.fp8 import e4m3_round
from oracle.sampler import EXP2_POLY, scale_constant
from synthetic import SHAPES, make_weight_blob
from synthetic.weights import BLOB_HEADER_BYTES, _to_bf16_bits, tensor_table

KINDS = 30                       # key dims 32 .. 61 of a head; dim 62: the filler's key, dim 63: a query that meets no key
FILLER = 0


def KEY(j):                      # tokens with key j that look for nothing, that look for key j, and both
    return 1 + j


def QUERY(j):
    return 1 + KINDS + j


def SELF(j):
    return 1 + 2 * KINDS + j


def set_tensors(shape, tensors, like=None):
    """Blob of a bf16 model with the named tensors set; the others as in `like`, or gains of one and zeros."""
    blob = make_weight_blob(shape, zero_linear=True) if like is None else like.copy()
    at = BLOB_HEADER_BYTES
    for name, dims, _ in tensor_table(shape):
        n = int(np.prod(dims))
        if name in tensors:
            a = np.asarray(tensors[name], np.float32)
            assert a.shape == dims, name
            blob[at:at + 2 * n].view(np.uint16)[:] = _to_bf16_bits(a.reshape(-1))
        at += 2 * n
    return blob


def _bf16(a):
    return (_to_bf16_bits(np.ascontiguousarray(a, np.float32).reshape(-1)).astype(np.uint32) << 16).view(np.float32).reshape(np.shape(a))


class Peaked:
    """Tokens are one-hot, so a token's query and key are single dims of 128^0.5: a query meets its own kind of key with a score of
    11.3 and e^11.3 = 82 000 times the weight of any other.  Values are random per kind and kv head."""

    def __init__(self, heads, kv8=False, seed=1):
        s = self.shape = SHAPES["small-d128"].replace(n_layers=1, hidden=256, intermediate=64, vocab=4096, n_q_heads=heads[0], n_kv_heads=heads[1],
                                                      rope_theta=1e30)
        rng = np.random.default_rng(seed)
        tokens = 1 + 3 * KINDS
        embed = np.zeros((s.vocab, s.hidden))
        embed[np.arange(tokens), np.arange(tokens)] = 1.0
        wq, wk = np.zeros((s.n_q_heads, 128, s.hidden)), np.zeros((s.n_kv_heads, 128, s.hidden))
        wq[:, 63, FILLER] = wk[:, 62, FILLER] = 1.0
        for j in range(KINDS):
            wq[:, 63, KEY(j)] = wq[:, 32 + j, QUERY(j)] = wq[:, 32 + j, SELF(j)] = 1.0
            wk[:, 32 + j, KEY(j)] = wk[:, 62, QUERY(j)] = wk[:, 32 + j, SELF(j)] = 1.0
        wv = _bf16(np.where(np.arange(s.hidden) < tokens, rng.standard_normal((s.n_kv_heads, 128, s.hidden)) / 16, 0.0))
        self.values, self.score = 16.0 * wv.astype(np.float64), 128 ** 0.5       # a one-hot row divided by its rms is 16
        if kv8:
            self.values, self.score = e4m3_round(self.values), float(e4m3_round(self.score))
        self.wo = _bf16(rng.standard_normal((s.hidden, s.n_q_heads * 128)) * (2.0 / (s.n_q_heads * 128)) ** 0.5)
        self.head = _bf16(rng.standard_normal((s.vocab, s.hidden)) / 16)
        self.key_of = np.full(tokens, 62)
        self.looks_for = np.full(tokens, 63)
        for j in range(KINDS):
            self.key_of[[KEY(j), SELF(j)]] = self.looks_for[[QUERY(j), SELF(j)]] = 32 + j
        self.blob = set_tensors(s, {"embed": embed, "l0.w_q": wq.reshape(-1, s.hidden), "l0.w_k": wk.reshape(-1, s.hidden),
                                    "l0.w_v": wv.reshape(-1, s.hidden), "l0.w_o": self.wo, "lm_head": self.head})

    def logits(self, tokens):
        """Of the last of `tokens`, in float64 from the closed form."""
        s, tokens = self.shape, np.asarray(tokens)
        w = np.where(self.key_of[tokens] == self.looks_for[tokens[-1]], np.exp(self.score), 1.0)
        values = self.values[:, :, tokens] @ (w / w.sum())
        h = self.wo.astype(np.float64) @ np.repeat(values, s.n_q_heads // s.n_kv_heads, 0).reshape(-1)
        h[tokens[-1]] += 1.0
        return self.head.astype(np.float64) @ (h / np.sqrt(np.mean(h * h) + 1e-6))

    def logprobs(self, tokens):
        z = self.logits(tokens)
        return z - z.max() - np.log(np.exp(z - z.max()).sum())


class ManySmallWeights:
    """One token of large weight, then any number whose softmax weight of an eighth lies just below half way to the next bf16 number:
    rounded, every one of them is too small by 0.375 %.  All others' values are zero, so that the output is the first
    one's value divided by the denominator.  Token 0: the many, token 1: the first."""

    def __init__(self, heads, most):
        s = self.shape = SHAPES["small-d128"].replace(n_layers=1, hidden=512, intermediate=64, vocab=4096, n_q_heads=heads[0], n_kv_heads=heads[1],
                                                      rope_theta=1e30, qk_norm=0)
        rng = np.random.default_rng(3)
        # query and key of one dim whose product is sqrt(128) log(8 / (1 + 0.48 / 128)): the best pair of bf16 numbers
        want = np.sqrt(128.0) * np.log(8.0 / (1 + 0.48 / 128))
        q, k = min(((a, b) for a in np.arange(128, 256) / 64 for b in np.arange(128, 256) / 16), key=lambda p: abs(p[0] * p[1] - want))
        self.weight = np.exp(-q * k / np.sqrt(128.0))
        self.rounded = float(_bf16(np.array([self.weight]))[0])
        embed = np.zeros((s.vocab, s.hidden))        # 128 dims of two, so that the norm changes nothing; dim 64 tells the two apart
        embed[:, :128] = 2.0
        embed[1, 64] = -2.0
        outs = s.n_q_heads * 128
        assert outs <= s.hidden - 128
        wq, wk = np.zeros((s.n_q_heads, 128, s.hidden)), np.zeros((s.n_kv_heads, 128, s.hidden))
        wv, wo = np.zeros((s.n_kv_heads, 128, s.hidden)), np.zeros((s.hidden, outs))
        wq[:, 63, 0] = q / 2
        wk[:, 63, 0], wk[:, 63, 64] = k / 4, -k / 4
        self.value = _bf16(rng.uniform(0.5, 1.0, (s.n_kv_heads, 128)) * most * self.weight)
        wv[:, :, 0], wv[:, :, 64] = self.value / 4, -self.value / 4
        wo[128 + np.arange(outs), np.arange(outs)] = 1.0
        head = np.zeros((s.vocab, s.hidden))
        head[0, 128:128 + outs] = 4.0 / outs
        self.blob = set_tensors(s, {"embed": embed, "l0.w_q": wq.reshape(-1, s.hidden), "l0.w_k": wk.reshape(-1, s.hidden),
                                    "l0.w_v": wv.reshape(-1, s.hidden), "l0.w_o": wo, "lm_head": head})

    def logprobs(self, n, weight=None):
        """Of token 0 behind one token 1 and 1 .. n - 1 tokens 0, in float64; weight: in the denominator."""
        s = self.shape
        d = 1.0 + np.arange(1, n) * (self.weight if weight is None else weight)
        o = np.repeat(self.value.astype(np.float64), s.n_q_heads // s.n_kv_heads, 0).reshape(-1)[:, None] / d
        z = 4.0 * o.mean(0) / np.sqrt((128 * 4 + (o * o).sum(0)) / s.hidden + 1e-6)
        return z - np.log(np.exp(z) + s.vocab - 1)


def _fma(a, b, c):
    return (np.float64(a) * np.float64(b) + np.float64(c)).astype(np.float32)


def normed_keys(x, first):
    """Rows of 128 fp32 numbers divided by their rms, in bf16, with the roundings of the kernels: sixteen lanes of four dims and their
    partners 64 further on, whose squares are added with one fused multiply-add; first: the dim's own square is the fused one."""
    lo, hi = x[:, :64], x[:, 64:]
    t = (_fma(lo, lo, hi * hi) if first else _fma(hi, hi, lo * lo)).reshape(-1, 16, 4)
    s = ((t[..., 0] + t[..., 1]) + t[..., 2]) + t[..., 3]
    for o in (8, 4, 2, 1):
        s = s + s[:, np.arange(16) ^ o]
    return _bf16(x * (np.float32(1) / np.sqrt(_fma(s[:, :1], np.float32(1 / 128), np.float32(1e-6)))))


class KeyBits:
    """Pairs of tokens whose keys agree in the one dim that a query token looks at, to the bit, and no longer do if the sum of
    squares of the first one's key is rounded the other way: one bf16 step of the key is then eight units of the score."""

    def __init__(self):
        s = self.shape = SHAPES["small-d128"].replace(n_layers=1, hidden=256, intermediate=64, vocab=4096, n_q_heads=2, n_kv_heads=2, rope_theta=1e30)
        dims = np.r_[32:64, 96:128]                    # those that do not rotate
        pairs = []                                     # (dim, its key, parts of the two rows)
        for seed in range(12):
            rng = np.random.default_rng(seed)
            part = _bf16(rng.uniform(1, 2, (2, 20000, 64)) * rng.choice([-1, 1], (2, 20000, 64)))
            x = np.zeros((20000, 128), np.float32)
            x[:, dims] = 16 * part[0] + part[1] / 16   # exact in fp32, their squares are not
            a, b = normed_keys(x, True), normed_keys(x, False)
            for r, c in zip(*np.nonzero(a != b)):
                same = np.nonzero((a[:, c] == a[r, c]) & (b[:, c] == a[r, c]))[0]
                pairs.append((c, a[r, c], part[:, r], part[:, same[0]]))
        self.pairs = len(pairs)
        tokens = 1 + 3 * self.pairs                    # token 0: no key; then first, second and query of every pair
        assert self.pairs >= 8 and 2 * tokens <= s.hidden
        embed = np.zeros((s.vocab, s.hidden))
        wq, wk = np.zeros((2, 128, s.hidden)), np.zeros((2, 128, s.hidden))
        for t in range(tokens):                        # divided by their rms: 16 and 1 / 16
            embed[t, 2 * t], embed[t, 2 * t + 1] = 1.0, 2.0 ** -8
        for i, (c, key, first, second) in enumerate(pairs):
            for t, part in ((1 + 3 * i, first), (2 + 3 * i, second)):
                wk[:, dims, 2 * t], wk[:, dims, 2 * t + 1] = part
            wq[:, c, 2 * (3 + 3 * i)] = np.sign(key)
        rng = np.random.default_rng(1)
        wv = np.zeros((2, 128, s.hidden))
        wv[:, :, 0:2 * tokens:2] = rng.standard_normal((2, 128, tokens)) / 16
        self.wv, self.wo = _bf16(wv), _bf16(rng.standard_normal((s.hidden, 256)) / 11)
        self.head = _bf16(rng.standard_normal((s.vocab, s.hidden)) / 16)
        self.blob = set_tensors(s, {"embed": embed, "l0.w_q": wq.reshape(-1, s.hidden), "l0.w_k": wk.reshape(-1, s.hidden), "l0.g_q": np.full(128, 1024.0),
                                    "l0.w_v": self.wv.reshape(-1, s.hidden), "l0.w_o": self.wo, "lm_head": self.head})

    def logits(self, i, share=0.5):
        """Behind the tokens of pair i in float64; share: of the first one."""
        t = 1 + 3 * i
        values = 16.0 * (share * self.wv[:, :, 2 * t] + (1 - share) * self.wv[:, :, 2 * t + 2]).astype(np.float64)
        h = self.wo.astype(np.float64) @ values.reshape(-1)
        h[2 * t + 4] += 1.0
        h[2 * t + 5] += 2.0 ** -8
        return self.head.astype(np.float64) @ (h / np.sqrt(np.mean(h * h) + 1e-6))


def weight_sum(z, temperature, by_lane=False):
    """The fp32 sum of the sampler's weights over a row of more than 16384 numbers in the kernels' order: a segment of 4096 by 256 threads
    of sixteen, a wave's 64 threads, four waves, 64 lanes of segments.  by_lane: the four waves' threads first."""
    f, v = np.float32, len(z)
    t = ((z - z.max()) * scale_constant(temperature)).astype(f)
    n = np.floor(t)
    p = np.full_like(t, EXP2_POLY[6])
    for c in EXP2_POLY[5::-1]:
        p = (p * (t - n)).astype(f) + c
    e = np.zeros(-(-v // 4096) * 4096, f)
    e[:v] = np.where(n < -40, f(0), np.ldexp(p, n.astype(np.int32) + 32))
    seg = e.reshape(-1, 4, 256, 4).transpose(0, 2, 1, 3).reshape(-1, 256, 16) if v % 4 == 0 else e.reshape(-1, 16, 256).transpose(0, 2, 1)

    def chain(x):                                # one after the other
        out = np.zeros(x.shape[:-1], f)
        for i in range(x.shape[-1]):
            out = out + x[..., i]
        return out

    def tree(x):                                 # 64 lanes, halves first
        for o in (32, 16, 8, 4, 2, 1):
            x = x[..., :o] + x[..., o:]
        return x[..., 0]

    def four(x):
        return (x[..., 0] + x[..., 1]) + (x[..., 2] + x[..., 3])
    threads = chain(seg).reshape(-1, 4, 64)
    sums = (tree(four(threads.transpose(0, 2, 1))) if by_lane else four(tree(threads))) * f(2.0 ** -32)
    k = len(sums)
    if k <= 64:
        return tree(np.r_[sums, np.zeros(64 - k, f)])
    lanes = np.r_[sums, np.zeros(-k % 256, f)].reshape(-1, 256).T
    return four(tree(chain(lanes).reshape(4, 64)))
