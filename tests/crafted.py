"""Weights under which one key, one page or one rounding decides the logits (test helper).

All models have one layer, an MLP of zeros and a RoPE base so large that the upper half of a head's dim pairs do not rotate.
"""
import numpy as np

from synthetic import SHAPES, make_weight_blob
from synthetic.weights import BLOB_HEADER_BYTES, _to_bf16_bits, tensor_table

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


s ManySmallWeights:
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


def
