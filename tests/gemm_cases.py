"""Shapes and row counts at which the matrix products' kernels can go wrong, and the variant that each is there for
(test helper).  The choice of a variant is a fitted estimate: test_gemm_plans.py holds every entry to it on the CPU."""
import random

from synthetic import SHAPES


def small(**change):
    return SHAPES["small-d128"].replace(n_layers=1, **change)


def _dims(hidden, n_q_heads, n_kv_heads, intermediate, vocab=512):
    return dict(hidden=hidden, n_q_heads=n_q_heads, n_kv_heads=n_kv_heads, intermediate=intermediate, vocab=vocab)


def split(rows, seed=1):
    """Lengths (20 to 120 tokens) of trajectories whose appended tokens make `rows` rows, one less than tokens each."""
    r, lens = random.Random(rows + seed), []
    left = rows
    while left > 0:
        n = min(left, r.randint(19, 119))
        lens.append(n + 1)
        left -= n
    return lens


# (change, lengths of the trajectories, tokens sampled behind them, what is there to be seen): pass -> product ->
# (kernel, width, K-slices, epilogue) that has to be taken; passes: append, recompute, score (rows of the lm-head)
_06B = _dims(1024, 16, 8, 3072, 4096)
_4B = _dims(2560, 32, 8, 9728, 4096)
MANY_ROWS = [
    (_06B, [2048, 2049], 2, dict(append=dict(qkv=("tile256", 4, 1, "qkv"), o=("wide128", 4, 2, "store")),     # 4095 rows: last tile one row short
                                 recompute=dict(qkv=("wide128", 4, 1, "qkv"), down=("wide128", 4, 1, "add")))),   # 4099 rows: 3 rows in the last tile
    (_06B, [3713], 2, dict(append=dict(qkv=("tile256", 4, 1, "qkv")), recompute=dict(down=("wide128", 4, 2, "store")))),
    (_dims(2560, 8, 1, 1088, 32768), [5, 3000], 130, dict(recompute=dict(qkv=("wide128", 4, 1, "qkv"), o=("tile256", 4, 1, "add")),
                                                          score=dict(score_head=("tile256", 4, 1, "logprob")))),
    (_4B, [300, 288], 1, dict(append=dict(qkv=("wide128", 4, 2, "store"), o=("wide128", 4, 5, "store"), gate_up=("tile256", 4, 1, "swiglu")))),
    (_4B, [130, 3], 1, dict(append=dict(qkv=("wide128", 4, 5, "store"), o=("tile128", 0, 6, "store"), gate_up=("wide128", 4, 1, "swiglu")))),
    (_dims(2560, 4, 1, 256), [3950, 3907], 0, dict(append=dict(qkv=("wide128", 4, 1, "qkv"), o=("tile128", 0, 1, "store"),
                                                               gate_up=("tile128", 0, 1, "swiglu")))),
    (_dims(2560, 31, 31, 9728, 4096), [901], 1, dict(append=dict(qkv=("tile256", 4, 1, "qkv"), gate_up=("tile256", 5, 1, "swiglu")))),
]

# widths that end inside a tile, many short trajectories (a few of them go through the oracle)
MANY_ROWS_ORACLE = [
    (_dims(640, 16, 8, 640, 1056), split(2049), 2, dict(append=dict(qkv=("tile256", 4, 1, "qkv")))),                  # one row in the last tile
    (_dims(640, 7, 7, 256), split(5000), 1, dict(append=dict(qkv=("tile256", 4, 1, "qkv")))),                         # 21 heads in tiles of two
    (_dims(256, 5, 5, 1088, 4096), split(2500), 2, dict(append=dict(qkv=("wide128", 4, 1, "qkv")))),                  # 15 heads
    (_dims(256, 32, 8, 1472, 1056), split(700), 2, dict(append=dict(qkv=("wide128", 4, 1, "qkv")))),                  # groups of 4, 60 rows in the last tile
    (_dims(2240, 2, 1, 640, 1056), split(3713), 1, dict(append=dict(down=("tile256", 4, 1, "add")))),                 # 192 of 256 columns
    (_dims(2496, 1, 1, 704), split(7855), 1, dict(append=dict(down=("tile256", 5, 1, "add")))),                       # 256 of 320 columns
    (_dims(2240, 6, 3, 256), split(8180), 1, dict(append=dict(o=("tile256", 5, 1, "add")))),
    (_dims(1664, 1, 1, 256), split(2500), 1, dict(append=dict(down=("wide128", 4, 1, "add")))),                       # 128 of 256 columns
    (_dims(128, 4, 1, 320, 1056), split(1153), 2, dict(append=dict(o=("tile256", 4, 2, "store")))),
    (_dims(2432, 4, 1, 2688), split(3713), 1, dict(append=dict(down=("tile256", 5, 2, "store")))),                    # 192 of 320 columns
    (_dims(128, 16, 2, 256), split(1153), 2, dict(append=dict(o=("wide128", 4, 7, "store")))),                        # seven slices
    (_dims(576, 1, 1, 8256, 1056), split(385), 1, dict(append=dict(gate_up=("tile256", 4, 1, "swiglu")))),
    (_dims(704, 2, 2, 9536, 4096), split(900), 1, dict(append=dict(gate_up=("tile256", 5, 1, "swiglu")))),
    (_dims(256, 6, 3, 8384, 4128), split(130), 1, dict(append=dict(gate_up=("wide128", 4, 1, "swiglu")))),
    (_dims(1152, 2, 1, 320, 4128), split(900) + [20] * 30, 22, dict(score=dict(score_head=("tile256", 4, 1, "logprob")))),   # 129 strips in tiles of 8
]

DECODE_ROWS = [1, 15, 17, 32, 33, 64, 65, 128, 129]
DECODE = [
    dict(),
    dict(hidden=2560, n_q_heads=8, n_kv_heads=1, intermediate=1088, vocab=4128),
    dict(hidden=4096, n_q_heads=4, n_kv_heads=4, intermediate=4096, vocab=4096),
    dict(hidden=4160, n_q_heads=4, n_kv_heads=4, intermediate=1024, vocab=4096),   # the norms' looping form
    _dims(128, 2, 1, 4160),
    _dims(1216, 8, 8, 512),
    _dims(128, 1, 1, 8256),         # gate-up ends inside a tile of 80 columns
    _dims(1408, 32, 8, 640),        # 80-column tiles with slices of unequal length
    _dims(2368, 2, 1, 2944),
    _dims(128, 2, 2, 10496),        # gate-up ends inside a tile of 96 columns
    _dims(3392, 24, 3, 448),        # 96-column tiles with slices of unequal length
    _dims(1536, 8, 8, 384),
    _dims(3392, 16, 2, 256),
    _dims(2816, 10, 5, 192),        # QKV: 80 columns, slices of unequal length, at most 64 rows
    _dims(1536, 14, 7, 256),        # QKV ends inside a tile of 96 columns, at most 64 rows
    _dims(2048, 11, 11, 256),       # QKV: 53 tiles in four slices, numbered by XCD with a remainder
    _dims(2112, 22, 11, 256),       # 59 tiles
]

# O and down with the residual add and the norm inside, two layers so that every consumer of the undivided rows runs
RESIDUAL_ROWS = [1, 16, 17, 33, 64, 65, 128, 129, 300, 512]
RESIDUAL = [
    _dims(64, 1, 1, 64),            # K of two 32-k steps: waves without any
    _dims(320, 3, 3, 448),          # K = 384 and 448: the waves' shares differ
    _dims(1024, 16, 8, 3072),
    _dims(2560, 32, 8, 1088),
    _dims(4096, 2, 2, 4096),        # 256 column blocks
    _dims(4160, 4, 4, 1024),        # 260: two rounds of the narrowest tile
    _dims(4160, 1, 1, 3072),        # down: 24 MB of weights, which one row tile reads past the caches
]
