"""The workspace queries grow with every size, so one buffer sized for a caller's largest call serves the
smaller ones (host arithmetic only; no GPU calls)."""
import ctypes
import os
import random

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2609_39813_amd", "libbsp.so")
pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="libbsp.so not built")

i32, i64 = ctypes.c_int, ctypes.c_int64
# query: argument types, (range, step) of the sizes that grow, how the call's arguments follow from them
QUERIES = {
    "norm": ("bs_rmsnorm_linear_workspace_size", [i64, i64, i64, i32, i32],
             [(1, 16384, 1), (8, 4096, 8), (8, 8192, 8), (1, 4096, 1)], lambda T, d, n, K: (T, d, n, 3, K)),
    "grid": ("bs_rmsnorm_linear_grid_workspace_size", [i64, i64, i64],
             [(1, 16384, 1), (8, 4096, 8), (8, 8192, 8)], lambda T, d, n: (T, d, n)),
    "attention": ("bs_attn_workspace_size", [i32] * 7,
                  [(1, 16, 1), (1, 32, 1), (1, 4096, 1), (1, 4096, 1)], lambda B, H, S, K: (B, H, S, 64, 3, K, 0)),
    "attention dK se": ("bs_attn_workspace_size", [i32] * 7,
                        [(1, 16, 1), (1, 32, 1), (1, 4096, 1), (1, 4096, 1)], lambda B, H, S, K: (B, H, S, 64, 3, K, 1)),
    "probability store": ("bs_attn_pstore_workspace_size", [i32] * 6,
                          [(1, 16, 1), (1, 32, 1), (4, 2048, 4), (1, 32, 1)], lambda B, H, S, K: (B, H, S, 64, K, 1)),
    "log-softmax": ("bs_logsoftmax_check_workspace_size", [i64, i32, i32],
                    [(1, 65536, 1), (4, 65536, 4), (1, 1 << 20, 1)], lambda r, C, K: (r, C, K)),
    "linear": ("bs_linear_bwd_workspace_size", [i64, i64, i64, i32, i32, i32],
               [(1, 16384, 1), (8, 4096, 8), (8, 8192, 8), (1, 4096, 1)], lambda M, k, n, K: (M, k, n, 2, K, 1)),
    "layer": ("bs_decoder_layer_workspace_size", [i32] * 7,
              [(1, 16, 1), (1, 4096, 1), (1, 32, 1), (8, 8192, 8), (1, 64, 1)],
              lambda B, S, H, F, K: (B, S, 64 * H, H, F, K, 0)),
    "layer all uses": ("bs_decoder_layer_workspace_size", [i32] * 7,
                       [(1, 16, 1), (1, 4096, 1), (1, 32, 1), (8, 8192, 8), (1, 64, 1)],
                       lambda B, S, H, F, K: (B, S, 64 * H, H, F, K, 1)),
    "layer per-use se": ("bs_decoder_layer_workspace_size", [i32] * 7,
                         [(1, 16, 1), (1, 4096, 1), (1, 32, 1), (8, 8192, 8), (1, 64, 1)],
                         lambda B, S, H, F, K: (B, S, 64 * H, H, F, K, 3)),
}
# neighbours across the limits where a launch takes fewer trials at a time, coarser tiles or fewer blocks
PAIRS = {
    "norm": [((1024, 1024, 1024, 256), (1088, 1024, 1024, 256)), ((1024, 1024, 1024, 32), (1024, 1024, 1088, 32)),
             ((1024, 1024, 1024, 128), (1024, 1024, 1024, 129)), ((64, 64, 64, 3), (64, 64, 64, 4)),
             ((8160, 256, 64, 32), (8200, 256, 64, 32))],
    "attention dK se": [((8, 16, 256, 16), (8, 16, 272, 16)), ((1, 16, 1024, 8), (1, 16, 1025, 8))],
    "log-softmax": [((1, 4, 4096), (1, 4, 4097)), ((100, 128, 4096), (100, 128, 4100))],
    "layer all uses": [((2, 256, 8, 1368, 8), (2, 258, 8, 1368, 8)), ((2, 256, 8, 1368, 8), (2, 256, 9, 1368, 8))],
    "layer per-use se": [((2, 256, 8, 1368, 8), (2, 258, 8, 1368, 8)), ((2, 512, 16, 1368, 16), (2, 512, 16, 1376, 17))],
}


def query(name):
    fn, types, ranges, args = QUERIES[name]
    f = getattr(ctypes.CDLL(LIB), fn)
    f.restype, f.argtypes = ctypes.c_size_t, types
    return (lambda *a: f(*args(*a))), ranges


@pytest.mark.parametrize("name", QUERIES)
def test_a_larger_shape_never_needs_less(name):
    q, ranges = query(name)
    rng = random.Random(name)

    def size(lo, hi, step):
        return max(lo, min(hi, round(lo * (hi / lo) ** rng.random() / step) * step))

    pairs = list(PAIRS.get(name, []))
    for _ in range(20000):
        a = [size(*r) for r in ranges]
        b = list(a)
        for i in rng.sample(range(len(a)), rng.choice((1, 1, 2, len(a)))):  # one size, some, or all of them
            lo, hi, step = ranges[i]
            b[i] = min(hi, a[i] + step * rng.choice((1, 2, 7, 33)) if rng.random() < 0.6 else size(a[i], hi, step))
        pairs.append((tuple(a), tuple(b)))
    for a, b in pairs:
        assert q(*a) > 0 and q(*b) >= q(*a), (name, a, q(*a), b, q(*b))
