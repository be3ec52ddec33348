"""GPU parity: bs_gemm_bf16_nt against the fp64 product, at the edges of its kernels' tiles.

Products of bf16 values are exact in fp32, so the only error is that of at most K + 2 fp32 additions
(the accumulation in any order, the scale, the added C): |C - ref| <= (K + 2) 2^-24 (|A| |B|^T + |C0|)
per entry, the tolerance below.
"""
import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu


def product(lib, M, N, K, lda, ldb, shift, accumulate):
    g = torch.Generator().manual_seed(M * 7919 + N * 31 + K)
    # one guard row behind each operand: rows past M and N and columns past K hold NaN
    a = torch.full((M + 1, lda), float("nan"), dtype=torch.bfloat16)
    b = torch.full((N + 1, ldb), float("nan"), dtype=torch.bfloat16)
    a[:M, :K] = torch.randn(M, K, generator=g).to(torch.bfloat16)
    b[:N, :K] = torch.randn(N, K, generator=g).to(torch.bfloat16)
    c0 = torch.randn(M, N, generator=g)
    place = lambda t: torch.cat((torch.zeros(shift, dtype=t.dtype), t.reshape(-1))).cuda()[shift:]
    ad, bd, c = place(a), place(b), c0.cuda()
    print(f"[gemm] M={M} N={N} K={K} lda={lda} ldb={ldb} shift={shift} accumulate={accumulate}", flush=True)
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    rc = lib._gemm(p(ad), lda, p(bd), ldb, p(c), N, M, N, K, 0.5, int(accumulate), lib._stream())
    assert rc == 0
    torch.cuda.synchronize()
    A, B = a[:M, :K].double(), b[:N, :K].double()
    ref = 0.5 * (A @ B.T) + (c0.double() if accumulate else 0.0)
    bound = (K + 2) * 2.0 ** -24 * (A.abs() @ B.abs().T + (c0.double().abs() if accumulate else 0.0))
    err = (c.cpu().double() - ref).abs()
    assert bool((err <= bound).all()), float((err - bound).max())


@pytest.mark.parametrize("M,N,K", [
    (1, 1, 8), (31, 33, 72), (64, 64, 512), (65, 31, 1544),            # 32 x 32 tiles, fewer chunks than waves, K tails
    (300, 1000, 520), (129, 2750, 64), (1030, 900, 200),               # 128 x 128 tiles, one and several chunks
    (515, 4090, 1032), (2050, 2049, 136),                               # 256 x 256 tiles, ragged
])
@pytest.mark.parametrize("accumulate", [False, True])
def test_product_matches_fp64(lib, M, N, K, accumulate):
    product(lib, M, N, K, K, K, 0, accumulate)


@pytest.mark.parametrize("M,N,K,lda,ldb,shift", [
    (40, 72, 136, 144, 200, 0),     # padded rows: the columns past K are not read into the product
    (300, 600, 328, 336, 392, 0),
    (70, 150, 136, 136, 136, 4),    # 8-byte aligned operands: the register-staged kernel
    (300, 300, 264, 272, 264, 4),
])
def test_padded_and_unaligned_operands(lib, M, N, K, lda, ldb, shift):
    product(lib, M, N, K, lda, ldb, shift, False)
