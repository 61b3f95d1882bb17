"""FP64 products of few output tiles and a long contraction, on every way they
can be split: chunks on 128 x 128 tiles (remainders of the last chunk around
one stage of 16), on 32 x 64 and 32 x 32 tiles, and in one piece.

Integer entries of magnitude at most 8 and k below 2^20: every partial sum is
an integer below 2^53, so the result is exact in any order and compared for
equality."""
import ctypes as C

import pytest
import torch

from paper_2112_07552_amd import _lib, ops

from .test_gpu_gemm_sizes import _matrix

pytestmark = pytest.mark.gpu

SIZES = [(300, 500, 20161), (300, 500, 20176), (300, 500, 20001), (129, 131, 20129),
         (129, 131, 70001), (1024, 128, 20512), (128, 1024, 65537), (768, 770, 8193),
         (100, 1500, 30001), (333, 777, 3333), (640, 1024, 2049), (16, 17, 100003),
         (1400, 1408, 1031)]


@pytest.mark.parametrize("pad,shift", [(0, 0), (1, 1)])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("m,n,k", SIZES)
def test_split_products(m, n, k, ta, tb, pad, shift):
    L = _lib.load()
    gen = torch.Generator("cuda").manual_seed(m * 7919 + n * 31 + k)
    A, lda = _matrix(*((k, m) if ta else (m, k)), pad, shift, gen)
    B, ldb = _matrix(*((n, k) if tb else (k, n)), pad, shift, gen)
    out = torch.full((m, n + pad), float("nan"), dtype=torch.float64, device="cuda")
    nb = int(L.tcu_gemm_f64_workspace_bytes(m, n, k))
    assert nb > 0
    ws = torch.full((nb // 8,), float("nan"), dtype=torch.float64, device="cuda")
    vp = C.c_void_p
    st = L.tcu_gemm_f64_ws(ta, tb, m, n, k, vp(A.data_ptr()), lda, vp(B.data_ptr()), ldb,
                           vp(out.data_ptr()), n + pad, vp(ws.data_ptr()), nb,
                           vp(torch.cuda.current_stream().cuda_stream))
    assert st == 0
    want = (A.t() if ta else A).contiguous() @ (B.t() if tb else B).contiguous()
    assert torch.equal(out[:, :n], want)
    assert bool(torch.isnan(out[:, n:]).all())


def _time(m, n, k, tb):
    A = torch.ones((m, k), dtype=torch.float64, device="cuda")
    B = torch.ones((n, k) if tb else (k, n), dtype=torch.float64, device="cuda")
    out = torch.empty((m, n), dtype=torch.float64, device="cuda")
    best = float("inf")
    for _ in range(8):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(4):
            ops.gemm_f64(A, B, trans_b=tb, out=out)
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


@pytest.mark.parametrize("tb", [False, True])
@pytest.mark.parametrize("m,n,k", [(1024, 128, 65536), (512, 512, 32768)])
def test_a_deep_product_fills_the_chip(m, n, k, tb):
    """A product of the work of 2048^3 (256 whole tiles) with a small output
    takes at most 1.5 times its time (1.1 to 1.2 measured; 1.5 to 2.0 where its
    contraction is not split far enough)."""
    assert m * n * k == 2048 ** 3
    assert _time(m, n, k, tb) <= 1.5 * _time(2048, 2048, 2048, tb)
