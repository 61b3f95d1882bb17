"""The FP64 product at the edges of its tiles: rows, columns and contraction
lengths around 16, 32, 64 and 128, odd leading dimensions, operands that start
at an odd element, the split contraction and accumulation-free overwriting.

Integer entries of magnitude at most 8 and k below 2^20: every partial sum is
an integer below 2^53, so the result is exact in any order and compared for
equality."""
import ctypes as C

import pytest
import torch

from paper_2112_07552_amd import _lib

pytestmark = pytest.mark.gpu

SIZES = [(1, 1, 1), (1, 2, 3), (2, 1, 17), (15, 33, 16), (17, 31, 15), (32, 32, 64), (33, 65, 63),
         (31, 64, 65), (64, 1, 129), (1, 200, 100), (127, 129, 48), (128, 128, 16), (129, 130, 31),
         (200, 96, 1024), (33, 47, 1300), (300, 1001, 77), (700, 1500, 130),
         (1500, 1777, 301), (3969, 3971, 333)]


def _matrix(rows, cols, pad, shift, gen):
    """A rows x cols integer matrix inside a buffer of leading dimension cols +
    pad that starts at element `shift`; the rest of the buffer is NaN."""
    ld = cols + pad
    buf = torch.full((rows * ld + shift + 1,), float("nan"), dtype=torch.float64, device="cuda")
    view = buf[shift:shift + rows * ld].reshape(rows, ld)[:, :cols]
    view.copy_(torch.randint(-8, 9, (rows, cols), generator=gen, device="cuda"))
    return view, ld


@pytest.mark.parametrize("pad,shift", [(0, 0), (1, 1), (2, 0)])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("m,n,k", SIZES)
def test_product_at_tile_edges(m, n, k, ta, tb, pad, shift):
    L = _lib.load()
    gen = torch.Generator("cuda").manual_seed(m * 7919 + n * 31 + k)
    A, lda = _matrix(*((k, m) if ta else (m, k)), pad, shift, gen)
    B, ldb = _matrix(*((n, k) if tb else (k, n)), pad, shift, gen)
    out = torch.full((m, n + pad), float("nan"), dtype=torch.float64, device="cuda")
    nb = int(L.tcu_gemm_f64_workspace_bytes(m, n, k))
    ws = torch.empty(max(nb, 256), dtype=torch.uint8, device="cuda")
    vp = C.c_void_p
    st = L.tcu_gemm_f64_ws(ta, tb, m, n, k, vp(A.data_ptr()), lda, vp(B.data_ptr()), ldb,
                           vp(out.data_ptr()), n + pad, vp(ws.data_ptr()), ws.numel(),
                           vp(torch.cuda.current_stream().cuda_stream))
    assert st == 0
    want = (A.t() if ta else A).contiguous() @ (B.t() if tb else B).contiguous()
    assert torch.equal(out[:, :n], want)
    # the padding of C's rows is not written
    assert bool(torch.isnan(out[:, n:]).all())
