"""FP64 products of operands with leading dimensions so large that a lane's
offset inside a stage of the contraction exceeds 32 bits.  Integer entries:
exact, compared for equality; what lies between the rows is NaN."""
import ctypes as C

import pytest
import torch

from paper_2112_07552_amd import _lib

from .gpu_util import cuda_or_skip

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("which", ["a", "b"])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("m,n,k", [(33, 35, 37), (70, 40, 131)])
def test_wide_leading_dimension(m, n, k, ta, tb, which):
    dev = cuda_or_skip()
    if torch.cuda.mem_get_info(dev)[0] < 64 << 30:
        pytest.skip("not enough GPU memory")
    L = _lib.load()
    gen = torch.Generator(dev).manual_seed(m + 2 * ta + tb)
    ops, lds = [], []
    for name, shape in (("a", (k, m) if ta else (m, k)), ("b", (n, k) if tb else (k, n))):
        rows, cols = shape
        # contraction along the rows: 32 rows in 2^32 bytes; else 16 of them
        ld = cols
        if name == which:
            contiguous = (name == "a" and not ta) or (name == "b" and tb)
            ld = (1 << 24) + 1 if contiguous else (1 << 25) + 1
        buf = torch.full(((rows - 1) * ld + cols,), float("nan"), dtype=torch.float64, device=dev)
        view = buf.as_strided((rows, cols), (ld, 1))
        view.copy_(torch.randint(-8, 9, shape, generator=gen, device=dev))
        ops.append(view)
        lds.append(ld)
    out = torch.full((m, n), float("nan"), dtype=torch.float64, device=dev)
    vp = C.c_void_p
    st = L.tcu_gemm_f64(ta, tb, m, n, k, vp(ops[0].data_ptr()), lds[0], vp(ops[1].data_ptr()),
                        lds[1], vp(out.data_ptr()), n,
                        vp(torch.cuda.current_stream().cuda_stream))
    assert st == 0
    a, b = (o.contiguous() for o in ops)
    want = (a.t() if ta else a).contiguous() @ (b.t() if tb else b).contiguous()
    assert torch.equal(out, want)
