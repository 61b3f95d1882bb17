"""Relations of so many records that both together exceed the 2^32 work-items
of one launch, while each alone does not.  Every record falls on one cell and
carries the same value, so declared unique (plain stores) the cell holds that
value; the columns of both relations share one tensor.  And products with so
many tiles."""
import pytest
import torch

from paper_2112_07552_amd import ops

from .gpu_util import cuda_or_skip

pytestmark = pytest.mark.gpu


def _columns(n, free_bytes):
    dev = cuda_or_skip()
    if torch.cuda.mem_get_info(dev)[0] < free_bytes:
        pytest.skip("not enough GPU memory")
    return torch.zeros(n, dtype=torch.int32, device=dev)


def test_sums_of_a_small_domain():
    g = _columns((1 << 31) + 4096, 20 << 30)
    C, _, ws = ops.join_agg_fwd(g, g, None, g, g, None, 1, 1, 1, unique=True)
    assert C.tolist() == [[1.0]]
    assert ops.sync_status(ws)[1]["skipped_a"] == 0


def test_pair_counts():
    g = _columns((1 << 31) + 4096, 20 << 30)
    C, count, _ = ops.join_agg_fwd(g, g, None, g, g, None, 130, 140, 150, unique=True,
                                   with_count=True)
    want = torch.zeros((130, 150), dtype=torch.float64, device=g.device)
    want[0, 0] = 1.0
    assert torch.equal(C, want) and torch.equal(count.double(), want)


def test_block_sparse():
    n = (1 << 31) - 1
    g = _columns(n, 140 << 30)
    v = torch.full((n,), 3.0, dtype=torch.float32, device=g.device)
    C, _ = ops.join_agg_bsr(g, g, v, g, g, v, 20, 30, 40, unique=True)
    want = torch.zeros((20, 40), dtype=torch.float64, device=g.device)
    want[0, 0] = 9.0
    assert torch.equal(C, want)


@pytest.mark.parametrize("ta,tb", [(False, False), (False, True), (True, False)])
@pytest.mark.parametrize("m,n", [((1 << 29) + 33, 3), (3, (1 << 29) + 33)])
def test_product_with_a_line_of_cells(m, n, ta, tb):
    """32 x 32 tiles of one line of 2^29 cells and more: as many workgroups of
    256 as 2^32 work-items and beyond."""
    dev = cuda_or_skip()
    if torch.cuda.mem_get_info(dev)[0] < 32 << 30:
        pytest.skip("not enough GPU memory")
    A = torch.full((2, m) if ta else (m, 2), 3.0, dtype=torch.float64, device=dev)
    B = torch.full((n, 2) if tb else (2, n), 5.0, dtype=torch.float64, device=dev)
    out = torch.zeros((m, n), dtype=torch.float64, device=dev)
    ops.gemm_f64(A, B, trans_a=ta, trans_b=tb, out=out)
    assert float(out.min()) == 30.0 and float(out.max()) == 30.0
