"""Relations of so many records that both together exceed the 2^32 work-items
of one launch, while each alone does not.  Every record falls on one cell and
carries the same value, so declared unique (plain stores) the cell holds that
value; the columns of both relations share one tensor."""
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
