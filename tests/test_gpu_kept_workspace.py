"""What a forward keeps for its backward: a workspace of the size that the
backward asks for, also where the forward used scratch for relations that
repeat cells; the gradients from it are those of re-encoded records."""
import pytest
import torch

from paper_2112_07552_amd import ops

from .gpu_util import cuda_or_skip
from .test_gpu_binned_encode import table

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N,n", [(100, 90, 110, 700_000), (1000, 900, 1100, 600_000),
                                     (100, 90, 110, 1000)])
@pytest.mark.parametrize("count", [False, True])
def test_kept_workspace(M, K, N, n, count):
    dev = cuda_or_skip()
    ga, ka, va = table(n, M, K, torch.float64, 5, dev, 3)
    gb, kb, vb = table(n, N, K, torch.float64, 6, dev, 2)
    A, B = ops.make_relation(ga, ka, va), ops.make_relation(gb, kb, vb)
    _, _, ws = ops.join_agg_fwd(ga, ka, va, kb, gb, vb, M, K, N, with_count=count,
                                for_backward=True)
    assert ws.numel() == ops.workspace_bytes(A, B, M, K, N, backward=True, count=count)
    assert ops.sync_status(ws)[1]["skipped_a"] == 6
    W = torch.randint(-4, 5, (M, N), device=dev).double()
    got = ops.join_agg_bwd(ga, ka, va, kb, gb, vb, M, K, N, W, ws=ws, saved_encodings=True)
    want = ops.join_agg_bwd(ga, ka, va, kb, gb, vb, M, K, N, W)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


def test_memory_between_forward_and_backward():
    dev = cuda_or_skip()
    M, K, N, n = 100, 90, 110, 2_000_000
    ga, ka, va = table(n, M, K, torch.float64, 7, dev)
    gb, kb, vb = table(n, N, K, torch.float64, 8, dev)
    va.requires_grad_(True)
    A, B = ops.make_relation(ga, ka, va), ops.make_relation(gb, kb, vb)
    need = ops.workspace_bytes(A, B, M, K, N, backward=True)
    before = torch.cuda.memory_allocated(dev)
    C = ops.join_agg(ga, ka, va, kb, gb, vb, M, K, N, checkpoint=False)
    held = torch.cuda.memory_allocated(dev) - before
    assert held <= need + 8 * M * N + 4096
    C.sum().backward()
    assert va.grad.shape == (n,)
