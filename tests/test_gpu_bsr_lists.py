"""The block-sparse product over the list lengths at which it changes path:
tile rows with more key tiles than LDS holds (1024), lists too long for the
meeting test (64), a short list against a long one on either side, odd
widths, and more column tiles than one workgroup takes (256).  Integer values, so
every sum is exact and the dense form must agree bit for bit."""
import pytest
import torch

from paper_2112_07552_amd import ops
from paper_2112_07552_amd import workloads as wl

from .gpu_util import cuda_or_skip

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N,na,nb", [
    (20, 40_000, 30, 60_000, 60_000),      # both lists long, X's beyond LDS
    (20, 40_000, 4990, 60_000, 15_000),    # short lists of Y against long ones of X
    (4990, 40_000, 20, 15_000, 60_000),    # and the other way round
    (700, 1_000, 4_099, 900, 5_000),       # odd width, two chunks
    (70_000, 300, 33, 60_000, 200),        # many tile rows
    (1, 1, 1, 3, 2),
])
def test_bsr_paths_match_dense_on_integers(M, K, N, na, nb):
    dev = cuda_or_skip()
    A = wl.random_relation(na, M, K, 21, 1, values="int", lo=-50, hi=50, device=dev)
    B = wl.random_relation(nb, N, K, 21, 2, values="int", lo=-50, hi=50, device=dev)
    args = (A.group, A.key, A.val, B.key, B.group, B.val, M, K, N)
    Cb, ws = ops.join_agg_bsr(*args)
    assert ops.sync_status(ws)[0] == 0
    Cd, _, _ = ops.join_agg_fwd(*args)
    assert torch.equal(Cb, Cd)
