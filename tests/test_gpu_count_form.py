"""COUNT over relations with unique cells: the product of the two 0/1
encodings on int8 planes.  Exact: equal to a torch product of the same 0/1
matrices, over tile edges (128 rows and columns, 32 keys), a shape too small
for the planes (which stays on the FP64 matrix cores), a result larger than
the last-level cache, skipped records, and with the pair counts beside it.
The adjoint with saved encodings rebuilds them, as this form keeps none."""
import pytest
import torch

from paper_2112_07552_amd import ops

from .gpu_util import cuda_or_skip

pytestmark = pytest.mark.gpu


def table(groups, keys, density, seed, dev):
    """Records of a random 0/1 matrix (groups x keys), and the matrix."""
    g = torch.Generator(device=dev).manual_seed(seed)
    Z = (torch.rand((groups, keys), generator=g, device=dev) < density)
    r, c = torch.nonzero(Z, as_tuple=True)
    return r.int(), c.int(), Z.double()


@pytest.mark.parametrize("M,K,N,density", [
    (1, 1, 1, 1.0), (3, 7, 5, 0.5), (128, 32, 128, 0.3), (129, 33, 127, 0.3), (257, 500, 385, 0.2),
    (1000, 1, 2000, 0.5), (130, 4097, 70, 0.4), (6001, 40, 6003, 0.1),
])
@pytest.mark.parametrize("count", [False, True])
def test_count_form_exact(M, K, N, density, count):
    dev = cuda_or_skip()
    ag, ak, X = table(M, K, density, M + K, dev)
    bg, bk, Y = table(N, K, density, N + 2 * K, dev)
    C, cnt, ws = ops.join_agg_fwd(ag, ak, None, bk, bg, None, M, K, N, with_count=count,
                                  unique=True)
    assert ops.sync_status(ws)[0] == 0
    want = torch.matmul(X, Y.t().contiguous())
    assert torch.equal(C, want)
    if count:
        assert torch.equal(cnt, want.int())


def test_count_form_skips_and_adjoint():
    dev = cuda_or_skip()
    M, K, N = 200, 90, 150
    ag, ak, X = table(M, K, 0.3, 1, dev)
    bg, bk, Y = table(N, K, 0.3, 2, dev)
    bad = torch.tensor([-1, M, 0, 5], dtype=torch.int32, device=dev)
    badk = torch.tensor([0, 0, K, -9], dtype=torch.int32, device=dev)
    ag2, ak2 = torch.cat([ag, bad]), torch.cat([ak, badk])
    bg2, bk2 = torch.cat([bad[2:], bg]), torch.cat([badk[2:], bk])
    C, _, ws = ops.join_agg_fwd(ag2, ak2, None, bk2, bg2, None, M, K, N, unique=True,
                                for_backward=True)
    st, info = ops.sync_status(ws)
    assert st == ops._lib.TCU_ERR_KEY_RANGE
    assert (info["skipped_a"], info["skipped_b"]) == (4, 2)
    assert torch.equal(C, torch.matmul(X, Y.t().contiguous()))
    W = torch.randint(-8, 9, (M, N), device=dev).double()  # integer sums are exact
    dA, dB, _ = ops.join_agg_bwd(ag2, ak2, None, bk2, bg2, None, M, K, N, W, ws=ws, unique=True,
                                 saved_encodings=True)
    dX, dY = torch.matmul(W, Y), torch.matmul(W.t().contiguous(), X)
    assert torch.equal(dA, torch.cat([dX[ag.long(), ak.long()], torch.zeros(4, device=dev).double()]))
    assert torch.equal(dB, torch.cat([torch.zeros(2, device=dev).double(), dY[bg.long(), bk.long()]]))
