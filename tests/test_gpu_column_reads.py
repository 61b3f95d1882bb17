"""Encoding and gathering on both sides of the size from which record columns
are read past the caches (72 MiB of columns and matrix), with unique and with
repeated cells, each value type, both placements and skipped records.  Integer
values: compared for equality."""
import pytest
import torch

from paper_2112_07552_amd import ops

from .gpu_util import cuda_or_skip

pytestmark = pytest.mark.gpu


def table(n, groups, keys, dtype, dev, unique):
    g = torch.Generator(device=dev).manual_seed(n + keys)
    if unique:
        cell = torch.randperm(groups * keys, generator=g, device=dev)[:n]
    else:
        cell = torch.randint(0, groups * keys, (n,), generator=g, device=dev)
        cell[n // 2:] = cell[:n - n // 2].clone()
    r, c = (cell // keys).int(), (cell % keys).int()
    r[0], c[-1] = groups, -1
    v = None if dtype is None else torch.randint(-8, 9, (n,), generator=g, device=dev).to(dtype)
    return r, c, v


def dense(r, c, v, rows, cols):
    ok = (r >= 0) & (r < rows) & (c >= 0) & (c < cols)
    w = torch.ones(r.numel(), dtype=torch.float64, device=r.device) if v is None else v.double()
    Z = torch.zeros(rows * cols, dtype=torch.float64, device=r.device)
    return Z.index_add_(0, r[ok].long() * cols + c[ok].long(), w[ok]).reshape(rows, cols)


@pytest.mark.parametrize("rows,cols", [(3072, 3071), (3072, 3072), (2711, 2709)])
@pytest.mark.parametrize("n", [2, 5000, 1_048_577])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32, None])
@pytest.mark.parametrize("unique", [False, True])
@pytest.mark.parametrize("transpose", [False, True])
def test_encode(rows, cols, n, dtype, unique, transpose):
    dev = cuda_or_skip()
    r, c, v = table(n, rows, cols, dtype, dev, unique)
    want = dense(r, c, v, rows, cols)
    g, k = (c, r) if transpose else (r, c)
    got = ops.encode(g, k, v, rows, cols, transpose=transpose, unique=unique)
    assert torch.equal(got, want)


@pytest.mark.parametrize("M,K", [(2709, 2709), (2711, 2709)])
@pytest.mark.parametrize("unique", [False, True])
def test_gradients(M, K, unique):
    dev = cuda_or_skip()
    N, n = 3, 1_048_577
    ga, ka, va = table(n, M, K, torch.float64, dev, unique)
    gb, kb, vb = table(4000, N, K, torch.float64, dev, unique)
    g = torch.Generator(device=dev).manual_seed(5)
    W = torch.randint(-3, 4, (M, N), generator=g, device=dev).double()
    da, db = ops.join_agg_bwd(ga, ka, va, kb, gb, vb, M, K, N, W)[:2]
    X, Y = dense(ga, ka, va, M, K), dense(kb, gb, vb, K, N)
    dX, dY = W @ Y.t().contiguous(), X.t().contiguous() @ W
    for got, src, r, c in ((da, dX, ga, ka), (db, dY, kb, gb)):
        ok = (r >= 0) & (r < src.shape[0]) & (c >= 0) & (c < src.shape[1])
        want = torch.zeros(r.numel(), dtype=torch.float64, device=dev)
        want[ok] = src[r[ok].long(), c[ok].long()]
        assert torch.equal(got, want)
