"""Relations whose records fall into few of the tiles that are summed in LDS,
one workgroup per tile: against sums and products made on the CPU (integer
values, exact) and against the time of the same records placed one by one, which
is what a workspace without the scratch gives."""
import numpy as np
import pytest
import torch

from paper_2112_07552_amd import ops

from .gpu_util import cuda_or_skip
from .test_gpu_binned_encode import table

pytestmark = pytest.mark.gpu


def dense(r, c, v, rows, cols):
    at = r.cpu().numpy().astype(np.int64) * cols + c.cpu().numpy()
    w = None if v is None else v.cpu().numpy()
    Z = np.bincount(at, weights=w, minlength=rows * cols).reshape(rows, cols)
    return torch.from_numpy(Z.astype(np.float64)).to(r.device)


def fastest(f):
    best = float("inf")
    for _ in range(4):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        f()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


@pytest.mark.parametrize("M,K,N,spread", [(16, 16, 16, 16), (1000, 1000, 1000, 20),
                                          (1000, 1000, 1000, 1), (300, 5000, 40, 3)])
@pytest.mark.parametrize("count", [False, True])
def test_encodings(M, K, N, spread, count):
    dev = cuda_or_skip()
    n = 1 << 21
    ga, ka, va = table(n, spread, spread, torch.float64, 1, dev)
    gb, kb, vb = table(n, spread, spread, torch.float64, 2, dev)
    A, B = ops.make_relation(ga, ka, va), ops.make_relation(gb, kb, vb)
    ws = ops.alloc_workspace(ops.workspace_bytes(A, B, M, K, N, count=count), dev)
    big = ops.alloc_workspace(ops.workspace_bytes(A, B, M, K, N, count=count, scratch=True), dev)
    assert big.numel() > ws.numel()
    args = (ga, ka, va, kb, gb, vb, M, K, N)
    C, cnt, _ = ops.join_agg_fwd(*args, with_count=count, ws=big)
    assert torch.equal(C, dense(ga, ka, va, M, K) @ dense(kb, gb, vb, K, N))
    if count:
        want = dense(ga, ka, None, M, K) @ dense(kb, gb, None, K, N)
        assert torch.equal(cnt.double(), want.clamp(max=2.0 ** 31 - 1))
    tiles = fastest(lambda: ops.join_agg_fwd(*args, with_count=count, ws=big))
    single = fastest(lambda: ops.join_agg_fwd(*args, with_count=count, ws=ws))
    assert tiles <= 1.2 * single


@pytest.mark.parametrize("spread", [100, 1])
def test_histogram(spread):
    dev = cuda_or_skip()
    n, K, N = 1 << 21, 100_000, 50
    _, ka, va = table(n, 1, spread, torch.float64, 3, dev)
    ka += 4321
    gb, kb, vb = table(5000, N, spread, torch.float64, 4, dev)
    kb += 4321
    c, cnt, _ = ops.join_agg_row(ka, va, kb, gb, vb, K, N, with_count=True)
    key, kb, gb = ka.cpu().numpy(), kb.cpu().numpy(), gb.cpu().numpy()
    h = np.bincount(key, weights=va.cpu().numpy(), minlength=K)
    m = np.bincount(key, minlength=K)
    want = np.bincount(gb, weights=h[kb] * vb.cpu().numpy(), minlength=N)
    assert np.array_equal(c.cpu().numpy(), want)
    assert np.array_equal(cnt.cpu().numpy(), np.bincount(gb, weights=m[kb], minlength=N))
