"""The block-sparse operator's tiles found by bits, and by the dictionary beyond
the bits' limits, against a dense torch product of integer-valued encodings
(exact in any order).  Key tiles around the 64-bit words, tile rows around the
scan's rounds of 1024 and around its limit of 65536, skipped records, repeated
and unique cells, both value types and none."""
import pytest
import torch

from paper_2112_07552_amd import ops

from .gpu_util import cuda_or_skip

pytestmark = pytest.mark.gpu


def table(n, groups, keys, dtype, seed, dev, outside):
    g = torch.Generator(device=dev).manual_seed(seed)
    r = torch.randint(0, groups, (n,), generator=g, device=dev, dtype=torch.int32)
    c = torch.randint(0, keys, (n,), generator=g, device=dev, dtype=torch.int32)
    # the corners, so that the first and the last tile are there
    r[0], c[0], r[-1], c[-1] = 0, 0, groups - 1, keys - 1
    if outside and n > 4:
        r[1], c[2] = -1, keys
    v = None if dtype is None else torch.randint(-8, 9, (n,), generator=g, device=dev).to(dtype)
    return r, c, v


def dense(r, c, v, rows, cols, unique):
    ok = (r >= 0) & (r < rows) & (c >= 0) & (c < cols)
    r, c = r[ok].long(), c[ok].long()
    w = torch.ones(r.numel(), dtype=torch.float64, device=r.device) if v is None else v[ok].double()
    Z = torch.zeros(rows * cols, dtype=torch.float64, device=r.device)
    return Z.index_add_(0, r * cols + c, w).reshape(rows, cols)


@pytest.mark.parametrize("M,K,N,na,nb,outside", [
    (1, 1, 1, 1, 1, False), (16, 16, 17, 30, 20, False), (33, 1023, 47, 900, 1000, True),
    (100, 1024, 100, 5000, 300, False), (100, 1025, 31, 800, 5000, True),
    (257, 20_000, 130, 3000, 4000, False), (16_384, 600, 40, 20_000, 2000, False),
    (16_400, 70, 50, 30_000, 500, True), (1_048_577, 40, 20, 50_000, 300, False),
])
@pytest.mark.parametrize("dta,dtb", [(torch.float64, torch.float32), (None, None)])
def test_tiles_at_the_edges(M, K, N, na, nb, outside, dta, dtb):
    dev = cuda_or_skip()
    ga, ka, va = table(na, M, K, dta, 1, dev, outside)
    gb, kb, vb = table(nb, N, K, dtb, 2, dev, outside)
    C, ws = ops.join_agg_bsr(ga, ka, va, kb, gb, vb, M, K, N)
    assert torch.equal(C, dense(ga, ka, va, M, K, False) @ dense(kb, gb, vb, K, N, False))
    _, info = ops.sync_status(ws)
    assert (info["skipped_a"], info["skipped_b"]) == (
        int(((ga < 0) | (ka >= K)).sum()), int(((gb < 0) | (kb >= K)).sum()))


@pytest.mark.parametrize("M,K,N", [(300, 1100, 200), (1_048_600, 33, 17)])
def test_unique_cells(M, K, N):
    dev = cuda_or_skip()
    g = torch.Generator(device=dev).manual_seed(9)
    at = torch.unique(torch.randint(0, M * K, (40_000,), generator=g, device=dev))
    bt = torch.unique(torch.randint(0, K * N, (400,), generator=g, device=dev))
    va = torch.randint(-8, 9, (at.numel(),), generator=g, device=dev).double()
    vb = torch.randint(-8, 9, (bt.numel(),), generator=g, device=dev).double()
    ga, ka = (at // K).int(), (at % K).int()
    kb, gb = (bt // N).int(), (bt % N).int()
    C, _ = ops.join_agg_bsr(ga, ka, va, kb, gb, vb, M, K, N, unique=True)
    assert torch.equal(C, dense(ga, ka, va, M, K, True) @ dense(kb, gb, vb, K, N, True))
