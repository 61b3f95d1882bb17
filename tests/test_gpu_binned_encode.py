"""SUM and COUNT over relations with repeated cells through tiles summed in
LDS, against a dense torch product of integer-valued encodings (every partial
sum an integer below 2^53: compared for equality).  Shapes around the tiles (16
to 32 rows, 16 to 256 columns) and the planes' padding (128 lines, 32 keys),
many records in few cells (multiplicities beyond int8), skipped records, both
value types and none, and saved encodings for the adjoint."""
import pytest
import torch

from paper_2112_07552_amd import ops

from .gpu_util import cuda_or_skip

pytestmark = pytest.mark.gpu


def table(n, groups, keys, dtype, seed, dev, outside=0, hot=0.0):
    g = torch.Generator(device=dev).manual_seed(seed)
    r = torch.randint(0, groups, (n,), generator=g, device=dev, dtype=torch.int32)
    c = torch.randint(0, keys, (n,), generator=g, device=dev, dtype=torch.int32)
    if hot:
        at = torch.rand(n, generator=g, device=dev) < hot
        r[at], c[at] = 0, keys - 1
    if outside:
        r[:outside] = -1
        c[-outside:] = keys
    v = None if dtype is None else torch.randint(-8, 9, (n,), generator=g, device=dev).to(dtype)
    return r, c, v


def dense(r, c, v, rows, cols):
    ok = (r >= 0) & (r < rows) & (c >= 0) & (c < cols)
    r, c = r[ok].long(), c[ok].long()
    w = torch.ones(r.numel(), dtype=torch.float64, device=r.device) if v is None else v[ok].double()
    Z = torch.zeros(rows * cols, dtype=torch.float64, device=r.device)
    return Z.index_add_(0, r * cols + c, w).reshape(rows, cols)


@pytest.mark.parametrize("M,K,N,na,nb,outside,hot", [
    (1, 1, 1, 140_000, 400_001, 0, 0.0),
    (16, 16, 16, 500_000, 70_000, 3, 0.0),
    (17, 33, 129, 350_000, 250_000, 7, 0.0),
    (100, 4097, 31, 600_000, 5, 1, 0.0),
    (513, 255, 257, 524_287, 1, 0, 0.0),
    (1000, 1537, 700, 400_003, 300_001, 11, 0.0),
    (2100, 600, 3000, 300_000, 500_000, 0, 0.01),
    (1030, 1025, 1100, 2_000, 3_000, 2, 0.0),
])
@pytest.mark.parametrize("dta,dtb", [(torch.float64, torch.float32), (None, torch.float64),
                                     (None, None)])
@pytest.mark.parametrize("count", [False, True])
def test_sums_and_counts(M, K, N, na, nb, outside, hot, dta, dtb, count):
    dev = cuda_or_skip()
    ga, ka, va = table(na, M, K, dta, 1, dev, outside, hot)
    gb, kb, vb = table(nb, N, K, dtb, 2, dev, min(outside, nb - 1), hot)
    C, cnt, ws = ops.join_agg_fwd(ga, ka, va, kb, gb, vb, M, K, N, with_count=count)
    X, Y = dense(ga, ka, va, M, K), dense(kb, gb, vb, K, N)
    assert torch.equal(C, X @ Y)
    if count:
        want = dense(ga, ka, None, M, K) @ dense(kb, gb, None, K, N)
        assert torch.equal(cnt.double(), want.clamp(max=2.0 ** 31 - 1))
    st, info = ops.sync_status(ws)
    bad_a = int(((ga < 0) | (ka >= K)).sum())
    bad_b = int(((gb < 0) | (kb >= K)).sum())
    assert (info["skipped_a"], info["skipped_b"]) == (bad_a, bad_b)


def test_adjoint_after_the_tiles():
    """The encodings left for the adjoint are the sums, also after a count
    whose multiplicities exceed int8."""
    dev = cuda_or_skip()
    M, K, N = 300, 200, 150
    ga, ka, va = table(300_000, M, K, torch.float64, 3, dev, 0, 0.2)
    gb, kb, vb = table(300_000, N, K, torch.float64, 4, dev, 0, 0.2)
    W = torch.randint(-4, 5, (M, N), device=dev).double()
    for count in (False, True):
        _, _, ws = ops.join_agg_fwd(ga, ka, va, kb, gb, vb, M, K, N, with_count=count,
                                    for_backward=True)
        dA, dB, _ = ops.join_agg_bwd(ga, ka, va, kb, gb, vb, M, K, N, W, ws=ws,
                                     saved_encodings=True)
        X, Y = dense(ga, ka, va, M, K), dense(kb, gb, vb, K, N)
        assert torch.equal(dA, (W @ Y.t().contiguous())[ga.long(), ka.long()])
        assert torch.equal(dB, (X.t().contiguous() @ W)[kb.long(), gb.long()])
