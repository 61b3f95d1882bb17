"""Q3 in re-associated form at the edges of its histograms: keys and groups
around the LDS limit (2048) and the copies of a bin, table lengths around the
workgroups' shares, many keys summed tile by tile (2^18 records and more) and by
global atomics (a workspace without the scratch), skipped records, no values.
Integer values: exact in any order."""
import ctypes as C

import pytest
import torch

from paper_2112_07552_amd import _lib, ops

from .gpu_util import cuda_or_skip

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("na,nb,K,N", [
    (1, 1, 1, 1), (2047, 2049, 64, 65), (5000, 4097, 2048, 33), (5000, 9000, 2049, 2048),
    (40_000, 40_000, 31, 2049), (262_143, 3000, 2049, 40), (262_144, 3000, 2049, 40),
    (600_001, 700_001, 100_003, 500), (600_001, 1000, 3_000_000, 7), (0, 100, 5000, 3),
])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32, None])
@pytest.mark.parametrize("outside", [0, 3])
def test_row_sums(na, nb, K, N, dtype, outside):
    dev = cuda_or_skip()
    g = torch.Generator(device=dev).manual_seed(na + K)

    def ints(lo, hi, n, dt=torch.int32):
        return torch.randint(lo, hi, (n,), generator=g, device=dev, dtype=dt)

    ka, kb, gb = ints(0, K, na), ints(0, K, nb), ints(0, N, nb)
    if outside and na > 3 and nb > 3:
        ka[:outside], kb[:1], gb[-1:] = K, -1, N
    av = None if dtype is None else ints(-8, 9, na).to(dtype)
    bw = None if dtype is None else ints(-8, 9, nb).to(dtype)
    oa = (ka >= 0) & (ka < K)
    ob = (kb >= 0) & (kb < K) & (gb >= 0) & (gb < N)
    one = lambda n: torch.ones(n, dtype=torch.float64, device=dev)
    va = one(na) if av is None else av.double()
    vb = one(nb) if bw is None else bw.double()
    h = torch.zeros(K, dtype=torch.float64, device=dev).index_add_(0, ka[oa].long(), va[oa])
    m = torch.zeros(K, dtype=torch.float64, device=dev).index_add_(0, ka[oa].long(), one(na)[oa])
    want = torch.zeros(N, dtype=torch.float64, device=dev)
    want.index_add_(0, gb[ob].long(), h[kb[ob].long()] * vb[ob])
    pairs = torch.zeros(N, dtype=torch.float64, device=dev)
    pairs.index_add_(0, gb[ob].long(), m[kb[ob].long()])
    c, cnt, ws = ops.join_agg_row(ka, av, kb, gb, bw, K, N, with_count=True)
    assert torch.equal(c, want) and torch.equal(cnt.double(), pairs)
    _, info = ops.sync_status(ws)
    assert (info["skipped_a"], info["skipped_b"]) == (int((~oa).sum()), int((~ob).sum()))
    # the same without the scratch
    L = _lib.load()
    A, B = ops.make_relation(ka, ka, av), ops.make_relation(gb, kb, bw)
    ws = ops.alloc_workspace(int(L.tcu_join_agg_row_workspace_bytes(K, N)), dev)
    c2 = torch.empty(N, dtype=torch.float64, device=dev)
    _lib.check(L.tcu_join_agg_row(C.byref(A), C.byref(B), K, N, C.c_void_p(c2.data_ptr()), None,
                                  C.c_void_p(ws.data_ptr()), ws.numel(),
                                  C.c_void_p(torch.cuda.current_stream().cuda_stream)), "row")
    assert torch.equal(c2, want)
