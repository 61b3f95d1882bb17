"""How long the chains of FP64 additions are inside a product whose
contraction is long against its output.

One entry of every row of op(A) is 2^56 and all others, and all of op(B), are
1.  Next to 2^56 a further 1 (or the four of one matrix instruction) is below
half a unit in the last place and is lost, so a cell's error counts the terms
added to the large one's chain after it.  The contraction of such outputs is
summed in chunks of at least 256 terms, as many chunks as give the chip two
workgroups of 128 x 128 cells per CU, so no chain may be longer than one
chunk; partial sums are multiples of 16, the unit in the last place of 2^56,
except around the large term itself (half a unit before it, half after)."""
import pytest
import torch

from paper_2112_07552_amd import ops

pytestmark = pytest.mark.gpu


def chunk(m, n, k):
    """Depth of a chunk: k over the parts, rounded up to whole stages of 16."""
    tiles = -(-m // 128) * -(-n // 128)
    parts = 1 if tiles >= 128 or k < 1024 else max(1, min(-(-512 // tiles), k // 256))
    return -(-(-(-k // parts)) // 16) * 16


@pytest.mark.parametrize("m,n,k", [
    (1024, 1024, 1024), (1024, 1024, 2048), (1024, 1024, 8192), (1408, 1408, 4096),
    (512, 512, 16384), (300, 500, 20032), (1024, 128, 65536), (768, 768, 8192), (64, 64, 4096),
    (100, 1500, 3008), (33, 47, 1344), (1000, 1001, 1088), (1024, 1024, 2063), (700, 900, 1030),
    (200, 200, 20015),
])
@pytest.mark.parametrize("ta,tb", [(False, False), (False, True), (True, False)])
def test_chains_are_no_longer_than_a_chunk(m, n, k, ta, tb):
    A = torch.ones((m, k), dtype=torch.float64, device="cuda")
    at = (torch.arange(m, device="cuda") * 16 * 7919) % k
    A[torch.arange(m, device="cuda"), at] = 2.0 ** 56
    B = torch.ones((n, k) if tb else (k, n), dtype=torch.float64, device="cuda")
    got = ops.gemm_f64(A.t().contiguous() if ta else A, B, trans_a=ta, trans_b=tb)
    lost = (k - 1) - (got - 2.0 ** 56)
    assert float(lost.abs().max()) <= chunk(m, n, k) + 16
