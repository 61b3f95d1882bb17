"""The dictionary at the sizes where its kernels change path: one sorted run
or several (2048 values), one merge pass or two (16384), the small hash table
or the full one (131072 values), codes from LDS or from memory (2048 distinct
values in 2^19 records).  Integer work, bit-exact against numpy."""
import numpy as np
import pytest
import torch

from paper_2112_07552_amd import ops

from .gpu_util import cuda_or_skip

pytestmark = pytest.mark.gpu

I64MIN, I64MAX = np.iinfo(np.int64).min, np.iinfo(np.int64).max


@pytest.mark.parametrize("n,distinct", [
    (1, 1), (63, 63), (3000, 2047), (3000, 2048), (3000, 2049), (3000, 1023), (3000, 1024), (3000, 1025), (20_000, 16_384),
    (20_000, 16_385), (131_072, 131_072), (140_000, 131_072), (140_000, 131_073),
    (600_000, 200_001), (1 << 19, 2048), (1 << 19, 2049), ((1 << 19) + 3, 7),
])
@pytest.mark.parametrize("low", [False, True])
def test_dictionary_at_path_edges(n, distinct, low):
    dev = cuda_or_skip()
    rng = np.random.default_rng(n * 31 + distinct)
    pool = np.unique(rng.integers(I64MIN + 1, I64MAX, 2 * distinct + 8, dtype=np.int64))
    pool = rng.permutation(pool)[:distinct]
    pool[0] = I64MAX
    if low:
        pool[-1] = I64MIN
    vals = rng.permutation(pool[np.arange(n) % distinct])
    a, b = vals[: n // 3], vals[n // 3:]
    want, codes = np.unique(vals, return_inverse=True)
    d, ca, cb = ops.dict_encode(torch.from_numpy(a).to(dev), torch.from_numpy(b.copy()).to(dev))
    assert np.array_equal(d.cpu().numpy(), want)
    assert np.array_equal(torch.cat([ca, cb]).cpu().numpy(), codes)
