"""The dictionary on each of its hash tables: the small one (2^18 slots), the
next (2^21) and the full one (twice the values), reached by the number of
distinct values or by values that fall on neighbouring slots.  Integer work,
bit-exact against numpy."""
import numpy as np
import pytest
import torch

from paper_2112_07552_amd import ops

from .gpu_util import cuda_or_skip

pytestmark = pytest.mark.gpu


def check(vals):
    dev = cuda_or_skip()
    want, codes = np.unique(vals, return_inverse=True)
    k = vals.size // 3
    d, ca, cb = ops.dict_encode(torch.from_numpy(vals[:k].copy()).to(dev),
                                torch.from_numpy(vals[k:].copy()).to(dev))
    assert np.array_equal(d.cpu().numpy(), want)
    assert np.array_equal(torch.cat([ca, cb]).cpu().numpy(), codes)


@pytest.mark.parametrize("n,distinct", [
    (1_100_000, 1 << 20), (1_100_000, (1 << 20) + 1), (1_100_000, 1_100_000),
    (2_200_000, 1_700_000), (1 << 20, 1 << 20), ((1 << 20) + 1, (1 << 20) + 1),
])
def test_many_distinct_values(n, distinct):
    rng = np.random.default_rng(n + distinct)
    pool = np.unique(rng.integers(-(2 ** 62), 2 ** 62, 2 * distinct, dtype=np.int64))
    check(rng.permutation(rng.permutation(pool)[:distinct][np.arange(n) % distinct]))


def unmix(h):
    """Inverse of MurmurHash3's 64-bit finaliser, the slot hash."""
    h = h ^ (h >> np.uint64(33))
    h *= np.uint64(pow(0xc4ceb9fe1a85ec53, -1, 1 << 64))
    h ^= h >> np.uint64(33)
    h *= np.uint64(pow(0xff51afd7ed558ccd, -1, 1 << 64))
    return h ^ (h >> np.uint64(33))


@pytest.mark.parametrize("bits", [18, 21])
@pytest.mark.parametrize("colliding,others", [(64, 0), (65, 0), (300, 500), (1500, 0),
                                              (200, 100_000)])
def test_values_of_one_slot(bits, colliding, others):
    """`colliding` values with the same slot in a table of 2^bits: from 65 on
    the probes run out and the next table is tried, also for a dictionary of
    few values."""
    rng = np.random.default_rng(bits + colliding)
    same = unmix((np.arange(colliding, dtype=np.uint64) << np.uint64(bits)) + np.uint64(12345))
    pool = np.concatenate([same.view(np.int64), rng.integers(-(2 ** 62), 2 ** 62, others,
                                                             dtype=np.int64)])
    check(rng.permutation(pool[np.arange(1_300_000) % pool.size]))
