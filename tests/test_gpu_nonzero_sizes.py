"""nonzero() where its passes change path: chunks (4096 cells) at and around a
quarter full, a last chunk of one cell, and more chunks than one round of the
offset scan takes (8192).  Cells and order bit-exact against numpy."""
import numpy as np
import pytest
import torch

from paper_2112_07552_amd import ops

from .gpu_util import cuda_or_skip

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,cols,per_chunk", [
    (64, 64, 1024), (64, 64, 1025), (64, 64, 1), (17, 241, 4096), (241, 34, 900),
    (5900, 5801, 3), (3, 4096, 2000),
])
def test_nonzero_chunk_fill(rows, cols, per_chunk):
    dev = cuda_or_skip()
    total = rows * cols
    rng = np.random.default_rng(rows + per_chunk)
    flat = np.zeros(total)
    for c0 in range(0, total, 4096):
        n = min(4096, total - c0)
        flat[c0 + rng.choice(n, size=min(n, per_chunk), replace=False)] = rng.uniform(1, 2)
    flat[total - 1] = -3.0
    Z = flat.reshape(rows, cols)
    r, c, _ = ops.nonzero(torch.from_numpy(Z).to(dev))
    er, ec = np.nonzero(Z)
    assert np.array_equal(r.cpu().numpy(), er) and np.array_equal(c.cpu().numpy(), ec)
