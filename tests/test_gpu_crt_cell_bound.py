"""The moduli of a large residue-form product (2^30 multiply-adds and more)
follow the largest bound of a cell's sum of |x||y|, computed here from the
encodings themselves, and not only the line sums.  Every row of X holds `c`
ones, every column of Y too, `d` of them on common keys: the truncations are
exact and every cell is d."""
import numpy as np
import pytest
import torch

from paper_2112_07552_amd import ops

from .gpu_util import cuda_or_skip

pytestmark = pytest.mark.gpu

M = K = N = 1024
TOL = 1e-12


def bounds(c, d):
    """(need, line sums' bound, cells' bound): a 1 is 0.5 * 2^1, its 7-bit
    magnitude 64."""
    T, s = 64 * 64 * d, 0.5 * c
    tcrt = (TOL - 2.0 ** -52) * (1 - 2.0 ** -40)
    r = 16384.0 * 2 * s * (1 + 2.0 ** -20)
    need = int(np.ceil(np.log2(r / (tcrt * T))))
    return need, s * (1 + 2.0 ** -20), (T + 128.0 * 2 * s) / 16384.0


def moduli(need, u):
    return ops.mixed_plan("crt_i8", K, TOL, need, u)[0]


def steps():
    """(c, d): the cells' bound takes one modulus more at d + 1 than at d, at
    the same width and a hundredth away from the step on both sides; and the
    line sums take more than at d."""
    found = []
    for c in range(64, 513, 8):
        for d in range(1, c):
            (need, line, cell), (need1, line1, cell1) = bounds(c, d), bounds(c, d + 1)
            if need != need1 or line < cell1 or moduli(need, line) <= moduli(need, cell):
                continue
            low, high = moduli(need, cell * (1 + 1e-5)), moduli(need, cell1 * (1 - 1e-5))
            if low == moduli(need, cell * (1 - 1e-5)) and high == low + 1 == \
                    moduli(need, cell1 * (1 + 1e-5)):
                found.append((c, d))
    return found


def ones(c, first, lines):
    dev = cuda_or_skip()
    line = torch.arange(lines, dtype=torch.int32, device=dev).repeat_interleave(c)
    key = torch.arange(first, first + c, dtype=torch.int32, device=dev).repeat(lines)
    return line, key, torch.ones(line.numel(), dtype=torch.float64, device=dev)


@pytest.mark.parametrize("which", [0, -1])
def test_moduli_around_a_step(which):
    cuda_or_skip()
    c, d = steps()[which]
    for e in (d, d + 1):
        need, line, cell = bounds(c, e)
        ga, ka, va = ones(c, 0, M)
        gb, kb, vb = ones(c, c - e, N)
        C, _, ws = ops.join_agg_fwd(ga, ka, va, kb, gb, vb, M, K, N, precision="crt_i8", tol=TOL,
                                    unique=True)
        st, info = ops.sync_status(ws)
        assert st == 0 and info["exceptions"] == 0
        assert info["bits"] == info["need"] == need
        assert info["slices"] == moduli(need, cell)
        assert bool((C == float(e)).all())
    assert moduli(need, cell) == moduli(need, bounds(c, d)[2]) + 1
    assert moduli(need, bounds(c, d)[1]) > moduli(need, bounds(c, d)[2])
