"""Rounding errors of the host-driven moves' long sums, on matrices whose
inverse is exact: Sylvester's Hadamard matrix H (every elimination step is
exact in binary), H^{-1} = H / n.

An addition whose result has the variance v adds 0.18 u^2 v to the error's
(u = 2^-53; the mean over results spread between two powers of two).  n terms
of variance s^2 added four at a time and then in pairs: 0.18 u^2 s^2 n (log2 n),
less than 0.18 u^2 s^2 n (log2 n + 4) with short chains in between; one chain:
0.09 u^2 s^2 n^2, chains of 64 and one of the blocks 3.5 times the limit and more."""
import numpy as np
import pytest

from gpu_util import require_gpu
from paper_1708_00744_amd import dsu

pytestmark = pytest.mark.gpu

U = 2.0**-53


def hadamard(n):
    h = np.ones((1, 1))
    while len(h) < n:
        h = np.block([[h, h], [h, -h]])
    return h


@pytest.mark.parametrize("n,complex_", [(64, False), (512, False), (2048, False), (64, True), (512, True)])
def test_ratio_is_summed_in_pairs(n, complex_):
    require_gpu()
    rng = np.random.default_rng(n)
    h = hadamard(n)
    moves = 300
    phi, es = rng.uniform(-1, 1, (moves, n)), rng.integers(0, n, moves)
    with (dsu.ZWalker(h + 0j, 4) if complex_ else dsu.Walker(h, 4)) as w:
        assert np.array_equal(w.inverse(), h / n)
        err = []
        for row, e in zip(phi, es):
            r = w.propose(int(e), row + 0j if complex_ else row)
            w.reject()
            err.append(float(np.real(r) - (row.astype(np.longdouble) * h[e]).sum() / n))
    s2 = 1.0 / 3.0 / n**2  # of a term phi H / n
    assert np.mean(np.square(err)) <= 0.18 * U**2 * s2 * n * (np.log2(n) + 4)
