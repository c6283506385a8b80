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


@pytest.mark.parametrize("n", [64, 512])
def test_complex_flush_is_summed_in_pairs(n):
    """One accepted move on A = (1 + i) H: the change is (Y - E) / R times a row of exact entries.  Y and R are sums
    of 2 n real terms, 0.18 (log2 2 n + 4) u^2 of their squares each and 2.0 to 2.5 u^2; products and the reciprocal
    add 0.2 u^2 each: 6.5 u^2 in all, the median over moves (R is near zero in some).  One chain along the row: 14."""
    require_gpu()
    rng = np.random.default_rng(n)
    a = (1 + 1j) * hadamard(n)
    b = (0.5 - 0.5j) * hadamard(n) / n
    var = []
    with dsu.ZWalker(a, 8) as w:
        w.set_flush_kernel(dsu.FLUSH_MFMA)
        assert np.array_equal(w.inverse(), b)
        for _ in range(24):
            row, e = rng.uniform(-1, 1, n) + 1j * rng.uniform(-1, 1, n), int(rng.integers(n))
            y = row.astype(np.clongdouble) @ b.astype(np.clongdouble)
            r = y[e]
            y[e] -= 1
            step = -np.outer(b[:, e], y / r)
            w.propose(e, row)
            w.accept()
            w.flush()
            d = w.inverse() - (b + step)
            var.append(float((np.abs(d) ** 2).mean() / (np.abs(step) ** 2).mean()))
            w.recompute(a)
    assert np.median(var) <= 6.5 * U**2
