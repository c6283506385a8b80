"""The flush on both sides of the size from which its products are launched one by
one (padded rows: FP32 320 up to 32 slots, 256 at 64, 128 above; FP64 128 up to
32 slots, 64 above)."""
import numpy as np
import pytest

from gpu_util import require_gpu
from paper_1708_00744_amd import dsu, inputs
from test_gpu_edges import well_conditioned

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,k", [(192, 1), (320, 16), (321, 16), (310, 32), (385, 32), (256, 33), (257, 64), (128, 65),
                                 (129, 128)])
def test_fp32_flush_both_sides(n, k):
    require_gpu()
    a = well_conditioned(61 + n, n)
    noise = inputs.rows(62, k, n)
    order = np.random.default_rng(n).permutation(n)[:k]
    b = a.copy()
    with dsu.Walker(a, min(256, k + 1), precision=dsu.FP32_MIXED) as w:
        w.set_flush_kernel(dsu.FLUSH_MFMA)
        for e, row in zip(order, noise):
            b[e] = 0.9 * a[e] + 0.1 * row / np.sqrt(n)
            w.propose(int(e), b[e])
            w.accept()
        assert w.pending() == k
        got = w.inverse()
    # entries below 1, N-term FP32 sums (unit roundoff 2^-24), x 64 for the chain of moves
    assert np.abs(got - np.linalg.inv(b)).max() <= 64.0 * np.sqrt(n) * 2.0**-24


@pytest.mark.parametrize("n,k", [(64, 33), (65, 33), (128, 32), (128, 64), (100, 65), (128, 128), (129, 32)])
def test_fp64_flush_both_sides(n, k):
    require_gpu()
    a = well_conditioned(63 + n, n)
    noise = inputs.rows(64, k, n)
    order = np.random.default_rng(n).permutation(n)[:k]
    b = a.copy()
    with dsu.Walker(a, min(256, k + 1)) as w:
        w.set_flush_kernel(dsu.FLUSH_MFMA)
        for e, row in zip(order, noise):
            b[e] = 0.9 * a[e] + 0.1 * row / np.sqrt(n)
            w.propose(int(e), b[e])
            w.accept()
        assert w.pending() == k
        got = w.inverse()
    # as above with 2^-53, and 2^10 more for the moves' borderings
    assert np.abs(got - np.linalg.inv(b)).max() <= 2.0**10 * 64.0 * np.sqrt(n) * 2.0**-53


# the automatic choice at and beside its lines agrees with both kernels
@pytest.mark.parametrize("n,k,prec", [(1, 1, dsu.FP64), (960, 2, dsu.FP64), (961, 2, dsu.FP64), (512, 3, dsu.FP64),
                                      (513, 3, dsu.FP64), (384, 4, dsu.FP64), (385, 4, dsu.FP64), (40, 5, dsu.FP64),
                                      (70, 2, dsu.FP32_MIXED), (256, 3, dsu.FP32_MIXED), (257, 3, dsu.FP32_MIXED),
                                      (448, 3, dsu.FP32_MIXED), (449, 3, dsu.FP32_MIXED), (300, 4, dsu.FP32_MIXED)])
def test_automatic_flush_kernel(n, k, prec):
    require_gpu()
    a = well_conditioned(65 + n, n)
    noise = inputs.rows(66, k, n)
    b, got = a.copy(), []
    for e in range(k):
        b[e] = 0.9 * a[e] + 0.1 * noise[e] / np.sqrt(n)
    for mode in (dsu.FLUSH_AUTO, dsu.FLUSH_VALU, dsu.FLUSH_MFMA):
        with dsu.Walker(a, min(256, k + 1), precision=prec) as w:
            w.set_flush_kernel(mode)
            for e in range(k):
                w.propose(e, b[e])
                w.accept()
            w.flush()
            got.append(w.inverse())
    assert np.array_equal(got[0], got[1]) or np.array_equal(got[0], got[2])
    tol = 64.0 * np.sqrt(n) * (2.0**-24 if prec == dsu.FP32_MIXED else 2.0**-43)
    for x in got:
        assert np.abs(x - np.linalg.inv(b)).max() <= tol
