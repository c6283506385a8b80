"""Kernel timing of a batch's sweep by phase."""
import numpy as np
import pytest

from gpu_util import require_gpu
from paper_1708_00744_amd import dsu, inputs

pytestmark = pytest.mark.gpu


# one window; several with a short last one; the widest window's own kernel
@pytest.mark.parametrize("prec", [dsu.FP64, dsu.FP32_MIXED])
@pytest.mark.parametrize("n,K", [(20, 32), (130, 16), (300, 64), (300, 140)])
def test_every_window_has_a_time_in_every_phase(prec, n, K):
    require_gpu()
    pos = np.stack([inputs.positions(3, w, n, 10.0) for w in range(2)])
    outs = []
    for level in (0, dsu.TIMING_FLUSH, dsu.TIMING_ALL):
        with dsu.Batch(n, pos, [3, 4], [0, 1], 0.2, K, precision=prec, box_l=10.0) as b:
            b.set_timing(level)
            b.sweep(2)
            windows = 2 * -(-n // K)
            want = {0: 0, dsu.TIMING_FLUSH: 0, dsu.TIMING_ALL: windows}[level]
            for phase in (dsu.PHASE_ROWS, dsu.PHASE_DECIDE):
                count, ms = b.kernel_time(phase)
                assert count == want and (ms > 0) == (want > 0)
            assert b.kernel_time(dsu.PHASE_FLUSH)[0] == (windows if level else 0)
            st = b.stats()
            outs.append((st["logdet"].tolist(), st["accepted"].tolist(), b.positions(1).tolist()))
    assert outs[0] == outs[1] == outs[2]


# one workgroup of states, a full one, one more; the counts of all determinants are
# set, and a trace starts over
@pytest.mark.parametrize("walkers", [1, 64, 65])
def test_set_sweep_and_trace_reach_every_determinant(walkers):
    require_gpu()
    n = 12
    pos = np.stack([inputs.positions(5, w, n, 10.0) for w in range(walkers)])
    with dsu.Batch(n, pos, [5] * walkers, list(range(walkers)), 0.2, 8, precision=dsu.FP64, box_l=10.0) as b:
        before = b.stats()
        b.set_sweep(41)
        after = b.stats()
        assert (after["sweeps"] == 41).all() and (before["sweeps"] == 0).all()
        assert all(np.array_equal(after[q], before[q]) for q in ("logdet", "sign", "accepted"))
        for _ in range(2):
            b.set_trace(1)
            b.sweep(1)
            taken = sum(int(b.trace(w)[1].sum()) for w in range(walkers))
            total = int(b.stats()["accepted"].sum())
            assert taken == total - int(after["accepted"].sum())
            after = b.stats()
        assert (after["sweeps"] == 43).all()
