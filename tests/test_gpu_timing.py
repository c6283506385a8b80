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
