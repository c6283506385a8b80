"""The blockings the recompute tuner times (no GPU)."""
import pytest

from paper_1708_00744_amd import tune


@pytest.mark.parametrize("n", [48, 64, 300, 960, 1024, 4096, 5000])
def test_candidates_differ_in_what_they_run(n):
    """Panel and chunk decide the kernels; the apply columns have no effect."""
    c = tune.recompute_candidates(n)
    assert len({(panel, chunk) for panel, chunk, _ in c}) == len(c) > 0
