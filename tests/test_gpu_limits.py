"""Limits of the workspace: what does not fit is refused, and what fitted
before the several-step forms had planes of their own still does."""
import numpy as np
import pytest

from paper_2105_13276_amd import binding as B
from paper_2105_13276_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,fits", [(4, 4, False), (20, 20, False), (63, 31, False),
                                        (63, 32, True), (64, 20, True)])
def test_weighted_sum_needs_its_staging_area(nx, ny, fits):
    """The 1025 partial sums go to the staging plane (64 floats a row up to 63
    cells, 128 up to 127): a grid whose plane is smaller is refused, and
    nothing beyond the plane (the live Hz of an earlier half level among it)
    is written."""
    cfg = W.make(nx, ny, 4, "uniform", 1)
    s = B.Sim(cfg, np.full((ny + 1, nx + 1), 1e18), None)
    s.step(11)
    before = s.save(np.zeros(s.state_bytes(), np.uint8))
    w = np.ones((ny + 1, nx + 1), np.float32)
    if fits:
        n = s.get("n", 0).astype(np.float64)
        assert abs(s.weighted_sum(w) - n.sum()) <= 1e-12 * n.sum()
    else:
        with pytest.raises(B.DmrError, match="ENOMEM"):
            s.weighted_sum(w)
    assert np.array_equal(s.save(np.zeros(s.state_bytes(), np.uint8)), before)
    s.close()
