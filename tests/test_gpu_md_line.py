"""The d-dimensional sweep on either side of the number of units where its units
change from 64 samples to 256 (whole rows of n = 5000: 20 items): 1792 up to
four dimensions, 5120 up to eight, 8192 above.  A lane's compensated folds are
the same in both, and only the FP64 sums over lanes and units are grouped anew
(320 terms of one sign at most, 320 x 2^-53 = 3.6e-14 of each sum), so g at the
bandwidths that both grids hold agrees within 1e-13 of its scale; a few points
are held to the oracle."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,hc,chunks", [(1, 16, 89), (3, 16, 89), (4, 16, 89), (5, 8, 255), (8, 8, 255), (12, 8, 409)])
def test_units_of_64_and_256_samples_agree(d, hc, chunks):
    import paper_1505_01998_amd as kde

    x = workloads.draw_matrix(5000, d, 80 + d, np.float32)
    grid = np.geomspace(0.2, 2.0, hc * (chunks + 2))
    with kde.Context(0) as c:
        g0, gs, _ = c.lscv_md_curve(x, grid[:hc * chunks])
        g1, _, _ = c.lscv_md_curve(x, grid)
    m = hc * chunks
    assert np.all(np.abs(g0 - g1[:m]) <= 1e-13 * gs)
    at = [0, m // 2, m - 1]
    o = oracle.lscv_md_curve(x, grid[at])
    assert np.all(np.abs(g0[at] - o.g) <= 1e-5 * o.gscale)
