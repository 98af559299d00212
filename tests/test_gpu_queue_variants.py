"""Every variant of the persistent dense sweep (bandwidths per block, samples
per LDS tile) against the sliced sweep of 16 bandwidths, bit for bit.  A small
"launch_evals" makes the pass longer than one launch, so that the persistent
kernels run; it also cuts the items to one tile, and the columns end inside a
run of 64, at the end of one and between the tile sizes, so that units end
with partly filled tiles of 256, 512 and 1024 samples and items have pieces."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("launch_evals", [10**3, 10**9])
@pytest.mark.parametrize("n,n_h", [(300, 40), (704, 100), (1025, 33), (5003, 100), (20011, 100)])
def test_persistent_variants_equal_the_sliced_sweep(n, n_h, launch_evals):
    import paper_1505_01998_amd as kde

    if 0.5 * n * (n - 1) * n_h <= launch_evals:
        launch_evals = 10**6
    x = workloads.draw("gamma", n, 30 + n, np.float32)
    grid = np.geomspace(0.01, 3.0, n_h)
    with kde.Context(0) as c:
        c.set_option("launch_evals", launch_evals)
        c.set_option("persistent", 0)
        want = c.lscv_sums(x, grid)
        c.set_option("persistent", 1)
        for hc, tj in kde.TUNE_VARIANTS:
            c.set_option("lscv_hc", hc)
            c.set_option("lscv_tj", tj)
            got = c.lscv_sums(x, grid)
            assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1]), (hc, tj)
