"""The LSCV_H sweep of wide samples (padded to 8 and 16 dimensions), whose form
follows the width and the number of work items: around a run of 64, a row of
256 and a tile of 512, and on either side of the 2048 items where 16 dimensions
change form (tile-long items: n = 22,784 has 2025, 23,040 has 2070).  g within
1e-5 of its scale of the oracle, for the long columns of the FP64 form."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d", [(2, 5), (63, 8), (65, 6), (257, 12), (513, 16), (1281, 9), (1281, 7)])
def test_wide_samples_against_the_oracle(n, d):
    import paper_1505_01998_amd as kde

    x = workloads.draw_matrix(n, d, 60 + n, np.float32)
    if n <= d:  # a few samples span no d dimensions: more of them, the rest far away
        x = np.concatenate([x, 50.0 * np.eye(d, dtype=np.float32), -50.0 * np.eye(d, dtype=np.float32)])
    S = np.cov(x.astype(np.float64), rowvar=False)
    H = np.stack([0.3 * S, 0.05 * np.diag(np.diag(S)), 2.0 * S])
    with kde.Context(0) as c:
        g, gs = c.lscv_H_eval(x, H)
    for k in range(3):
        assert abs(g[k] - oracle.lscv_H(x, H[k])) <= 1e-5 * gs[k]


@pytest.mark.parametrize("n", [22784, 23040])
@pytest.mark.parametrize("d", [8, 9, 16])
def test_wide_samples_of_many_items_against_fp64(n, d):
    import paper_1505_01998_amd as kde

    x = workloads.draw_matrix(n, d, 5, np.float32)
    S = np.cov(x.astype(np.float64), rowvar=False)
    H = np.stack([0.3 * S, 0.05 * np.diag(np.diag(S))])
    with kde.Context(0) as c, kde.Context(0, "fp64") as f:
        g, gs = c.lscv_H_eval(x, H)
        want, _ = f.lscv_H_eval(x, H)
    assert np.all(np.abs(g - want) <= 1e-5 * gs)
