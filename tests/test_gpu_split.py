"""The cut of small passes: items of one tile cut into pieces of at least 64
samples, each with its own partial-sum slot, and units that end at the last
sample.  Checked where that can go wrong: columns around one run (64), one row
(256) and one tile (512), and grids whose chunk count changes the number of
pieces.  Bars as in test_gpu_parity.py: pair sums within 1e-5 (mixed, plus the
FP32 range limit) and 1e-10 (FP64 form) of the oracle; the items' sums, each
the sum of its pieces, add up to the pass's within 1e-12 (FP64 sums of at most
a few thousand positive terms)."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def kde():
    import paper_1505_01998_amd as kde

    return kde


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
@pytest.mark.parametrize("n,n_h", [(2, 1), (63, 5), (64, 16), (65, 17), (256, 100), (257, 1), (511, 33), (512, 128),
                                   (513, 128), (1000, 100), (1025, 500), (3001, 40), (5003, 128)])
def test_pieces_and_items_add_up(kde, precision, n, n_h):
    x = workloads.draw("bimodal", n, 500 + n, np.float32)
    grid = np.geomspace(0.02, 2.0, n_h) if n_h > 1 else np.array([0.3])
    o = oracle.lscv_curve(x, grid)
    tol = 1e-5 if precision == "mixed" else 1e-10
    atol = n * (n - 1) / 2 * 2.0**-126
    with kde.Context(0, precision) as c:
        s1, s2 = c.lscv_sums(x, grid)
        n_items, ranges, sums = c.lscv_item_sums(x, grid, np.arange(len(kde.kde_plan_items(n, n_h)[0])))
        p = c.bw_plugin(x, 3)[1].psi if n > 64 else None
    assert np.allclose(s1, o.s1, rtol=tol, atol=atol) and np.allclose(s2, o.s2, rtol=tol, atol=atol)
    assert n_items == len(ranges)
    assert np.allclose(sums[:, :, 0].sum(0), s1, rtol=1e-12, atol=0)
    assert np.allclose(sums[:, :, 1].sum(0), s2, rtol=1e-12, atol=0)
    for (i0, j0, j1), got in zip(ranges[:3], sums[:3]):
        o1, _ = oracle.lscv_block_sums(x, int(i0), min(int(i0) + 256, n), int(j0), min(int(j1), n), grid)
        assert np.allclose(got[:, 0], o1, rtol=tol, atol=atol)
    if p is not None:
        q = oracle.bw_plugin(x, 3)
        for s in range(3):
            assert p[s] == pytest.approx(q.psi[s], rel=1e-5 if precision == "mixed" else 1e-10 * max(1.0, q.kappa[s]))


def _older(ck, n, n_h):
    """The checkpoint as it was written with one psi slot an item: the header
    names the items, the block lacks the other slots, and the cursor of an
    interrupted stage counts items."""
    def al(b):
        return (b + 255) // 256 * 256

    head = ck[:128].copy()
    slots, _, block = head[64:88].view(np.int64)
    items = slots // 4
    gap = al(64 * items) - al(16 * items)
    # samples, x32, x64, moment partials, their range and counts, y32
    at = al(4 * n) + al(4 * (n + 768)) + al(8 * (n + 768)) + 8192 + 8192 + 4096 + al(4 * (n + 768))
    start = ck.size - block - 16 * n_h  # the header's size
    end = start + at + al(64 * items)
    out = np.concatenate([ck[:start + at], ck[start + at:start + at + al(16 * items)], ck[end:]])
    out[64:72].view(np.int64)[0] = items
    out[80:88].view(np.int64)[0] = block - gap
    cursor = out[112:120].view(np.int64)
    cursor[0] = min(cursor[0] // 4, items)
    return out


@pytest.mark.parametrize("older", [False, True])
@pytest.mark.parametrize("frac", [0.0, 0.02, 0.4, 1.0])
def test_checkpoint_of_the_cut_by_launch_size_resumes(kde, frac, older):
    """Up to about 3e4 samples the cut by launch size alone is whole rows,
    which "seg" = 0 asks for: a checkpoint written under it, also in the older
    form, resumes in a job of the automatic cut and ends bitwise as the
    whole-row batch; one written under the automatic cut resumes in another
    automatic job; another column's is refused."""
    A = kde.KDE_METHOD_ROT | kde.KDE_METHOD_PLUGIN | kde.KDE_METHOD_LSCV
    req = kde.Request(workloads.draw("gamma", 4099, 3, np.float32), A, 3, workloads.BATCH_GRID)
    with kde.Context(0) as rows, kde.Context(0) as auto:
        rows.set_option("seg", 0)
        for src in (rows,) if older else (rows, auto):
            want = src.batch([req])[0]
            with kde.Job(src, req) as job:
                _, total, _ = job.progress()
                if frac == 1.0:
                    job.run_to_end()
                elif frac > 0:
                    job.run(frac * total)
                ck = job.checkpoint()
            if older:
                ck = _older(ck, 4099, workloads.BATCH_GRID[3])
            with kde.Job(auto, req) as job2:
                job2.resume(ck)
                got = job2.run_to_end(total / 3)
            assert got.status == want.status == 0
            assert np.array_equal(got.g, want.g) and np.array_equal(got.gscale, want.gscale)
            assert got.plugin.psi == want.plugin.psi and got.k_lscv == want.k_lscv and got.h_plugin == want.h_plugin
        for bad_req, buf in ((kde.Request(req.x[:4000], A, 3, workloads.BATCH_GRID), ck), (req, ck[:-8])):
            with kde.Job(auto, bad_req) as other:
                with pytest.raises(kde.KdeError) as e:
                    other.resume(buf)
                assert e.value.status == kde.KDE_E_INVAL


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
@pytest.mark.parametrize("n,d", [(5, 2), (63, 3), (64, 2), (65, 4), (127, 2), (128, 1), (129, 3), (255, 2), (257, 4),
                                 (513, 2), (1281, 3), (700, 6)])
def test_d_dimensional_sweeps_at_the_edges(kde, precision, n, d):
    """LSCV_h and LSCV_H around a run, a wave's two samples a lane, a row and
    a tile: g within 1e-5 (mixed) and 1e-10 (FP64) of its scale."""
    x = workloads.draw_matrix(n, d, 40 + n, np.float32 if precision == "mixed" else np.float64)
    tol = 1e-5 if precision == "mixed" else 1e-10
    grid = np.geomspace(0.2, 2.0, 19)
    S = np.atleast_2d(np.cov(x.astype(np.float64), rowvar=False))
    with kde.Context(0, precision) as c:
        g, gs, _ = c.lscv_md_curve(x, grid)
        H = np.stack([0.3 * S, 0.05 * np.diag(np.diag(S))])
        gH, gsH = c.lscv_H_eval(x, H)
        one = [c.lscv_H_prepare(x).eval(h)[0][0] for h in H]
    o = oracle.lscv_md_curve(x, grid)
    assert np.all(np.abs(g - o.g) <= tol * o.gscale)
    for k in range(2):
        assert abs(gH[k] - oracle.lscv_H(x, H[k])) <= tol * gsH[k]
    assert np.array_equal(one, gH)


@pytest.mark.parametrize("hc", [8, 16, 32])
@pytest.mark.parametrize("n,n_h", [(300, 17), (2049, 9), (5003, 40), (12000, 100)])
def test_pruned_parts_of_a_chunk(kde, hc, n, n_h):
    """The pruned sweep leaves out parts of a bandwidth chunk run by run: every
    sum within 2^-34 of the dense one, and 1e-6 for the order of the samples
    (two clusters, so that runs of every part are left out); the count of
    evaluations is whole and no larger than with whole chunks."""
    rng = np.random.Generator(np.random.PCG64(n))
    x = np.concatenate([rng.normal(0, 1, n // 2), rng.normal(9, 0.3, n - n // 2)]).astype(np.float32)
    rng.shuffle(x)
    grid = np.geomspace(0.002, 1.5, n_h)
    req = kde.Request(x, kde.KDE_METHOD_LSCV, 2, grid)
    with kde.Context(0) as dense, kde.Context(0) as pr:
        pr.set_option("lscv_hc", hc)
        pr.set_option("prune", 1)
        sd, sp = dense.lscv_sums(x, grid), pr.lscv_sums(x, grid)
        a, b = dense.batch([req])[0], pr.batch([req])[0]
    for u, v in zip(sd, sp):
        assert np.all(np.abs(u - v) <= (1e-6 + 2.0**-34) * u + n * n * 2.0**-126)
    assert b.lscv_evals == int(b.lscv_evals) and 0 < b.lscv_evals < a.lscv_evals
    assert a.k_lscv == b.k_lscv
