"""Timed cases of the library: what a program that selects bandwidths with it
calls, from one small column to the largest sweep that ends within seconds.

A case is a dict: "kind" names the call, the other entries its sizes and
options.  Kinds and the use each stands for:

  column   every selector of one column in one call (rule of thumb, plug-in,
           LSCV over a grid): the library's main call, in the mixed form, the
           FP64 form, or with tile pruning
  plugin   the plug-in bandwidth alone, which a program that needs no grid asks for
  batch    the columns of a table, uneven in size, in one call
  served   the same requests arriving at a running server
  md       LSCV_h over a grid for d-dimensional samples
  H        one step of a search over bandwidth matrices: g(H) of a staged sample
  density  the estimate at query points
  ranges   COUNT / SUM / AVG of ranges of a column

Samples follow the families of workloads.py; device columns are what a program
has after loading a table to the GPU, host columns what it has before.
"""
import math

import numpy as np
import torch

import paper_1505_01998_amd as kde
import workloads

ALL = kde.KDE_METHOD_ROT | kde.KDE_METHOD_PLUGIN | kde.KDE_METHOD_LSCV


def listed():
    return [
        # the plain method on a small column held on the host: latency
        {"name": "column-1k", "kind": "column", "family": "normal", "n": 1000, "dtype": "f64", "where": "host",
         "grid": "log", "n_h": 100, "h_lo": 0.01, "h_hi": 1.0, "stages": 2, "precision": "mixed", "prune": False},
        # an ordinary column: FP32 mixture, 256 bandwidths, three stages
        {"name": "column-100k", "kind": "column", "family": "mixture", "n": 100_000, "dtype": "f32", "where": "device",
         "grid": "log", "n_h": 256, "h_lo": 0.005, "h_hi": 2.0, "stages": 3, "precision": "mixed", "prune": False},
        # the largest: a long-tailed column over the finest grid in use
        {"name": "column-200k", "kind": "column", "family": "lognormal", "n": 200_000, "dtype": "f32",
         "where": "device", "grid": "log", "n_h": 512, "h_lo": 0.00225, "h_hi": 0.58, "stages": 3,
         "precision": "mixed", "prune": False},
        # a ragged FP64 column in the FP64 form over the paper's default grid
        {"name": "column-fp64", "kind": "column", "family": "gamma", "n": 12_345, "dtype": "f64", "where": "host",
         "grid": "paper", "n_h": 150, "h_lo": 0.25, "h_hi": 4.0, "stages": 3, "precision": "fp64", "prune": False},
        # the pruned sweep of a large column over a wide grid
        {"name": "column-prune", "kind": "column", "family": "bimodal", "n": 150_001, "dtype": "f32",
         "where": "device", "grid": "log_rot", "n_h": 128, "h_lo": 1.0 / 64.0, "h_hi": 4.0, "stages": 3,
         "precision": "mixed", "prune": True},
        # the plug-in bandwidth of a large column
        {"name": "plugin-500k", "kind": "plugin", "family": "lognormal", "n": 500_000, "dtype": "f32",
         "where": "device", "stages": 3},
        # the columns of one table
        {"name": "batch-48", "kind": "batch", "count": 48, "n_lo": 1000, "n_hi": 30_000, "n_h": 128},
        # small requests reaching a running server together
        {"name": "served-24", "kind": "served", "count": 24, "n_lo": 2000, "n_hi": 20_000, "n_h": 128},
        # LSCV_h of three-dimensional samples
        {"name": "md-40k", "kind": "md", "d": 3, "n": 40_000, "n_h": 64, "dtype": "f32"},
        # one matrix of a search over 2 x 2 bandwidth matrices
        {"name": "H-100k", "kind": "H", "d": 2, "n": 100_000, "m": 1, "dtype": "f32"},
        # the estimate of a large column drawn on a screen's worth of points
        {"name": "density-1m", "kind": "density", "family": "lognormal", "n": 1_000_000, "points": 4096,
         "dtype": "f32"},
        # a dashboard's ranges over the same column
        {"name": "ranges-1m", "kind": "ranges", "family": "lognormal", "n": 1_000_000, "ranges": 256,
         "dtype": "f32"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["column", "column", "column", "plugin", "batch", "served", "md", "H", "density", "ranges"])
    dtype = rng.choice(["f32", "f32", "f64"])
    where = rng.choice(["host", "device"])
    family = rng.choice(list(workloads.FAMILIES))
    if kind == "column":
        grid = rng.choice(["log", "log_rot", "paper"])
        n_h = rng.choice([64, 100, 128, 150, 256, 512, rng.randrange(17, 400)])
        precision = rng.choice(["mixed", "mixed", "mixed", "fp64"])
        prune = precision == "mixed" and rng.random() < 0.25
        # no dearer than the largest listed column
        most = math.sqrt(2.0 * (1.5e12 if precision == "fp64" else 9e12) / n_h)
        lo, hi = {"log": (0.005, 2.0), "log_rot": (1.0 / 64.0, 4.0), "paper": (0.25, 4.0)}[grid]
        return {"kind": kind, "family": family, "n": _log(rng, 600, min(250_000, most)), "dtype": dtype,
                "where": where, "grid": grid, "n_h": n_h, "h_lo": lo, "h_hi": hi, "stages": rng.choice([2, 3, 3]),
                "precision": precision, "prune": prune}
    if kind == "plugin":
        return {"kind": kind, "family": family, "n": _log(rng, 1000, 600_000), "dtype": dtype, "where": where,
                "stages": rng.choice([2, 3])}
    if kind in ("batch", "served"):
        n_lo = _log(rng, 1000, 4000)
        return {"kind": kind, "count": rng.randrange(6, 64), "n_lo": n_lo, "n_hi": _log(rng, 2 * n_lo, 50_000),
                "n_h": rng.choice([64, 128, 150])}
    if kind == "md":
        return {"kind": kind, "d": rng.choice([2, 3, 4, 5, 8]), "n": _log(rng, 1500, 60_000),
                "n_h": rng.choice([32, 64, 150]), "dtype": dtype}
    if kind == "H":
        return {"kind": kind, "d": rng.choice([2, 2, 3, 4, 6]), "n": _log(rng, 2000, 150_000),
                "m": rng.choice([1, 1, 3, 8]), "dtype": dtype}
    if kind == "density":
        return {"kind": kind, "family": family, "n": _log(rng, 5000, 2_000_000), "points": _log(rng, 64, 8192),
                "dtype": dtype}
    return {"kind": kind, "family": family, "n": _log(rng, 5000, 2_000_000), "ranges": _log(rng, 8, 1024),
            "dtype": dtype}


# ---- inputs
_NP = {"f32": np.float32, "f64": np.float64}
_CTX = {}


def _context(precision="mixed", prune=False, server=False):
    """The program's context: opened once, used for every column it has."""
    key = (precision, prune, server)
    if key not in _CTX:
        c = kde.Context(0, precision)
        if prune:
            c.set_option("prune", 1)
        if server:
            c.server_start(4 << 30, 64)
        _CTX[key] = c
    return _CTX[key]


def _column(case, seed, salt=0):
    return workloads.draw(case["family"], case["n"], 7919 * seed + salt, _NP[case.get("dtype", "f32")])


def _held(x, where):
    """The column as the program holds it: a host array or a device tensor."""
    return x if where == "host" else torch.from_numpy(x).to("cuda:0")


def _grid(case):
    if case["grid"] == "log":
        return np.geomspace(case["h_lo"], case["h_hi"], case["n_h"])
    if case["grid"] == "paper":
        return ("paper", case["n_h"])
    return ("log_rot", case["h_lo"], case["h_hi"], case["n_h"])


def _columns(case, seed):
    """Sizes spread log-uniformly over the case's range (the same for every
    seed, so a case is one amount of work), samples from the seed."""
    k = case["count"]
    out = []
    for j in range(k):
        n = int(round(case["n_lo"] * (case["n_hi"] / case["n_lo"]) ** ((j * 7 % k + 0.5) / k)))
        fam = workloads.BATCH_FAMILIES[(j * 5 + j // 4) % 4]
        out.append(workloads.draw(fam, n, 104729 * seed + j, np.float32))
    return out


def _scale(case):
    """Normal-reference scale s of a bandwidth matrix s^2 Sigma (or of h0 at d = 1)."""
    d = case.get("d", 1)
    return (4.0 / ((d + 2.0) * case["n"])) ** (1.0 / (d + 4.0))


def _matrices(case, seed, x):
    rng = np.random.default_rng(seed)
    d = case["d"]
    S = np.cov(x.astype(np.float64), rowvar=False)
    out = []
    for _ in range(case["m"]):
        B = np.eye(d) + 0.15 * rng.standard_normal((d, d))
        out.append(math.exp(0.4 * rng.standard_normal()) * _scale(case) ** 2 * (B @ S @ B.T))
    return np.stack(out)


def _points(case, seed, x):
    """Half on a regular axis over the column's range, half at samples."""
    rng = np.random.default_rng(seed + 5)
    m = case["points"]
    a = np.linspace(float(x.min()), float(np.quantile(x, 0.999)), m - m // 2)
    return np.concatenate([a, rng.choice(x, m // 2).astype(np.float64)])


def _ranges(case, seed, x):
    rng = np.random.default_rng(seed + 6)
    ends = np.sort(rng.choice(x, (case["ranges"], 2)).astype(np.float64), axis=1)
    lo, hi = ends[:, 0].copy(), ends[:, 1].copy()
    lo[0], hi[-1] = -np.inf, np.inf
    return lo, hi


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("column", "plugin"):
        x = _column(case, seed)
        s = {"case": case, "x": _held(x, case["where"]),
             "ctx": _context(case.get("precision", "mixed"), case.get("prune", False))}
        if kind == "column":
            s["request"] = kde.Request(s["x"], ALL, case["stages"], _grid(case))
        return s
    if kind in ("batch", "served"):
        cols = _columns(case, seed)
        grid = ("log_rot", 1.0 / 64.0, 4.0, case["n_h"])
        return {"case": case, "ctx": _context(server=kind == "served"),
                "requests": [kde.Request(x, ALL, workloads.BATCH_STAGES, grid) for x in cols]}
    if kind in ("md", "H"):
        x = workloads.draw_matrix(case["n"], case["d"], 3571 * seed + 1, _NP[case["dtype"]])
        xd = torch.from_numpy(x).to("cuda:0")
        torch.cuda.synchronize()
        ctx = _context()
        if kind == "md":
            s0 = _scale(case)
            return {"case": case, "ctx": ctx, "x": xd, "grid": np.geomspace(0.1 * s0, 3.0 * s0, case["n_h"])}
        return {"case": case, "ctx": ctx, "x": xd, "prep": ctx.lscv_H_prepare(xd), "H": _matrices(case, seed, x)}
    x = _column(case, seed)
    h = 0.3 * _scale(case) * float(x.std(dtype=np.float64))
    s = {"case": case, "ctx": _context(), "x": _held(x, "device"), "h": h}
    if kind == "density":
        s["points"] = _points(case, seed, x)
    else:
        s["lo"], s["hi"] = _ranges(case, seed, x)
    return s


# ---- one pass
def _result(r):
    p = r.plugin
    return {"sigma": r.sigma, "h_rot": r.h_rot, "h_plugin": r.h_plugin, "h_lscv": r.h_lscv, "k": int(r.k_lscv),
            "pilot": np.array(p.g), "psi": np.array(p.psi), "g": r.g, "gscale": r.gscale}


def _together(results):
    return {"sigma": np.array([r.sigma for r in results]), "h_rot": np.array([r.h_rot for r in results]),
            "h_plugin": np.array([r.h_plugin for r in results]), "h_lscv": np.array([r.h_lscv for r in results]),
            "k": np.array([r.k_lscv for r in results], np.int64), "psi": np.array([r.plugin.psi for r in results]),
            "g": np.stack([r.g for r in results]), "gscale": np.stack([r.gscale for r in results])}


def run(state):
    kind, c = state["case"]["kind"], state["ctx"]
    if kind == "column":
        return _result(c.batch([state["request"]])[0])
    if kind == "plugin":
        h, info = c.bw_plugin(state["x"], state["case"]["stages"])
        return {"h": h, "sigma": info.sigma, "pilot": np.array(info.g), "psi": np.array(info.psi)}
    if kind == "batch":
        return _together(c.batch(state["requests"]))
    if kind == "served":
        tickets = [c.submit(r) for r in state["requests"]]
        return _together([c.wait(t) for t in tickets])
    if kind == "md":
        g, gs, _ = c.lscv_md_curve(state["x"], state["grid"])
        return {"g": g, "gscale": gs}
    if kind == "H":
        g, gs = state["prep"].eval(state["H"])
        return {"g": g, "gscale": gs}
    if kind == "density":
        return {"f": c.density(state["x"], state["h"], state["points"])}
    count, total, avg = c.range_aggregates(state["x"], state["h"], state["lo"], state["hi"])
    return {"count": count, "sum": total, "avg": avg}


# ---- what a pass cannot do without
def _column_work(n, n_h, stages, esz):
    """Every sample read once, every result written once; per pair the
    difference and its square, per (pair, h) the product, the exponential, its
    square and two sums, per (pair, stage) the two products, the exponential,
    the polynomial and two sums."""
    pairs = 0.5 * n * (n - 1.0)
    flops = pairs * (2.0 + 5.0 * n_h) if n_h else 0.0
    for r in ((8, 6, 4) if stages == 3 else (6, 4)):
        flops += pairs * (7.0 + r)
    return {"bytes": float(esz * n + 16 * n_h + 128), "flops": flops}


def work(case):
    kind = case["kind"]
    esz = 8 if case.get("dtype") == "f64" else 4
    if kind in ("column", "plugin"):
        return _column_work(case["n"], case.get("n_h", 0), case["stages"], esz)
    if kind in ("batch", "served"):
        parts = [_column_work(x.size, case["n_h"], workloads.BATCH_STAGES, 4) for x in _columns(case, 0)]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    n = case["n"]
    if kind in ("md", "H"):
        d, m = case["d"], case["n_h"] if kind == "md" else case["m"]
        pairs = 0.5 * n * (n - 1.0)
        per = 3.0 * d + 5.0 * m if kind == "md" else m * (3.0 * d + 4.0)
        return {"bytes": float(esz * n * d + 16 * m), "flops": pairs * per}
    if kind == "density":
        return {"bytes": float(esz * n + 16 * case["points"]), "flops": 5.0 * n * case["points"]}
    # per end of a range and sample: the standardised distance, the normal
    # integral and density, and the sums they enter
    return {"bytes": float(esz * n + 40 * case["ranges"]), "flops": 12.0 * n * case["ranges"]}


# ---- the same in 64 bits, without the library
_PHI0 = 1.0 / math.sqrt(2.0 * math.pi)
_TERMS = 2.0e11  # pair terms that the definitions below evaluate within seconds


def _blocks(n):
    b = max(1, min(n, int(4e7 // n) or 1))
    return [(i, min(n, i + b)) for i in range(0, n, b)]


def _pairs(x, i0, i1):
    """Squared differences of rows i0..i1 against every later sample (0 where j <= i is set to inf)."""
    t = (x[i0:i1, None] - x[None, i0:]).square_()
    m = torch.ones(i1 - i0, i1 - i0, dtype=torch.bool, device=x.device).tril_()
    t[:, : i1 - i0].masked_fill_(m, math.inf)
    return t


def _lscv(x, grid):
    n = x.numel()
    s = np.zeros((len(grid), 2))
    for i0, i1 in _blocks(n):
        t = _pairs(x, i0, i1)
        for k, h in enumerate(grid):
            e = torch.exp(t * (-0.25 / (h * h)))
            s[k, 0] += float(e.sum())
            s[k, 1] += float(e.square_().sum())
    a, b = s[:, 0] / math.sqrt(4.0 * math.pi), s[:, 1] * _PHI0
    diag = 1.0 / (n * math.sqrt(4.0 * math.pi))
    return (2.0 / n**2 * (a - 2.0 * b) + diag) / grid, (2.0 / n**2 * (a + 2.0 * b) + diag) / grid


def _herm(r, w):
    if r == 4:
        return (w - 6.0) * w + 3.0
    if r == 6:
        return ((w - 15.0) * w + 45.0) * w - 15.0
    return (((w - 28.0) * w + 210.0) * w - 420.0) * w + 105.0


def _plugin(x, sigma, stages):
    n = x.numel()
    zero = {4: 3.0, 6: -15.0, 8: 105.0, 10: -945.0}

    def normal_scale(r):
        return zero[r] / (2.0 ** (r // 2 + 1) * math.sqrt(math.pi) * sigma ** (r + 1))

    psi, pilot = [math.nan] * 3, [math.nan] * 3
    above = normal_scale(10)
    if stages == 2:
        psi[0] = above = normal_scale(8)
    for s in range(0 if stages == 3 else 1, 3):
        r = 8 - 2 * s
        g = (-2.0 * zero[r] * _PHI0 / (above * n)) ** (1.0 / (r + 3))
        total = 0.0
        for i0, i1 in _blocks(n):
            w = _pairs(x, i0, i1).mul_(1.0 / (g * g)).clamp_(max=2000.0)
            total += float((_herm(r, w) * torch.exp(-0.5 * w)).sum())
        above = (2.0 * total + n * zero[r]) * _PHI0 / (n * n * g ** (r + 1))
        psi[s], pilot[s] = above, g
    return (0.5 / math.sqrt(math.pi) / (psi[2] * n)) ** 0.2, np.array(pilot), np.array(psi)


def _exact_column(x, case):
    n = x.size
    xd = torch.from_numpy(x.astype(np.float64)).to("cuda:0")
    sigma = float(x.astype(np.float64).std(ddof=1))
    h_rot = (4.0 / 3.0) ** 0.2 * n ** -0.2 * sigma
    out = {"sigma": sigma, "h_rot": h_rot}
    out["h_plugin"], out["pilot"], out["psi"] = _plugin(xd, sigma, case["stages"])
    if case["grid"] == "log":
        grid = np.geomspace(case["h_lo"], case["h_hi"], case["n_h"])
    elif case["grid"] == "paper":
        grid = h_rot * np.linspace(0.25, 4.0, case["n_h"])
    else:
        grid = h_rot * np.geomspace(case["h_lo"], case["h_hi"], case["n_h"])
    out["g"], out["gscale"] = _lscv(xd, grid)
    out["h_lscv"] = float(grid[int(np.argmin(out["g"]))])
    out["k"] = None
    return out


def _quadratic_sums(y, coefs):
    """Per coefficient c: the sums over pairs of exp(-c S) and its square, S the squared distance of rows of y."""
    n = y.shape[0]
    s = np.zeros((len(coefs), 2))
    for i0, i1 in _blocks(n):
        t = _pairs(y[:, 0].contiguous(), i0, i1)
        for a in range(1, y.shape[1]):
            t += (y[i0:i1, a, None] - y[None, i0:, a]).square_()
        for k, c in enumerate(coefs):
            e = torch.exp(t * -c)
            s[k, 0] += float(e.sum())
            s[k, 1] += float(e.square_().sum())
    return s


def _sphered(x, S):
    z = torch.from_numpy(x.astype(np.float64) - x.astype(np.float64).mean(0)).to("cuda:0")
    L = torch.from_numpy(np.linalg.cholesky(S)).to("cuda:0")
    return torch.linalg.solve_triangular(L, z.T, upper=False).T.contiguous()


def _objective(s, n, d, logdet, hd):
    sq = math.exp(-0.5 * logdet)
    A, B = (4.0 * math.pi) ** (-0.5 * d) * sq, (2.0 * math.pi) ** (-0.5 * d) * sq
    lo, hi = A * s[:, 0], 2.0 * B * s[:, 1]
    return hd * (2.0 / n**2 * (lo - hi) + A / n), hd * (2.0 / n**2 * (lo + hi) + A / n)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("column", "plugin"):
        n = case["n"]
        if 0.5 * n * n * (case.get("n_h", 0) + 6 * case["stages"]) > _TERMS:
            return None
        x = _column(case, seed)
        if kind == "column":
            return _exact_column(x, case)
        sigma = float(x.astype(np.float64).std(ddof=1))
        h, pilot, psi = _plugin(torch.from_numpy(x.astype(np.float64)).to("cuda:0"), sigma, case["stages"])
        return {"h": h, "sigma": sigma, "pilot": pilot, "psi": psi}
    if kind in ("batch", "served"):
        cols = _columns(case, seed)
        if sum(0.5 * x.size**2 for x in cols) * case["n_h"] > _TERMS:
            return None
        one = {"grid": "log_rot", "h_lo": 1.0 / 64.0, "h_hi": 4.0, "n_h": case["n_h"],
               "stages": workloads.BATCH_STAGES}
        parts = [_exact_column(x, one) for x in cols]
        out = {k: np.stack([np.asarray(p[k]) for p in parts]) for k in parts[0] if k not in ("k", "pilot")}
        return dict(out, k=None)
    n = case["n"]
    if kind in ("md", "H"):
        m = case["n_h"] if kind == "md" else case["m"]
        if 0.5 * n * n * (m + case["d"]) > _TERMS:
            return None
        x = workloads.draw_matrix(n, case["d"], 3571 * seed + 1, _NP[case["dtype"]])
        if kind == "md":
            s0 = _scale(case)
            grid = np.geomspace(0.1 * s0, 3.0 * s0, m)
            S = np.cov(x.astype(np.float64), rowvar=False)
            s = _quadratic_sums(_sphered(x, S), 0.25 / grid**2)
            g, gs = _objective(s, n, case["d"], np.linalg.slogdet(S)[1], grid ** -float(case["d"]))
            return {"g": g, "gscale": gs}
        g, gs = [], []
        for H in _matrices(case, seed, x):
            s = _quadratic_sums(_sphered(x, H), [0.25])
            a, b = _objective(s, n, case["d"], np.linalg.slogdet(H)[1], 1.0)
            g.append(a[0])
            gs.append(b[0])
        return {"g": np.array(g), "gscale": np.array(gs)}
    x = _column(case, seed)
    h = 0.3 * _scale(case) * float(x.std(dtype=np.float64))
    xd = torch.from_numpy(x.astype(np.float64)).to("cuda:0")
    if kind == "density":
        p = torch.from_numpy(_points(case, seed, x)).to("cuda:0")
        f = torch.empty_like(p)
        for k in range(0, p.numel(), 32):
            z = (p[k:k + 32, None] - xd[None, :]).div_(h)
            f[k:k + 32] = torch.exp(z.square_().mul_(-0.5)).sum(1)
        return {"f": f * (_PHI0 / (n * h))}
    lo, hi = _ranges(case, seed, x)
    cnt, tot = np.zeros(len(lo)), np.zeros(len(lo))

    def tail(z):
        return 0.5 * torch.special.erfc(z * math.sqrt(0.5))

    for k in range(len(lo)):
        a, b = (float(lo[k]) - xd) / h, (float(hi[k]) - xd) / h
        p = torch.where(a >= 0, tail(a) - tail(b), torch.where(b <= 0, tail(-b) - tail(-a), 1.0 - tail(-a) - tail(b)))
        d = _PHI0 * (torch.exp(-0.5 * a * a) - torch.exp(-0.5 * b * b))
        cnt[k], tot[k] = float(p.sum()), float((xd * p + h * d).sum())
    return {"count": cnt, "sum": tot, "avg": tot / cnt}
