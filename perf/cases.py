"""The work that programs have this library do, as timed cases.

A case is a dict of plain values; its "kind" names the call:

  step     factorize + solve in one call, for a point set whose plan is kept
           (new lengthscales or new right-hand sides on the same points)
  solve    one solve with a kept factor
  super    the same step on a supernodal plan
  batch    many independent small problems, one replay of their captured graph
  dense    one product with the dense covariance matrix
  pcg      conjugate gradients on the dense system with the factor as preconditioner
  request  everything for points seen once: analysis, factor, solve, solution on the host

Point sets: "uniform2d" and "uniform3d" (iid in the unit square and cube),
"grid2d" (jittered grid over the unit square, n a square number) and "sphere20"
(two intrinsic dimensions embedded in R^20, what a serving request carries).
"""
import math

import numpy as np
import torch

import paper_1706_02205_amd as kchol

TAU = 1e-6  # pivot floor of the mixed-precision factor
EXACT_MOST = 12_500  # points up to which exact() forms the dense factor in 64 bits


def listed():
    return [
        # one small problem: launches and the latency of each level count
        _step("step_2k_fp64", "uniform2d", 2000, 1.5, 0.2, 3.0, 1, "fp64", False),
        # three dimensions, the scaling workload of the method, an odd size
        _step("step_20k_3d_fp64", "uniform3d", 20_011, 0.5, 0.2, 3.0, 1, "fp64", False),
        # one factor for 50,000 points of a serving request in R^20, used once, so without match masks
        _step("step_50k_sphere_mixed", "sphere20", 50_003, 1.5, 0.2, 3.0, 4, "mixed", False),
        # the jittered-grid benchmark recipe, mixed precision, refactored with kept match masks
        _step("step_90k_grid_mixed_masks", "grid2d", 301 * 301, 0.5, 0.1, 4.0, 8, "mixed", True),
        # the same recipe in FP64 at the largest size here
        _step("step_360k_grid_fp64_masks", "grid2d", 600 * 600, 0.5, 0.1, 4.0, 8, "fp64", True),
        # supernodal aggregation in 3-D, whose mixed factor runs on the matrix cores
        dict(_step("super_10k_3d_mixed", "uniform3d", 10_007, 0.5, 0.2, 3.0, 1, "mixed", False), kind="super"),
        # a new right-hand side for a kept factor
        dict(_step("solve_160k_grid_fp64", "grid2d", 400 * 400, 0.5, 0.1, 4.0, 1, "fp64", False), kind="solve"),
        # the dense system to a 1e-10 residual, four right-hand sides
        dict(_step("pcg_9k_fp64", "uniform2d", 9001, 0.5, 0.2, 3.0, 4, "fp64", False), kind="pcg"),
        # a batch of independent problems of uneven size, each with its own lengthscale
        {"name": "batch_48_mixed", "kind": "batch", "instances": 48, "n_lo": 500, "n_hi": 5000, "nu": 1.5, "rho": 3.0,
         "prec": "mixed"},
        # the dense product: one small system and one that fills the device
        {"name": "dense_3k", "kind": "dense", "points": "uniform2d", "n": 3001, "nu": 1.5, "ell": 0.2, "nrhs": 1},
        {"name": "dense_100k", "kind": "dense", "points": "uniform3d", "n": 100_000, "nu": 0.5, "ell": 0.2, "nrhs": 8},
        # points seen once, from the host arrays to the solution on the host
        {"name": "request_8k_sphere", "kind": "request", "points": "sphere20", "n": 8009, "nu": 1.5, "ell": 0.2,
         "rho": 3.0, "nrhs": 4, "prec": "mixed"},
    ]


def _step(name, points, n, nu, ell, rho, nrhs, prec, masks):
    c = {"kind": "step", "points": points, "n": n, "nu": nu, "ell": ell, "rho": rho, "nrhs": nrhs, "prec": prec,
         "masks": masks}
    return dict(c, name=name) if name else c


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["step", "step", "step", "solve", "solve", "super", "batch", "dense", "dense", "pcg", "request"])
    nu = rng.choice([0.5, 1.5, 2.5])
    if kind == "batch":
        return {"kind": kind, "instances": log_int(2, 64), "n_lo": log_int(300, 800), "n_hi": log_int(1000, 6000),
                "nu": nu, "rho": rng.choice([2.0, 3.0]), "prec": rng.choice(["fp64", "mixed"])}
    if kind == "dense":
        return {"kind": kind, "points": rng.choice(["uniform2d", "uniform3d", "sphere20"]), "n": log_int(500, 70_000),
                "nu": nu, "ell": rng.uniform(0.05, 0.3), "nrhs": rng.randint(1, 11)}
    if kind == "pcg":
        return {"kind": kind, "points": "uniform2d", "n": log_int(800, 9000), "nu": 0.5, "ell": rng.uniform(0.1, 0.3),
                "rho": rng.choice([3.0, 4.0]), "nrhs": rng.randint(1, 8), "prec": rng.choice(["fp64", "mixed"])}
    if kind == "request":
        return {"kind": kind, "points": "sphere20", "n": log_int(1000, 12_000), "nu": 1.5, "ell": 0.2, "rho": 3.0,
                "nrhs": rng.randint(1, 4), "prec": "mixed"}
    if kind == "super":
        return dict(_step(None, "uniform3d", log_int(1000, 10_007), 0.5, rng.uniform(0.1, 0.3), rng.choice([2.0, 3.0]),
                          rng.randint(1, 8), "mixed", False), kind=kind)
    points, most = rng.choice([("uniform2d", 150_000), ("grid2d", 200_000), ("uniform3d", 20_000), ("sphere20", 50_000)])
    # rough kernels in more than two dimensions: the range in which the factor keeps nearly all its pivots
    nu = 0.5 if points == "uniform3d" else min(nu, 1.5) if points != "sphere20" else 1.5
    rho = 3.0 if points in ("uniform3d", "sphere20") else rng.choice([3.0, 4.0])
    prec = rng.choice(["fp64", "mixed"])
    n = log_int(700, most)
    return dict(_step(None, points, math.isqrt(n) ** 2 if points == "grid2d" else n, nu, rng.uniform(0.05, 0.25), rho,
                      rng.randint(1, 11), prec, kind == "step" and rng.random() < 0.4), kind=kind)


# ---------------------------------------------------------------- inputs

def _points(kind, n, g):
    if kind == "uniform2d":
        return g.random((n, 2))
    if kind == "uniform3d":
        return g.random((n, 3))
    if kind == "grid2d":
        m = math.isqrt(n)
        h = 1.0 / m
        i, j = np.meshgrid(np.arange(m), np.arange(m), indexing="ij")
        base = np.stack([(i.ravel() + 0.5) * h, (j.ravel() + 0.5) * h], axis=1)
        return np.ascontiguousarray(base + g.uniform(-0.4 * h, 0.4 * h, size=base.shape))
    w = g.normal(0.0, 3.0, size=(10, 2))
    ph = g.random((n, 2)) @ w.T
    x = np.empty((n, 20))
    x[:, 0::2] = np.sin(ph)
    x[:, 1::2] = np.cos(ph)
    return x / math.sqrt(10)


def _host_inputs(case, seed):
    g = np.random.Generator(np.random.PCG64(seed))
    if case["kind"] == "batch":
        # the sizes belong to the case, the points and lengthscales to the seed
        sizes = np.random.Generator(np.random.PCG64(case["n_hi"])).uniform(
            math.log(case["n_lo"]), math.log(case["n_hi"]), size=case["instances"])
        sizes = [int(v) for v in np.exp(sizes)]
        pts = [g.random((n, 2)) for n in sizes]
        return pts, g.uniform(0.05, 0.3, size=len(sizes)), g.standard_normal((sum(sizes), 1))
    pts = _points(case["points"], case["n"], g)
    return pts, case.get("ell"), g.standard_normal((len(pts), case["nrhs"]))


def _pivot(case):
    return ("zero", 0.0) if case["prec"] == "fp64" else ("shift", TAU)


def prepare(case, seed):
    pts, ell, b = _host_inputs(case, seed)
    s = {"case": case, "nu": case["nu"], "ell": ell}
    if case["kind"] == "request":
        s.update(pts=pts, b=b)
        return s
    s["b"] = torch.from_numpy(b).cuda()
    s["x"] = torch.from_numpy(np.concatenate(pts) if case["kind"] == "batch" else pts).cuda()
    if case["kind"] == "dense":
        return s
    pivot, tau = _pivot(case)
    if case["kind"] == "batch":
        f = kchol.Factor(kchol.analyze_batched(pts, case["rho"]), case["prec"])
        s["ells"] = torch.from_numpy(ell).cuda()
        s["graph"] = f.capture(s["x"], s["b"], case["nu"], ell_dev=s["ells"], pivot=pivot, tau=tau)
    elif case["kind"] == "super":
        f = kchol.Factor(kchol.analyze_supernodal(pts, case["rho"]), case["prec"])
    else:
        f = kchol.Factor(kchol.analyze(pts, case["rho"]), case["prec"])
        if case.get("masks"):
            f.build_matches()
        if case["kind"] in ("solve", "pcg"):
            f.factorize(s["x"], case["nu"], ell, pivot, tau)
    s["factor"] = f
    return s


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "dense":
        return kchol.dense_matvec(state["x"], state["b"], state["nu"], state["ell"])
    if kind == "batch":
        return state["graph"].launch()
    if kind == "solve":
        return state["factor"].solve(state["b"])
    if kind == "pcg":
        return state["factor"].pcg(state["x"], state["b"], state["nu"], state["ell"], tol=1e-10)[0]
    pivot, tau = _pivot(case)
    if kind == "request":
        f = kchol.Factor(kchol.analyze(state["pts"], case["rho"], nthreads=1), case["prec"])
        x = torch.from_numpy(state["pts"]).cuda()
        f.factorize(x, state["nu"], state["ell"], pivot, tau)
        return f.solve(torch.from_numpy(state["b"]).cuda()).cpu().numpy()
    return state["factor"].factorize_solve(state["x"], state["b"], state["nu"], state["ell"], pivot, tau)


# ---------------------------------------------------------------- work

def _pattern_work(pts, rho, supernodal=False):
    """(entries of S, Schur updates) of one problem.  An entry's updates are the parents that its row and its
    column's row share: nine tenths of the row's entries before it, on all point sets here."""
    plan = kchol.analyze_supernodal(pts, rho) if supernodal else kchol.analyze(pts, rho)
    rows = np.bincount(plan.export()[3], minlength=len(pts)).astype(np.float64)
    return float(rows.sum()), 0.45 * float((rows * (rows - 1)).sum())


def work(case):
    """Points, pattern (4-byte indices) and right-hand sides read once, L and the solution written once; two flops a
    Schur update, four an entry and right-hand side in the sweeps, about 20 a covariance entry."""
    if case["kind"] == "dense":
        n, r = case["n"], case["nrhs"]
        d = {"uniform3d": 3, "sphere20": 20}.get(case["points"], 2)
        return {"bytes": 8.0 * n * (d + 2 * r), "flops": float(n) * n * (3 * d + 20 + 2 * r)}
    pts, _, b = _host_inputs(case, 1)
    vt = 8 if case["prec"] == "fp64" else 4
    nnz = upd = size = 0.0
    for p in pts if case["kind"] == "batch" else [pts]:
        e, u = _pattern_work(p, case["rho"], case["kind"] == "super")
        nnz, upd, size = nnz + e, upd + u, size + p.size
    sweeps = 4.0 * nnz * b.shape[1]
    if case["kind"] == "solve":
        return {"bytes": (4 + vt) * nnz + 16.0 * b.size, "flops": sweeps}
    w = {"bytes": (4 + vt) * nnz + 16.0 * b.size + 8.0 * size, "flops": 2 * upd + sweeps + 20 * nnz}
    if case["kind"] == "pcg":  # at least one product and one preconditioner solve
        n = float(len(b))
        return {"bytes": (4 + vt) * nnz + 32.0 * b.size, "flops": sweeps + n * n * (26 + 2 * b.shape[1])}
    return w


# ---------------------------------------------------------------- exact values

def _kernel(r, nu, ell):
    if nu == 0.5:
        return torch.exp(-r / ell)
    if nu == 1.5:
        a = math.sqrt(3.0) * r / ell
        return (1 + a) * torch.exp(-a)
    a = math.sqrt(5.0) * r / ell
    return (1 + a + a * a / 3) * torch.exp(-a)


def _distances(x, y):
    s = torch.zeros(len(x), len(y), dtype=torch.float64, device=x.device)
    for t in range(x.shape[1]):
        s += (x[:, t, None] - y[None, :, t]) ** 2
    return s.sqrt_()


def _maximin(x):
    """The maximin ordering from point 0 (ties to the lowest index) and its lengths."""
    n = len(x)
    xt = np.ascontiguousarray(x.T)
    near = np.full(n, np.inf)
    perm, length = np.empty(n, np.int64), np.empty(n)
    c = 0
    for k in range(n):
        perm[k], length[k] = c, near[c]
        s = np.zeros(n)
        for row in xt:
            df = row - row[c]
            s += df * df
        np.minimum(near, np.sqrt(s), out=near)
        near[c] = -1.0
        c = int(near.argmax())
    return perm, length


def _exact_solution(x, b, nu, ell, rho, pivot, tau, device):
    """x = P^T L^-T L^-1 P b with the incomplete Cholesky factor L on the pattern dist <= rho * max(l_i, l_j),
    kept as a dense lower triangle (zero outside the pattern)."""
    n = len(x)
    perm, length = _maximin(x)
    xh = torch.from_numpy(x[perm]).to(device)
    dist = _distances(xh, xh)
    inside = dist <= rho * torch.from_numpy(length).to(device)[None, :]  # column j: l_j is the larger length
    inside = torch.tril(inside)
    L = torch.where(inside, _kernel(dist, nu, ell), torch.zeros((), dtype=torch.float64, device=device))
    del dist
    cols = inside.T.nonzero()  # (column, row), by column
    ends = np.concatenate([[0], torch.bincount(cols[:, 0], minlength=n).cumsum(0).cpu().numpy()])
    rows_of = cols[:, 1].contiguous()
    par = inside.nonzero()     # (row, column), by row
    pends = np.concatenate([[0], torch.bincount(par[:, 0], minlength=n).cumsum(0).cpu().numpy()])
    cols_of = par[:, 1].contiguous()
    del cols, par, inside
    zero = torch.zeros((), dtype=torch.float64, device=device)
    for j in range(n):
        rows = rows_of[ends[j]:ends[j + 1]]
        parents = cols_of[pends[j]:pends[j + 1] - 1]
        a = L[rows, j]
        if len(parents):
            a = a - L[rows[:, None], parents[None, :]] @ L[j, parents]
        p = a[0]
        if pivot == "zero":
            a = torch.where(p > 0, a / torch.where(p > 0, p, torch.ones_like(p)).sqrt(), zero)
        else:
            p = torch.where(p > tau, p, torch.full_like(p, tau))
            a = a / p.sqrt()
            a[0] = p.sqrt()
        L[rows, j] = a
    dead = L.diagonal() == 0
    L.diagonal()[dead] = 1.0  # a zeroed column has no entries: its component is set to 0 below
    v = torch.from_numpy(b[perm]).to(device)
    v = torch.linalg.solve_triangular(L, torch.where(dead[:, None], zero, v), upper=False)
    v = torch.where(dead[:, None], zero, v)
    v = torch.linalg.solve_triangular(L.T, v, upper=True)
    v = torch.where(dead[:, None], zero, v)
    out = torch.empty_like(v)
    out[torch.from_numpy(perm).to(device)] = v
    return out.cpu()


def exact(case, seed):
    device = "cuda" if torch.cuda.is_available() else "cpu"
    pts, ell, b = _host_inputs(case, seed)
    kind = case["kind"]
    if kind == "dense":
        x, X = torch.from_numpy(pts).to(device), torch.from_numpy(b).to(device)
        step = max(1, (1 << 28) // (8 * len(x)))
        return torch.cat([(_kernel(_distances(x[i:i + step], x), case["nu"], ell) @ X).cpu()
                          for i in range(0, len(x), step)])
    if kind == "super":  # the aggregated ordering is the library's own
        return None
    if kind == "pcg":
        x = torch.from_numpy(pts).to(device)
        return torch.linalg.solve(_kernel(_distances(x, x), case["nu"], ell), torch.from_numpy(b).to(device)).cpu()
    pivot, tau = _pivot(case)
    if kind == "batch":
        if sum(len(p) for p in pts) > 120_000:
            return None
        at = np.concatenate([[0], np.cumsum([len(p) for p in pts])])
        return torch.cat([_exact_solution(p, b[at[i]:at[i + 1]], case["nu"], ell[i], case["rho"], pivot, tau, device)
                          for i, p in enumerate(pts)])
    if len(pts) > EXACT_MOST:
        return None
    out = _exact_solution(pts, b, case["nu"], ell, case["rho"], pivot, tau, device)
    return out.numpy() if kind == "request" else out
