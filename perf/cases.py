"""Timed work of the framework's users, through its public entry points.

What a program does with this library: build a preconditioner of an R-matrix from random
walks (`build_factor`), apply it in PCG (`pcg_solve`, `apply`), do both at once for one
right-hand side, do them for a batch of matrices (`build_factor_batched`,
`pcg_solve_batched`), for an asymmetric matrix (`build_factor_ldu`, `bicgstab_solve`), and
train or serve the walk-budget network (`mlp_train_step_rows`; `row_features`,
`mlp_forward`, `mlp_budgets`).  The matrices are the families of `workloads.py`, drawn on
the GPU: 2D and 3D resistor grids, the Dirichlet Laplacians of the paper's Table 1, 3D
random geometric graphs, asymmetric 3D grids and batches of pruned 2D grids, with the walk
budgets, drop tolerances and solver tolerances those workloads are run with.

A case is a dict of plain values: `kind` (which of the calls above), `family` and `size`
(grid side, or nodes of a random geometric graph), `walks` per row, `drop` and `tol`,
`precision` of the factor, `reuse` of walks, `count` and `nrhs` of a batch, `rows` of a
minibatch.
"""
from __future__ import annotations

import math

import torch

from paper_math_0609672_amd import budget, srw

# walks per row and drop tolerance each family is run with
WALKS = {"grid2d": 64, "grid3d": 256, "laplace3d": 24, "rgg": 512, "grid3d_asym": 256, "pruned": 64}
DROP = {"grid2d": 1e-3, "grid3d": 1e-4, "laplace3d": 0.0, "rgg": 1e-4, "grid3d_asym": 1e-4, "pruned": 1e-3}
TOL = {"grid2d": 1e-8, "grid3d": 1e-8, "laplace3d": 1e-6, "rgg": 1e-10, "grid3d_asym": 1e-8, "pruned": 1e-8}


def _case(kind, family, size, **more):
    c = {"kind": kind, "family": family, "size": int(size), "walks": WALKS[family], "drop": DROP[family],
         "tol": TOL[family], "precision": "fp32" if family == "rgg" else "fp64", "reuse": False}
    c.update(more)
    return c


def listed():
    return [
        # the smallest call: build and solve a circuit-sized 32 x 32 grid, where launches,
        # host round trips and allocations count
        _case("solve", "grid2d", 32, name="solve_grid2d_32"),
        # one row of the paper's Table 1 (m1, 50^3), build and solve
        _case("solve", "laplace3d", 50, name="solve_laplace3d_50"),
        # the headline workload's two halves: the preconditioner of the 128^3 resistor
        # grid (2.1 M rows, 256 walks each) ...
        _case("build", "grid3d", 128, name="build_grid3d_128"),
        # ... and one right-hand side solved with it
        _case("pcg", "grid3d", 128, name="pcg_grid3d_128"),
        # one application of the preconditioner in a caller's own Krylov loop, middle size
        _case("apply", "grid3d", 64, name="apply_grid3d_64"),
        # the largest single matrix: an irregular graph of 2 M nodes, mean degree 24, with
        # the FP32 factor it is run with
        _case("build", "rgg", 2_000_000, name="build_rgg_2m"),
        _case("pcg", "rgg", 2_000_000, name="pcg_rgg_2m"),
        # 256 pruned 2D grids of 1e3 .. 2e5 nodes in one factor, and all their systems,
        # eight right-hand sides each, at once
        _case("batch_build", "pruned", 200_000, count=256, nrhs=8, name="batch_build_256"),
        _case("batch_pcg", "pruned", 200_000, count=256, nrhs=8, name="batch_pcg_256"),
        # an asymmetric matrix: two walk games, then BiCGSTAB
        _case("solve_ldu", "grid3d_asym", 64, name="solve_ldu_grid3d_64"),
        # serving learned walk budgets for the 128^3 grid: features, network, budgets
        _case("budgets", "grid3d", 128, name="budgets_grid3d_128"),
        # one training step of the budget network on a minibatch of 65,536 rows
        _case("train", "grid3d", 64, rows=65536, name="train_step_65536"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "build", "build", "pcg", "apply", "batch_build", "batch_pcg",
                       "solve_ldu", "budgets", "train"])
    if kind == "train":
        return _case(kind, "grid3d", rng.randint(24, 64), rows=_log(rng, 1000, 65536))
    if kind == "budgets":
        return _case(kind, "grid3d", rng.randint(16, 127))
    if kind == "solve_ldu":
        return _case(kind, "grid3d_asym", rng.randint(12, 72), walks=rng.choice([64, 256]))
    if kind in ("batch_build", "batch_pcg"):
        return _case(kind, "pruned", _log(rng, 4000, 200_000), count=_log(rng, 4, 160), nrhs=rng.randint(1, 8),
                     precision=rng.choice(["fp64", "fp64", "fp32"]))
    family = rng.choice(["grid2d", "grid3d", "grid3d", "laplace3d", "rgg"])
    size = {"grid2d": lambda: _log(rng, 9, 700), "grid3d": lambda: rng.randint(11, 120),
            "laplace3d": lambda: rng.randint(13, 100), "rgg": lambda: _log(rng, 2000, 900_000)}[family]()
    c = _case(kind, family, size)
    if kind in ("build", "solve"):
        c["walks"] = max(8, c["walks"] // rng.choice([1, 1, 2, 4]))
        if family != "rgg" and size <= 64:  # walk reuse: few walks, each counted many times
            if rng.random() < 0.2:
                c.update(reuse=True, walks=32)
    if family in ("grid3d", "grid2d"):
        c["precision"] = rng.choice(["fp64", "fp64", "fp32"])
    return c


# --------------------------------------------------------------------- the matrices
def _device():
    return torch.device("cuda") if torch.cuda.is_available() else torch.device("cpu")


def _assemble(n, u, v, g_uv, g_vu, excess):
    """CSR of the network with edges (u, v): entries -g_uv at (u, v), -g_vu at (v, u); the
    diagonal is the larger of a node's row and column sums, plus its excess."""
    dev = u.device
    ids = torch.arange(n, device=dev)
    key = torch.cat([u * n + v, v * n + u, ids * (n + 1)])
    val = torch.cat([-g_uv, -g_vu, torch.zeros_like(excess)])
    key, at = torch.sort(key)
    val = val[at]
    # row sums in entry order (equal seeds are to give equal matrices)
    r = torch.div(key, n, rounding_mode="floor")
    col = key - r * n
    rowptr = torch.searchsorted(r, torch.arange(n + 1, device=dev))
    off = torch.where(r == col, torch.zeros_like(val), -val)
    rs = torch.segment_reduce(off, "sum", lengths=rowptr[1:] - rowptr[:-1])
    if g_uv is not g_vu:
        tkey, tat = torch.sort(col * n + r)
        cs = torch.segment_reduce(off[tat], "sum", lengths=rowptr[1:] - rowptr[:-1])
        rs = torch.maximum(rs, cs)
    val = torch.where(r == col, (rs + excess)[r], val)
    return srw.Matrix(n, rowptr.to(torch.int64), col.to(torch.int32), val)


def _ground(n, frac, lo, hi, gen, dev):
    ng = min(n, max(1, int(round(frac * n))))
    exc = torch.zeros(n, dtype=torch.float64, device=dev)
    at = torch.randperm(n, generator=gen, device=dev)[:ng]
    exc[at] = lo + (hi - lo) * torch.rand(ng, generator=gen, device=dev, dtype=torch.float64)
    return exc


def _grid_edges(dims, dev):
    ids = torch.arange(math.prod(dims), device=dev).reshape(dims[::-1])
    us, vs = [], []
    for ax in range(len(dims) - 1, -1, -1):
        m = ids.shape[ax]
        us.append(ids.narrow(ax, 0, m - 1).reshape(-1))
        vs.append(ids.narrow(ax, 1, m - 1).reshape(-1))
    return torch.cat(us), torch.cat(vs)


def _uniform(k, lo, hi, gen, dev):
    return lo + (hi - lo) * torch.rand(k, generator=gen, device=dev, dtype=torch.float64)


def _rgg_edges(n, gen, dev):
    """Points uniform in the unit cube joined below the radius of expected mean degree 24
    (cell list, each cell against itself and 13 of its neighbours)."""
    def p(r):  # probability that two points lie within r, boundary included
        return 4 * math.pi / 3 * r ** 3 - 1.5 * math.pi * r ** 4 + 1.6 * r ** 5 - r ** 6 / 6
    lo, hi = 0.0, 1.0
    for _ in range(80):
        mid = 0.5 * (lo + hi)
        lo, hi = (mid, hi) if (n - 1) * p(mid) < 24.0 else (lo, mid)
    r = 0.5 * (lo + hi)
    pts = torch.rand(n, 3, generator=gen, device=dev, dtype=torch.float64)
    m = max(1, int(1.0 / r))
    cell = (pts * m).long().clamp_(max=m - 1)
    cid = cell[:, 0] + m * (cell[:, 1] + m * cell[:, 2])
    cs, order = torch.sort(cid, stable=True)
    start = torch.searchsorted(cs, torch.arange(m ** 3 + 1, device=dev))
    pc, ps = cell[order], pts[order]
    us, vs, ds = [], [], []
    near = [(dx, dy, dz) for dz in (-1, 0, 1) for dy in (-1, 0, 1) for dx in (-1, 0, 1) if (dz, dy, dx) >= (0, 0, 0)]
    for dx, dy, dz in near:
        nc = pc + torch.tensor([dx, dy, dz], device=dev)
        src = torch.nonzero(((nc >= 0) & (nc < m)).all(1)).reshape(-1)
        to = nc[src, 0] + m * (nc[src, 1] + m * nc[src, 2])
        first = src + 1 if (dx, dy, dz) == (0, 0, 0) else start[to]
        cnt = start[to + 1] - first
        a = torch.repeat_interleave(src, cnt)
        at = torch.repeat_interleave(first - (torch.cumsum(cnt, 0) - cnt), cnt) + torch.arange(a.numel(), device=dev)
        d = (ps[a] - ps[at]).square().sum(1).sqrt()
        keep = d < r
        us.append(order[a[keep]])
        vs.append(order[at[keep]])
        ds.append(d[keep])
    return torch.cat(us), torch.cat(vs), torch.cat(ds)


def _pruned_grid(n_target, gen, dev):
    """2D grid, 10 % of its edges removed outside a random spanning tree (every node keeps
    the edge to its left or lower neighbour, drawn at random)."""
    nx = max(2, int(round(math.sqrt(n_target))))
    ny = max(2, int(round(n_target / nx)))
    n = nx * ny
    u, v = _grid_edges((nx, ny), dev)
    across = torch.arange(u.numel(), device=dev) < (nx - 1) * ny  # x edges come first
    left = torch.rand(n, generator=gen, device=dev) < 0.5
    x, y = v % nx, torch.div(v, nx, rounding_mode="floor")
    tree = torch.where(across, left[v] | (y == 0), ~left[v] | (x == 0))
    key = torch.where(tree, 2.0, torch.rand(u.numel(), generator=gen, device=dev, dtype=torch.float64))
    n_drop = int(round(0.1 * u.numel()))
    keep = torch.ones(u.numel(), dtype=torch.bool, device=dev)
    keep[torch.argsort(key)[:n_drop]] = False
    u, v = u[keep], v[keep]
    g = _uniform(u.numel(), 0.1, 10.0, gen, dev)
    return _assemble(n, u, v, g, g, _ground(n, 0.02, 0.1, 10.0, gen, dev))


def _batch_sizes(case):
    """`count` sizes from 1,000 nodes to `size`, evenly spread over the logarithm."""
    k = case["count"]
    return [1000.0 * (case["size"] / 1000.0) ** ((i + 0.5) / k) for i in range(k)]


def _matrix(case, seed):
    dev = _device()
    gen = torch.Generator(device=dev).manual_seed(int(seed))
    f, m = case["family"], case["size"]
    if f == "rgg":
        u, v, d = _rgg_edges(m, gen, dev)
        g = (1.0 / d).clamp(1.0, 1e3)
        exc = _ground(m, 0.005, 0.1, 10.0, gen, dev)
        # a component without a grounded node: ground its smallest node
        label = torch.arange(m, device=dev)
        while True:
            low = label.scatter_reduce(0, u, label[v], "amin").scatter_reduce(0, v, label[u], "amin")
            low = low[low]
            if bool((low == label).all()):
                break
            label = low
        has = torch.zeros(m, dtype=torch.bool, device=dev)
        has[label[exc > 0]] = True
        alone = (label == torch.arange(m, device=dev)) & ~has
        return _assemble(m, u, v, g, g, torch.where(alone, torch.ones_like(exc), exc))
    dims = (m, m) if f == "grid2d" else (m, m, m)
    n = math.prod(dims)
    u, v = _grid_edges(dims, dev)
    k = u.numel()
    if f == "grid2d":
        g = _uniform(k, 0.5, 1.5, gen, dev)
        return _assemble(n, u, v, g, g, _ground(n, 0.05, 0.1, 1.0, gen, dev))
    if f == "laplace3d":
        g = torch.ones(k, dtype=torch.float64, device=dev)
        deg = torch.bincount(u, minlength=n) + torch.bincount(v, minlength=n)
        return _assemble(n, u, v, g, g, (6 - deg).to(torch.float64))
    g = torch.exp(_uniform(k, math.log(1e-2), math.log(1e2), gen, dev))
    if f == "grid3d":
        return _assemble(n, u, v, g, g, _ground(n, 0.01, 0.01, 1.0, gen, dev))
    t = _uniform(k, -0.5, 0.5, gen, dev)
    return _assemble(n, u, v, g * (1 + t), g * (1 - t), _ground(n, 0.01, 0.01, 1.0, gen, dev))


def _batch(case, seed):
    dev = _device()
    gen = torch.Generator(device=dev).manual_seed(int(seed))
    return [_pruned_grid(s, gen, dev) for s in _batch_sizes(case)]


def _rhs(n, seed, *more):
    gen = torch.Generator(device=_device()).manual_seed(int(seed) + 7919)
    return torch.randn(n, *more, generator=gen, device=_device(), dtype=torch.float64)


# ------------------------------------------------------------------------ the passes
def _build(case, A, seed):
    return srw.build_factor(A, case["walks"], case["drop"], seed, precision=case["precision"], reuse=case["reuse"])


# room per row for the exported entries of Y (the entries differ a little by seed; a
# program that exports factors keeps buffers that are large enough)
ROOM = {"grid2d": 24, "grid3d": 36, "laplace3d": 26, "rgg": 130, "pruned": 16}


def _room(case, n):
    k = int(n * (ROOM[case["family"]] * (3 if case["reuse"] else 1)) + 64)
    t = torch.float32 if case["precision"] == "fp32" else torch.float64
    return (torch.zeros(k, dtype=torch.int32, device=_device()), torch.zeros(k, dtype=t, device=_device()))


def _export(s, F):
    """The whole factor: row starts, columns and values of Y (in the program's buffers), D
    and the ordering."""
    out = F.export()
    m = out["ycol"].numel()
    s["ycol"][:m].copy_(out["ycol"])
    s["yval"][:m].copy_(out["yval"])
    return {"yptr": out["yptr"], "ycol": s["ycol"], "yval": s["yval"], "d": out["d"], "rank": out["rank"]}


def _train_data(case, seed):
    """Features and targets of the training set: rows of a grid and labels of the size the
    measured ones have."""
    A = _matrix(case, seed)
    X = srw.row_features(A, srw.ordering(A.n, seed, A.rowptr.device))
    gen = torch.Generator(device=_device()).manual_seed(int(seed) + 1)
    y = X[:, 3] - 0.5 * X[:, 6] + 0.2 * torch.randn(A.n, generator=gen, device=X.device)
    rows = torch.randint(0, A.n, (case["rows"],), generator=gen, device=X.device, dtype=torch.int32)
    return X, y, rows


def prepare(case, seed):
    kind = case["kind"]
    s = {"kind": kind, "case": case, "seed": int(seed)}
    if kind in ("batch_build", "batch_pcg"):
        s["mats"] = _batch(case, seed)
        s["seeds"] = [int(seed) + i for i in range(case["count"])]
        if kind == "batch_pcg":
            s["F"] = srw.build_factor_batched(s["mats"], case["walks"], case["drop"], s["seeds"],
                                              precision=case["precision"])
            s["B"] = _rhs(sum(m.n for m in s["mats"]), seed, case["nrhs"])
            del s["mats"]
        else:
            s["ycol"], s["yval"] = _room(case, sum(m.n for m in s["mats"]))
        return s
    if kind == "train":
        s["X"], s["y"], s["rows"] = _train_data(case, seed)
        s["mu_sd"], _ = srw.mlp_standardize(s["X"], s["y"])
        s["P"] = budget.init_params(seed, _device())
        s["m"], s["v"] = torch.zeros_like(s["P"]), torch.zeros_like(s["P"])
        s["loss"] = torch.zeros(1, dtype=torch.float32, device=_device())
        s["grad"] = torch.zeros_like(s["P"])
        s["step"] = 0
        return s
    s["A"] = _matrix(case, seed)
    if kind == "budgets":
        s["P"] = budget.init_params(seed, _device())
        s["rank"] = srw.ordering(s["A"].n, seed, _device())  # the build's own ordering
        s["mu_sd"] = srw.mlp_standardize(srw.row_features(s["A"], s["rank"]))
        return s
    if kind == "build":
        s["ycol"], s["yval"] = _room(case, s["A"].n)
    if kind in ("solve", "solve_ldu", "pcg", "apply"):
        s["b"] = _rhs(s["A"].n, seed)
    if kind in ("pcg", "apply"):
        s["F"] = _build(case, s["A"], seed)
    return s


def run(s):
    case, kind = s["case"], s["kind"]
    if kind == "build":
        F = _build(case, s["A"], s["seed"])
        out = _export(s, F)
        F.free()
        return out
    if kind == "solve":
        F = _build(case, s["A"], s["seed"])
        _, x, it, _ = srw.pcg_solve(s["A"], F, s["b"], case["tol"])
        F.free()
        return {"x": x, "iters": it}
    if kind == "pcg":
        _, x, it, _ = srw.pcg_solve(s["A"], s["F"], s["b"], case["tol"])
        return {"x": x, "iters": it}
    if kind == "apply":
        return srw.apply(s["F"], s["b"])
    if kind == "batch_build":
        F = srw.build_factor_batched(s["mats"], case["walks"], case["drop"], s["seeds"], precision=case["precision"])
        out = _export(s, F)
        F.free()
        return out
    if kind == "batch_pcg":
        _, X, it, _ = srw.pcg_solve_batched(s["F"], s["B"], case["tol"], 1000)
        return {"x": X, "iters": it}
    if kind == "solve_ldu":
        F = srw.build_factor_ldu(s["A"], case["walks"], case["drop"], s["seed"], precision=case["precision"])
        _, x, it, _ = srw.bicgstab_solve(s["A"], F, s["b"], case["tol"])
        F.free()
        return {"x": x, "iters": it}
    if kind == "budgets":
        feat = srw.row_features(s["A"], s["rank"])
        pred = srw.mlp_forward(s["P"], s["mu_sd"], feat)
        return {"features": feat, "pred": pred, "walks": srw.mlp_budgets(pred, 5e-3, 8, 8192)}
    s["step"] += 1
    srw.mlp_train_step_rows(s["P"], s["mu_sd"], s["X"], s["y"], s["rows"], adam_m=s["m"], adam_v=s["v"],
                            step=s["step"], lr=2e-3, grad=s["grad"], loss=s["loss"])
    return {"params": s["P"], "m": s["m"], "v": s["v"], "grad": s["grad"], "loss": s["loss"]}


# -------------------------------------------------------------------------- the work
# entries of Y per row (drop and budget as listed) that the families give
Y_PER_ROW = {"grid2d": 6.0, "grid3d": 21.0, "laplace3d": 13.0, "rgg": 89.0, "grid3d_asym": 9.0, "pruned": 8.0}
DEGREE = {"grid2d": 4.0, "grid3d": 6.0, "laplace3d": 6.0, "rgg": 24.0, "grid3d_asym": 6.0, "pruned": 3.6}
ITERS = {"grid2d": 9, "grid3d": 11, "laplace3d": 19, "rgg": 11, "grid3d_asym": 4, "pruned": 15}


def work(case):
    """One pass: the matrix read, the factor written (build) or read twice an iteration
    (solves), vectors read and written; two operations per entry that is multiplied, and
    for a build one comparison per step of every walk (about 2.3 ln n steps a walk on the
    graphs whose walks end at lower ranks only, 4 on the asymmetric grids)."""
    f, kind = case["family"], case["kind"]
    n = case["size"] ** (2 if f == "grid2d" else 1 if f in ("rgg", "pruned") else 3)
    if f == "pruned":
        n = sum(_batch_sizes(case))
    nrhs = case.get("nrhs", 1) if kind == "batch_pcg" else 1
    value = 4 if case["precision"] == "fp32" else 8
    a = n * (8 + 12 * (DEGREE[f] + 1))
    y = n * (8 + (4 + value) * Y_PER_ROW[f] + value)
    steps = n * case["walks"] * (4.0 if f == "grid3d_asym" else 2.3 * math.log(max(n, 3)))
    games = 2 if kind == "solve_ldu" else 1
    build = {"bytes": a + games * y, "flops": games * steps}
    entries = n * nrhs * 2 * (DEGREE[f] + 1 + 2 * Y_PER_ROW[f])
    solve = {"bytes": ITERS[f] * (a + 2 * y) + 16 * n * nrhs, "flops": ITERS[f] * entries}
    if kind in ("build", "batch_build"):
        return build
    if kind in ("pcg", "batch_pcg"):
        return solve
    if kind == "apply":
        return {"bytes": 2 * y + 16 * n, "flops": 4 * n * Y_PER_ROW[f]}
    if kind in ("solve", "solve_ldu"):
        return {k: build[k] + solve[k] for k in build}
    net = 2.0 * (8 * 64 + 64 * 64 + 64)
    if kind == "budgets":
        return {"bytes": a + 4 * n + 40 * n, "flops": n * net}
    return {"bytes": case["rows"] * 40.0, "flops": 3 * case["rows"] * net}


# ------------------------------------------------------------------ the values in 64 bits
def _csr(A):
    return torch.sparse_csr_tensor(A.rowptr, A.col.long(), A.val, size=(A.n, A.n))


def _diag(A):
    r = torch.repeat_interleave(torch.arange(A.n, device=A.val.device), A.rowptr[1:] - A.rowptr[:-1])
    return A.val[r == A.col]


def _cg(A, B):
    """A x = b by conjugate gradients with the diagonal, to rounding; None if it stalls."""
    S, D = _csr(A), _diag(A)
    cols = []
    for b in B.unbind(1):
        x, r = torch.zeros_like(b), b.clone()
        z = r / D
        p, rho = z, torch.dot(r, z)
        best, worth = None, math.inf
        for k in range(6000):
            q = S @ p
            alpha = rho / torch.dot(p, q)
            x = x + alpha * p
            r = r - alpha * q
            z = r / D
            new = torch.dot(r, z)
            p = z + (new / rho) * p
            rho = new
            if k % 25 == 24:
                rel = float(torch.linalg.vector_norm(r) / torch.linalg.vector_norm(b))
                if rel < 1e-15:
                    break
        true = float(torch.linalg.vector_norm(b - S @ x) / torch.linalg.vector_norm(b))
        if not true < 1e-12:
            return None
        cols.append(x)
    return torch.stack(cols, 1)


def _bicgstab(A, b):
    S, D = _csr(A), _diag(A)
    x, r = torch.zeros_like(b), b.clone()
    rt, p, v = r.clone(), torch.zeros_like(b), torch.zeros_like(b)
    rho = alpha = w = torch.ones((), dtype=b.dtype, device=b.device)
    for _ in range(3000):
        new = torch.dot(rt, r)
        p = r + (new / rho) * (alpha / w) * (p - w * v)
        rho = new
        y = p / D
        v = S @ y
        alpha = rho / torch.dot(rt, v)
        h = r - alpha * v
        z = h / D
        t = S @ z
        w = torch.dot(t, h) / torch.dot(t, t)
        x = x + alpha * y + w * z
        r = h - w * t
        if float(torch.linalg.vector_norm(r) / torch.linalg.vector_norm(b)) < 1e-15:
            break
    ok = float(torch.linalg.vector_norm(b - S @ x) / torch.linalg.vector_norm(b)) < 1e-12
    return x if ok else None


def _net(P, mu_sd, X):
    W1, b1 = P[:512].reshape(8, 64), P[512:576]
    W2, b2 = P[576:4672].reshape(64, 64), P[4672:4736]
    W3, b3 = P[4736:4800], P[4800]
    h = torch.relu(((X - mu_sd[:8]) / mu_sd[8:]) @ W1 + b1)
    return torch.relu(h @ W2 + b2) @ W3 + b3


def _features(A, rank):
    n, dev = A.n, A.val.device
    cnt = A.rowptr[1:] - A.rowptr[:-1]
    r = torch.repeat_interleave(torch.arange(n, device=dev), cnt)
    col = A.col.long()
    off = r != col
    a = A.val[~off]
    r, col, w = r[off], col[off], -A.val[off]
    deg = cnt - 1

    def over(x, how="sum"):
        return torch.segment_reduce(x.double(), how, lengths=deg, unsafe=True)

    e = a - over(w)
    up = (rank[col] > rank[r]).double()
    some = deg > 0
    d = deg.clamp(min=1).double()
    spread = torch.where(some, torch.log(over(w, "max") / over(w, "min")), torch.zeros_like(a))
    return torch.stack([deg.double(), torch.log(a), e / a, over(w * up) / a, over(up) / d, spread,
                        torch.log(n / (rank.double() + 1.0)), over((e / a)[col]) / d], 1)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("build", "batch_build", "apply"):
        return None  # the factor is a sample of the walks: no value of its own in 64 bits
    if kind in ("solve", "pcg"):
        A = _matrix(case, seed)
        x = _cg(A, _rhs(A.n, seed).unsqueeze(1))
        return None if x is None else {"x": x[:, 0], "iters": None}
    if kind == "solve_ldu":
        A = _matrix(case, seed)
        x = _bicgstab(A, _rhs(A.n, seed))
        return None if x is None else {"x": x, "iters": None}
    if kind == "batch_pcg":
        mats = _batch(case, seed)
        row, nz, ptr, cols = 0, 0, [torch.zeros(1, dtype=torch.int64, device=_device())], []
        for m in mats:
            ptr.append(m.rowptr[1:] + nz)
            cols.append(m.col + row)
            row, nz = row + m.n, nz + m.nnz
        A = srw.Matrix(row, torch.cat(ptr), torch.cat(cols), torch.cat([m.val for m in mats]))
        if row * case["nrhs"] > 30_000_000:
            return None
        x = _cg(A, _rhs(row, seed, case["nrhs"]))
        return None if x is None else {"x": x, "iters": None}
    if kind == "budgets":
        s = prepare(case, seed)
        X = _features(s["A"], s["rank"])
        return {"features": X, "pred": _net(s["P"].double(), s["mu_sd"].double(), X), "walks": None}
    s = prepare(case, seed)
    P = s["P"].double().requires_grad_(True)
    at = s["rows"].long()
    err = _net(P, s["mu_sd"].double(), s["X"].double()[at]) - s["y"].double()[at]
    loss = err.square().mean()
    (g,) = torch.autograd.grad(loss, P)
    return {"params": None, "m": None, "v": None, "grad": g, "loss": loss.detach().reshape(1)}
