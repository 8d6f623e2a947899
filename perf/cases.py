"""The calls whose speed counts, as a program of this package makes them.

Every case prepares a matrix on the GPU, the solver context (or batch engine)
such a program keeps, and a right-hand side b = A x* with x* drawn from the
seed, and then makes one call through the package's public entry points:

  solve     Solver.solve: Algorithm II (eps1 = "auto"), Algorithm I (a fixed
            eps1) or FP64-only CG ("none"), with or without Jacobi
            preconditioning, down to a true relative residual of 1e-10
  jacobi    Solver.solve_jacobi, the two-stage Jacobi iteration
  spmv      Solver.spmv, one product in FP64 or FP32
  features  Solver.features, the 2BFS and the k0 prefix
  batch     BatchSolver.submit + wait_all of many systems at once

Matrix families: the 5-point Laplacian of a square grid (lap2d), the 7-point
variable-coefficient diffusion of a cubic grid with face coefficients
10^U(0,3) (varcoef3d), the full random band of half-width w (banded), the
random dominant band of half-width 8, density 0.8 and mu = 3 (domband), the
Laplacian of a random graph of mean degree 16 (er), and random trees with
extra edges (tree; n = 1000, the sizes of the labelling experiment).

Iteration counts are returned where a call is reproducible bit for bit; an
Algorithm II solve of more than 524,288 rows is not (its FP32 products take
another grid while the 2BFS runs beside them), so there the solution, the
status, the chosen class and the graph features are returned.
"""

import math

import numpy as np
import torch

from paper_2412_08059_amd import DEFAULT_MODEL, MPCG_EPS1_AUTO, MPCG_EPS1_NONE, BatchSolver, DeviceCSR, Solver

EPS2 = 1e-10
REPRODUCIBLE_ROWS = 524288


def listed():
    return [
        # the smallest solve: a 64 x 64 Poisson grid (launches and latency decide)
        {"name": "solve_lap2d_64", "kind": "solve", "family": "lap2d", "size": 64, "eps1": 1e-4, "precond": 0},
        # a mid-sized grid with an odd, ragged side, the tolerance chosen by the kNN
        {"name": "auto_varcoef3d_49", "kind": "solve", "family": "varcoef3d", "size": 49, "eps1": "auto", "precond": 0},
        # the benchmark's system: the mixed solve and the FP64-only comparator
        {"name": "auto_varcoef3d_128", "kind": "solve", "family": "varcoef3d", "size": 128, "eps1": "auto", "precond": 0},
        {"name": "fp64_varcoef3d_128", "kind": "solve", "family": "varcoef3d", "size": 128, "eps1": "none", "precond": 0},
        # the Jacobi-preconditioned two-stage solve
        {"name": "pcg_varcoef3d_97", "kind": "solve", "family": "varcoef3d", "size": 97, "eps1": 1e-6, "precond": 1},
        # the two graphs of the diameter contrast: a band (a deep 2BFS) and a random graph (scattered gathers)
        {"name": "auto_banded_1m", "kind": "solve", "family": "banded", "size": 1000000, "eps1": "auto", "precond": 0},
        {"name": "auto_er_1m", "kind": "solve", "family": "er", "size": 1000000, "eps1": "auto", "precond": 0},
        # two-stage Jacobi on the 2^21 band
        {"name": "jacobi_domband_2m", "kind": "jacobi", "family": "domband", "size": 2097152, "eps1": 1e-4},
        # one product of the largest matrix (68 M entries, beyond the 256 MB Infinity Cache)
        {"name": "spmv_banded_4m", "kind": "spmv", "family": "banded", "size": 4000000, "precision": 64},
        # graph features alone, on a square grid whose 2BFS is about 2,000 levels deep
        {"name": "features_lap2d_1001", "kind": "features", "family": "lap2d", "size": 1001},
        # many systems of every family at once, each choosing its own tolerance
        {"name": "batch_mixed_96", "kind": "batch", "family": "mixed", "count": 96, "n_lo": 1000, "n_hi": 100000,
         "eps1": "auto"},
        # the labelling experiment: many n = 1000 systems at one fixed tolerance
        {"name": "batch_tree_512", "kind": "batch", "family": "tree", "count": 512, "n_lo": 1000, "n_hi": 1000,
         "eps1": 1e-4},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _grid_side(rng, family, lo, hi):
    n = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(3, int(round(n ** (0.5 if family == "lap2d" else 1.0 / 3.0))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "solve", "jacobi", "spmv", "features", "batch"])
    if kind == "batch":
        family = rng.choice(["mixed", "tree"])
        eps1 = rng.choice(["auto", "none", 1e-4, 1e-6])
        if family == "tree":
            return {"kind": kind, "family": family, "count": _log_int(rng, 16, 512), "n_lo": 300, "n_hi": 1000,
                    "eps1": eps1}
        return {"kind": kind, "family": family, "count": _log_int(rng, 8, 96), "n_lo": 1000,
                "n_hi": _log_int(rng, 2000, 100000), "eps1": eps1}
    if kind == "jacobi":
        return {"kind": kind, "family": "domband", "size": _log_int(rng, 1000, 2097152),
                "eps1": rng.choice([1e-2, 1e-4, 1e-6, "none"])}
    family = rng.choice(["lap2d", "varcoef3d", "banded", "er"])
    if kind == "spmv":
        size = _grid_side(rng, family, 1000, 4e6) if family in ("lap2d", "varcoef3d") else \
            _log_int(rng, 1000, 4000000 if family == "banded" else 1000000)
        return {"kind": kind, "family": family, "size": size, "precision": rng.choice([32, 64])}
    if kind == "features":
        size = _grid_side(rng, family, 1000, 1e6) if family in ("lap2d", "varcoef3d") else _log_int(rng, 1000, 1000000)
        return {"kind": kind, "family": family, "size": size}
    size = _grid_side(rng, family, 1000, 1e6 if family == "lap2d" else 2097152) \
        if family in ("lap2d", "varcoef3d") else _log_int(rng, 1000, 1000000)
    return {"kind": kind, "family": family, "size": size, "eps1": rng.choice(["auto", "auto", "none", 1e-3, 1e-5]),
            "precond": rng.choice([0, 0, 0, 1])}


# ---------------------------------------------------------------- matrices --


def _gen(seed, device="cuda"):
    g = torch.Generator(device=device)
    g.manual_seed(0x5EED + 7919 * int(seed))
    return g


def _uniform(shape, g, lo=0.0, hi=1.0):
    return torch.rand(shape, generator=g, dtype=torch.float64, device=g.device) * (hi - lo) + lo


def _from_diagonals(n, offs, vals, here):
    """CSR of the diagonals `offs` (increasing), vals/here: [n, len(offs)] by row."""
    i = torch.arange(n, dtype=torch.int64, device=vals.device)
    col = i[:, None] + torch.tensor(offs, dtype=torch.int64, device=vals.device)[None, :]
    here = here & (col >= 0) & (col < n)
    rp = torch.zeros(n + 1, dtype=torch.int64, device=vals.device)
    rp[1:] = torch.cumsum(here.sum(dim=1), 0)
    return rp.to(torch.int32), col[here].to(torch.int32), vals[here].contiguous()


def _lap2d(N, g):
    n = N * N
    i = torch.arange(n, device="cuda")
    x, y = i % N, i // N
    offs = [-N, -1, 0, 1, N]
    here = torch.stack([y > 0, x > 0, torch.ones_like(x, dtype=torch.bool), x < N - 1, y < N - 1], dim=1)
    vals = torch.tensor([-1.0, -1.0, 4.0, -1.0, -1.0], dtype=torch.float64, device="cuda").expand(n, 5)
    return _from_diagonals(n, offs, vals, here)


def _varcoef3d(N, g):
    n = N ** 3
    fx = 10.0 ** _uniform((N, N, N + 1), g, 0.0, 3.0)
    fy = 10.0 ** _uniform((N, N + 1, N), g, 0.0, 3.0)
    fz = 10.0 ** _uniform((N + 1, N, N), g, 0.0, 3.0)
    faces = [fz[:-1], fy[:, :-1, :], fx[:, :, :-1], fx[:, :, 1:], fy[:, 1:, :], fz[1:]]
    diag = ((((faces[2] + faces[3]) + faces[1]) + faces[4]) + faces[0]) + faces[5]
    vals = torch.stack([-faces[0], -faces[1], -faces[2], diag, -faces[3], -faces[4], -faces[5]],
                       dim=-1).reshape(n, 7)
    i = torch.arange(n, device="cuda")
    x, y, z = i % N, (i // N) % N, i // (N * N)
    here = torch.stack([z > 0, y > 0, x > 0, torch.ones_like(x, dtype=torch.bool), x < N - 1, y < N - 1, z < N - 1],
                       dim=1)
    return _from_diagonals(n, [-N * N, -N, -1, 0, 1, N, N * N], vals, here)


def _band(n, w, g, density, mu):
    """Symmetric band of half-width w: full and U[-1, 0) with a slightly
    dominant diagonal (mu None), or present with probability `density` and
    +-U(0, 3) / +-U(7, 10) with a_ii = mu * sum |a_ij|."""
    vals = torch.zeros((n, 2 * w + 1), dtype=torch.float64, device="cuda")
    here = torch.zeros((n, 2 * w + 1), dtype=torch.bool, device="cuda")
    here[:, w] = True
    for d in range(1, w + 1):
        if mu is None:
            v = _uniform(n, g, -1.0, 0.0)
            v[v == 0.0] = -0.5
            keep = torch.ones(n, dtype=torch.bool, device="cuda")
        else:
            u = _uniform((n, 4), g)
            mag = torch.where(u[:, 0] > 0.5, 3.0 * u[:, 2], 7.0 + 3.0 * u[:, 2])
            v = torch.where(u[:, 1] > 0.5, mag, -mag)
            keep = (u[:, 3] < density) & (v != 0.0)
        keep[max(0, n - d):] = False
        v = torch.where(keep, v, torch.zeros_like(v))
        vals[:, w + d] = v
        here[:, w + d] = keep
        if n > d:
            vals[d:, w - d] = v[:n - d]
            here[d:, w - d] = keep[:n - d]
    s = torch.zeros(n, dtype=torch.float64, device="cuda")
    for k in range(2 * w + 1):
        s = s + vals[:, k].abs()
    vals[:, w] = s + 1e-4 if mu is None else torch.clamp(mu * s, min=1.0)
    return _from_diagonals(n, list(range(-w, w + 1)), vals, here)


def _graph_csr(n, lo, hi, w, diag):
    """CSR from distinct edges (lo < hi) with weights w and the diagonal."""
    i = torch.arange(n, dtype=torch.int64, device=lo.device)
    rows, cols = torch.cat([lo, hi, i]), torch.cat([hi, lo, i])
    order = torch.argsort(rows * n + cols)
    rp = torch.zeros(n + 1, dtype=torch.int64, device=lo.device)
    rp[1:] = torch.cumsum(torch.bincount(rows, minlength=n), 0)
    return rp.to(torch.int32), cols[order].to(torch.int32), torch.cat([w, w, diag])[order].contiguous()


def _er(n, g):
    m = 8 * n
    ij = torch.randint(0, n, (int(2.3 * m) + 64,), generator=g, device=g.device)
    a, b = ij[::2], ij[1::2]
    k = min(a.numel(), b.numel())
    a, b = a[:k], b[:k]
    ok = a != b
    lo, hi = torch.minimum(a, b)[ok], torch.maximum(a, b)[ok]
    key = torch.unique(lo * n + hi)
    key = key[torch.randperm(key.numel(), generator=g, device=g.device)[:m]]
    lo, hi = key // n, key % n
    deg = torch.bincount(lo, minlength=n) + torch.bincount(hi, minlength=n)
    return _graph_csr(n, lo, hi, -torch.ones(key.numel(), dtype=torch.float64, device=g.device),
                      deg.double() + 1e-3)


def _tree(n, g):
    """Random recursive tree plus a share of extra edges, +-U values, mu = 1.1 (host: small)."""
    i = torch.arange(1, n)
    p = (torch.rand(n - 1, generator=g, dtype=torch.float64) * i).long()
    c = [0.1, 0.5, 1.0, 2.0, 3.0, 5.0][int(torch.randint(0, 6, (1,), generator=g))]
    e = torch.randint(0, n, (2, int(c * n)), generator=g)
    a, b = torch.cat([p, e[0]]), torch.cat([i, e[1]])
    ok = a != b
    key = torch.unique(torch.minimum(a, b)[ok] * n + torch.maximum(a, b)[ok])
    lo, hi = key // n, key % n
    u = torch.rand((key.numel(), 3), generator=g, dtype=torch.float64)
    mag = torch.where(u[:, 0] > 0.5, 3.0 * u[:, 2], 7.0 + 3.0 * u[:, 2]) + 1e-3
    w = torch.where(u[:, 1] > 0.5, mag, -mag)
    s = np.bincount(lo.numpy(), weights=mag.numpy(), minlength=n) + np.bincount(hi.numpy(), weights=mag.numpy(),
                                                                              minlength=n)
    rp, col, val = _graph_csr(n, lo, hi, w, torch.from_numpy(1.1 * s))
    return rp.cuda(), col.cuda(), val.cuda()


def _matrix(family, size, seed):
    if family == "tree":
        return _tree(size, _gen(seed, "cpu"))
    g = _gen(seed)
    if family == "lap2d":
        return _lap2d(size, g)
    if family == "varcoef3d":
        return _varcoef3d(size, g)
    if family == "banded":
        return _band(size, 8, g, 1.0, None)
    if family == "domband":
        return _band(size, 8, g, 0.8, 3.0)
    return _er(size, g)


def _row_sums(rp, v):
    """Sum of v over each CSR row, entry by entry in row order (no atomics)."""
    lens = (rp[1:] - rp[:-1]).long()
    start = rp[:-1].long()
    s = torch.zeros(lens.numel(), dtype=torch.float64, device=v.device)
    for k in range(int(lens.max())):
        at = (start + k).clamp(max=v.numel() - 1)
        s = torch.where(lens > k, s + v[at], s)
    return s


def _system(family, size, seed):
    """(DeviceCSR, x*, b = A x*)."""
    rp, col, val = _matrix(family, size, seed)
    n = rp.numel() - 1
    xs = _uniform(n, _gen(seed + 1000003), -1.0, 1.0)
    b = _row_sums(rp, val * xs[col.long()])
    return DeviceCSR(rp, col, val, n), xs, b


def _eps1(v):
    return MPCG_EPS1_AUTO if v == "auto" else MPCG_EPS1_NONE if v == "none" else float(v)


def _batch_plan(case, seed):
    """(family, size, seed) of each system of a batch, sizes log-uniform."""
    r = np.random.default_rng(991 + case["count"])   # the mix belongs to the case, the values to the seed
    out = []
    for k in range(case["count"]):
        fam = case["family"] if case["family"] != "mixed" else ("lap2d", "varcoef3d", "banded", "er")[k % 4]
        n = int(round(math.exp(r.uniform(math.log(case["n_lo"]), math.log(case["n_hi"])))))
        size = int(round(n ** 0.5)) if fam == "lap2d" else int(round(n ** (1 / 3))) if fam == "varcoef3d" else n
        out.append((fam, size, 1009 * int(seed) + k))
    return out


def _slots(n):
    return -(-n // 64) * 64


# ------------------------------------------------------------------ a pass --


def prepare(case, seed):
    if case["kind"] == "batch":
        systems, rows, entries = [], 0, 0
        plan = [_system(*p) for p in _batch_plan(case, seed)]
        x = torch.empty(sum(A.n for A, _, _ in plan), dtype=torch.float64, device="cuda")
        at = 0
        for A, _, b in plan:
            lens = A.row_ptr[1:] - A.row_ptr[:-1]
            pad = torch.zeros(_slots(A.n), dtype=lens.dtype, device="cuda")
            pad[:A.n] = lens
            entries += 64 * int(pad.view(-1, 64).max(dim=1).values.sum())
            rows += _slots(A.n)
            systems.append((A, b, x[at:at + A.n], _eps1(case["eps1"]), EPS2))
            at += A.n
        return {"case": case, "engine": BatchSolver(rows, entries, len(systems)), "systems": systems, "x": x}
    A, xs, b = _system(case["family"], case["size"], seed)
    solver = Solver(A.n, A.nnz, model=DEFAULT_MODEL, precond=case.get("precond", 0))
    state = {"case": case, "A": A, "b": b, "solver": solver}
    if case["kind"] == "spmv":
        state["v"] = xs if case["precision"] == 64 else xs.float()
    return state


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "batch":
        ids = state["engine"].submit(state["systems"])
        got = state["engine"].wait_all(ids)
        stats = [got[i][0] for i in ids]
        return {"x": state["x"], "counts": np.array([[s.status, s.n1, s.n2, s.eps1_class, s.feat.pdiam]
                                                     for s in stats], dtype=np.int64)}
    A, solver = state["A"], state["solver"]
    if kind == "spmv":
        status, y = solver.spmv(A, state["v"], case["precision"])
        return {"y": y, "status": int(status)}
    if kind == "features":
        status, f = solver.features(A, state["b"])
        return {"graph": np.array([status, f.n, f.m, f.pdiam, f.bfs_t, f.bfs_u, f.n_components, f.k0_used],
                                  dtype=np.int64), "v": float(f.v)}
    if kind == "jacobi":
        status, x, s = solver.solve_jacobi(A, state["b"], _eps1(case["eps1"]), EPS2)
        return {"x": x, "counts": np.array([status, s.n1, s.n2], dtype=np.int64)}
    status, x, s = solver.solve(A, state["b"], _eps1(case["eps1"]), EPS2)
    counts = [status, s.eps1_class, s.feat.pdiam, s.feat.bfs_t, s.feat.bfs_u, s.feat.n_components]
    if case["eps1"] != "auto" or A.n <= REPRODUCIBLE_ROWS:
        counts += [s.n1, s.n2, s.restarts]
    return {"x": x, "counts": np.array(counts, dtype=np.int64)}


def exact(case, seed):
    if case["kind"] == "features":
        return None   # integers, and ratios of FP32 norms
    if case["kind"] == "batch":
        return {"x": torch.cat([_system(*p)[1] for p in _batch_plan(case, seed)]), "counts": None}
    A, xs, b = _system(case["family"], case["size"], seed)
    if case["kind"] == "spmv":
        v = xs if case["precision"] == 64 else xs.float().double()
        return {"y": _row_sums(A.row_ptr, A.val * v[A.col.long()]), "status": None}
    return {"x": xs, "counts": None}   # b = A x* was formed from it


# ------------------------------------------------------------- work a pass --

_NNZ = {"lap2d": 5, "varcoef3d": 7, "banded": 17, "domband": 14, "er": 17, "tree": 5}


def _iterations(family, n, eps1, precond=0):
    """(FP32, FP64) iterations, roughly: from the families' condition numbers."""
    if family == "lap2d":
        full = 3.1 * n ** 0.5
    elif family == "varcoef3d":
        full = (5.0 if precond else 8.8) * n ** (1 / 3)
    elif family == "banded":
        full = min(n, 1300)
    elif family == "er":
        full = 45
    elif family == "domband":
        full = 15
    else:
        full = 70
    if eps1 == "none":
        return 0, full
    t = 6 if eps1 == "auto" else -math.log10(eps1)
    return 0.1 * t * full, (1.0 - 0.07 * t) * full


def _solve_work(family, size, eps1, precond=0, jacobi=False):
    n = size ** 2 if family == "lap2d" else size ** 3 if family == "varcoef3d" else size
    m = _NNZ[family] * n
    idx = 4 if family in ("er", "tree") else 0   # a fixed stencil or band needs no stored columns
    n1, n2 = _iterations(family, n, eps1, precond)
    vecs = 4 if jacobi else 9 + 2 * precond
    bytes_ = n1 * ((4 + idx) * m + vecs * 4 * n) + n2 * ((8 + idx) * m + vecs * 8 * n) + 12 * m + 16 * n
    return bytes_, (n1 + n2) * (2 * m + 10 * n)


def work(case):
    kind = case["kind"]
    if kind == "batch":
        parts = [_solve_work(f, s, case["eps1"]) for f, s, _ in _batch_plan(case, 0)]
        return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}
    if kind in ("solve", "jacobi"):
        b, f = _solve_work(case["family"], case["size"], case["eps1"], case.get("precond", 0), kind == "jacobi")
        return {"bytes": b, "flops": f}
    size, family = case["size"], case["family"]
    n = size ** 2 if family == "lap2d" else size ** 3 if family == "varcoef3d" else size
    m = _NNZ[family] * n
    if kind == "spmv":   # CSR in, the vector in, the product out
        return {"bytes": 12 * m + 4 * n + case["precision"] // 8 * 2 * n, "flops": 2 * m}
    return {"bytes": 12 * m + 2 * (4 * m + 8 * n) + 20 * (4 * m + 36 * n), "flops": 20 * (2 * m + 10 * n)}
