"""Matrices on few diagonals that are symmetric only to rounding: SELL-64's bits,
wherever the unequal pair lies, and no second ingest for the usual ones."""

import time

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _unequal(a, which):
    """a with some upper entries one unit in the last place smaller."""
    rows = np.repeat(np.arange(a.n), np.diff(a.row_ptr))
    upper = np.flatnonzero(a.col > rows)
    at = {"all": upper, "first": upper[:1], "last": upper[-1:], "middle": upper[len(upper) // 2:][:1]}[which]
    val = a.val.copy()
    val[at] = np.nextafter(val[at], 0.0)
    return W.CSR(a.n, a.row_ptr, a.col, val, a.name)


@pytest.mark.parametrize("which", ["all", "first", "middle", "last"])
@pytest.mark.parametrize("name,gen", [
    ("grid", lambda: W.poisson2d(77)), ("stencil", lambda: W.varcoef3d(18, seed=2)), ("band", lambda: W.banded(5000, 8, seed=3)),
    ("path", lambda: W.path(65)), ("small", lambda: W.banded(40, 3, seed=4)),
])
def test_same_bits_as_sell(name, gen, which):
    import torch
    from paper_2412_08059_amd import DeviceCSR, Solver
    a = _unequal(gen(), which)
    dev = DeviceCSR.from_host(a)
    b = torch.from_numpy(W.rhs(a, seed=5)[1]).cuda()
    got = []
    for variant in (0, 1):
        s = Solver(a.n, a.nnz, spmv_variant=variant, maxit1=50, maxit2=50, max_restarts=1)
        st, x, stats = s.solve(dev, b, 1e-4, 1e-9)
        js, jx, jstats = s.solve_jacobi(dev, b, 1e-4, 1e-9)
        got.append((st, stats.n1, stats.n2, stats.flags, js, jstats.n1, jstats.n2, x.cpu().numpy().view(np.int64),
                    jx.cpu().numpy().view(np.int64)))
        s.close()
    assert got[0][:7] == got[1][:7]
    assert np.array_equal(got[0][7], got[1][7]) and np.array_equal(got[0][8], got[1][8])


@pytest.mark.parametrize("name,gen", [("grid_1001", lambda: W.poisson2d(1001)), ("stencil_128", lambda: W.varcoef3d(128, seed=2))])
def test_one_ingest(name, gen):
    """A solve of one iteration a phase takes at most a quarter more than with
    SELL-64 asked for (least of 20 calls each, in turn; a second ingest takes
    two fifths of it)."""
    import torch
    from paper_2412_08059_amd import DeviceCSR, Solver
    a = _unequal(gen(), "all")
    dev = DeviceCSR.from_host(a)
    b = torch.ones(a.n, dtype=torch.float64, device="cuda")
    x = torch.empty_like(b)
    solvers = [Solver(a.n, a.nnz, spmv_variant=v, maxit1=1, maxit2=1) for v in (0, 1)]
    best = [np.inf, np.inf]
    for _ in range(20):
        for k, s in enumerate(solvers):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            s.solve(dev, b, 1e-4, 1e-10, x=x)
            best[k] = min(best[k], time.perf_counter() - t0)
    for s in solvers:
        s.close()
    print(f"  {name}: {1e3 * best[0]:.3f} ms, SELL-64 {1e3 * best[1]:.3f} ms", flush=True)
    assert best[0] <= 1.25 * best[1]


@pytest.mark.parametrize("links", [14, 15, 16, 40])
@pytest.mark.parametrize("n,hub", [(100, 50), (5000, 0), (5000, 2501), (70000, 69999)])
def test_one_long_row(n, hub, links):
    """A path with one vertex linked to `links` more, its row as long as eight
    distances allow (17 entries) or longer: SELL-64's bits."""
    import scipy.sparse as sp
    import torch
    from paper_2412_08059_amd import DeviceCSR, Solver
    far = [v for v in (np.arange(1, links + 1) * (n // (links + 2))).tolist() if abs(v - hub) > 1]
    i = np.concatenate([np.arange(n - 1), np.full(len(far), hub)])
    j = np.concatenate([np.arange(1, n), far])
    w = sp.coo_matrix((-np.random.default_rng(links).uniform(0.5, 1.0, len(i)), (i, j)), shape=(n, n)).tocsr()
    w = w + w.T
    m = (w + sp.diags(1e-2 - np.asarray(w.sum(axis=1)).ravel())).tocsr()
    m.sort_indices()
    a = W.CSR(n, m.indptr.astype(np.int64), m.indices.astype(np.int32), m.data, "hub")
    dev = DeviceCSR.from_host(a)
    b = torch.from_numpy(W.rhs(a, seed=5)[1]).cuda()
    got = []
    for variant in (0, 1):
        s = Solver(a.n, a.nnz, spmv_variant=variant, maxit1=50, maxit2=50, max_restarts=1)
        st, x, stats = s.solve(dev, b, 1e-4, 1e-9)
        got.append((st, stats.n1, stats.n2, stats.flags, x.cpu().numpy().view(np.int64)))
        s.close()
    assert got[0][:4] == got[1][:4] and np.array_equal(got[0][4], got[1][4])
