"""Diagonal storage against the SELL-64 kernels: the same bits.

spmv_variant 0 stores a symmetric matrix on few diagonals as its main and
upper diagonals; spmv_variant 1 keeps SELL-64.  Both run each row's fma chain
in CSR order and leave the same partial sums, so products, solves (with their
iteration counts) and Jacobi iterations agree bit for bit -- at slice edges,
for distances beyond the matrix's ends, with holes in the diagonals, and for
what diagonal storage must refuse (unsymmetric values or pattern, a diagonal
that few rows have, too many of them)."""

import numpy as np
import pytest
import scipy.sparse as sp

import workloads as W
from workloads import paper_family as PF

pytestmark = pytest.mark.gpu


def _band(n, dists, seed, density=1.0):
    """Symmetric, diagonally dominant, entries at the given distances."""
    rng = np.random.default_rng(seed)
    a = sp.lil_matrix((n, n)).tocsr()
    for d in dists:
        if d >= n:
            continue
        v = rng.uniform(-1.0, -0.1, size=n - d)
        v[rng.uniform(size=n - d) >= density] = 0.0
        a = a + sp.diags([v, v], [d, -d], shape=(n, n))
    a = sp.csr_matrix(a)
    s = np.asarray(np.abs(a).sum(axis=1)).ravel()
    return W.CSR.from_scipy(a + sp.diags(s + 0.5))


def _unsymmetric(n):
    a = _band(n, [1, 7], 3).to_scipy().tolil()
    a[n // 2, n // 2 + 1] *= 1.0 + 2.0 ** -50
    return W.CSR.from_scipy(a.tocsr())


def _one_sided(n):
    a = _band(n, [1, 9], 4).to_scipy().tolil()
    a[n // 3, n // 3 + 9] = 0.0
    return W.CSR.from_scipy(a.tocsr())


def _rare_diagonal(n):
    a = _band(n, [1, 2], 5).to_scipy().tolil()
    i = n // 2 + 1
    a[i, i + 31] = a[i + 31, i] = -0.25
    return W.CSR.from_scipy(a.tocsr())


CASES = [
    ("n1", lambda: W.CSR.from_scipy(sp.csr_matrix(np.array([[3.0]])))),
    ("path_2", lambda: _band(2, [1], 0)),
    ("path_63", lambda: _band(63, [1], 1)),
    ("path_64", lambda: _band(64, [1], 1)),
    ("path_129", lambda: _band(129, [1], 2)),
    ("near_32", lambda: _band(1000, [1, 32], 3)),
    ("far_33", lambda: _band(1000, [1, 33], 3)),
    ("reach_n", lambda: _band(300, [1, 150, 299], 4)),
    ("four", lambda: _band(777, [1, 2, 5, 11], 5)),
    ("five", lambda: _band(777, [1, 2, 5, 11, 100], 6)),
    ("six", lambda: _band(2000, [1, 2, 3, 4, 5, 6], 7)),
    ("seven_far", lambda: _band(2000, [1, 2, 3, 4, 5, 6, 700], 8)),
    ("band8", lambda: W.banded(5003, 8, seed=1)),
    ("band8_far", lambda: _band(3001, [1, 2, 3, 4, 5, 6, 7, 500], 9)),
    ("band9", lambda: W.banded(3000, 9, seed=2)),                     # too many distances
    ("holes", lambda: PF.random_banded(4099, 17, 0.8, 3.0, 5)),
    ("sparse_holes", lambda: _band(3000, [1, 5, 9], 10, density=0.3)),  # below the two-thirds rule
    ("lap2d", lambda: W.poisson2d(67)),
    ("lap3d", lambda: W.varcoef3d(17, seed=3)),
    ("band_600k", lambda: W.banded(600_001, 3, seed=4)),              # several slice groups per block
    ("star", lambda: W.star(3000)),                                   # a row of several chunks
    ("unsymmetric", lambda: _unsymmetric(1500)),
    ("one_sided", lambda: _one_sided(1500)),
    ("rare_diagonal", lambda: _rare_diagonal(40_000)),
]


@pytest.fixture(scope="module")
def matrices():
    return {name: gen() for name, gen in CASES}


@pytest.mark.parametrize("name", [c[0] for c in CASES])
def test_same_bits_as_sell(matrices, name):
    import torch
    from paper_2412_08059_amd import MPCG_EPS1_NONE, DeviceCSR, Solver
    a = matrices[name]
    xs, b = W.rhs(a, seed=11)
    A = DeviceCSR.from_host(a)
    A64 = DeviceCSR.from_host(a, row_ptr_i64=True)
    B = torch.from_numpy(b).cuda()
    V = torch.from_numpy(xs).cuda()
    spd = name not in ("unsymmetric", "one_sided")
    # (eps1, precond, dot_acc); an unsymmetric system may not converge: cap it
    runs = [(1e-3, 0, 0), (1e-5, 1, 0), (1e-3, 0, 1), (MPCG_EPS1_NONE, 0, 0)]
    for eps1, pc, acc in runs:
        got = []
        for variant, mat in ((0, A), (1, A), (0, A64)):
            s = Solver(a.n, a.nnz, precond=pc, dot_acc=acc, spmv_variant=variant, maxit1=60, maxit2=60,
                       max_restarts=1)
            st, x, stats = s.solve(mat, B, eps1, 1e-8)
            y = [s.spmv(mat, V, 64)[1], s.spmv(mat, V.float(), 32)[1]]
            js, jx, jstats = s.solve_jacobi(mat, B, eps1 if eps1 > 0 else MPCG_EPS1_NONE, 1e-8)
            got.append((st, stats.n1, stats.n2, stats.flags, js, jstats.n1, jstats.n2, x.clone(), jx.clone(), *y))
            s.close()
        for other in got[1:]:
            assert got[0][:7] == other[:7], (name, eps1, pc, acc)
            for u, v in zip(got[0][7:], other[7:]):
                assert torch.equal(u.view(torch.uint8), v.view(torch.uint8)), (name, eps1, pc, acc)
    if spd:
        ref = torch.from_numpy(a.to_scipy() @ xs)
        assert float((got[0][9].cpu() - ref).norm()) <= 1e-12 * float(ref.norm())


@pytest.mark.parametrize("lower", [False, True])
@pytest.mark.parametrize("row", [0, 31, 63, 64, 100, 128, 1000 - 33])
def test_unsymmetric_value_is_seen_across_slices(row, lower):
    """One changed value of a pair whose rows lie in one slice or in two."""
    import torch
    from paper_2412_08059_amd import MPCG_EPS1_NONE, DeviceCSR, Solver
    a = _band(1000, [1, 32], 13).to_scipy().tolil()
    i, j = (row + 32, row) if lower else (row, row + 32)
    a[i, j] *= 1.5
    m = W.CSR.from_scipy(a.tocsr())
    A, B = DeviceCSR.from_host(m), torch.linspace(-1.0, 1.0, m.n, dtype=torch.float64, device="cuda")
    x = []
    for variant in (0, 1):
        s = Solver(m.n, m.nnz, spmv_variant=variant, precond=1, maxit1=40, maxit2=40, max_restarts=0)
        x.append(s.solve(A, B, MPCG_EPS1_NONE, 1e-8)[1].clone())
        s.close()
    assert torch.equal(x[0].view(torch.uint8), x[1].view(torch.uint8))


@pytest.mark.parametrize("bad", ["column", "order", "nan", "inf_b"])
def test_malformed_entries_are_reported(bad):
    """Found by the diagonal pass or not, an error is the general pass's."""
    import torch
    from paper_2412_08059_amd import DeviceCSR, Solver
    a = _band(5000, [1, 4], 12)
    col, val, b = a.col.copy(), a.val.copy(), np.ones(a.n)
    k = int(a.row_ptr[2501])
    if bad == "column":
        col[int(a.row_ptr[2502]) - 1] = a.n + 3
    elif bad == "order":
        col[k], col[k + 1] = col[k + 1], col[k]
    elif bad == "nan":
        val[k] = np.nan
    else:
        b[17] = np.inf
    A = DeviceCSR.from_host(W.CSR(a.n, a.row_ptr, col, val))
    want = -1 if bad in ("column", "order") else -6
    for variant in (0, 1):
        s = Solver(a.n, a.nnz, spmv_variant=variant)
        st, _, _ = s.solve(A, torch.from_numpy(b).cuda(), 1e-3, 1e-8)
        assert st == want, (bad, variant, st)
        for prec, dt in ((64, torch.float64), (32, torch.float32)):
            st, _ = s.spmv(A, torch.ones(a.n, dtype=dt, device="cuda"), prec)
            assert st == (want if bad != "inf_b" else 0), (bad, variant, prec, st)
        s.close()
    if bad == "column":   # row pointers: nothing is read through them, y stays as it was
        from paper_2412_08059_amd import capi
        rp = a.row_ptr.copy()
        rp[2000] = a.nnz + 10_000_000
        bad_a = DeviceCSR.from_host(W.CSR(a.n, rp, a.col, a.val))
        s = Solver(a.n, a.nnz)
        x = torch.ones(a.n, dtype=torch.float64, device="cuda")
        y = torch.full_like(x, 7.0)
        assert capi.mpcg_spmv(s.ctx, bad_a.desc, 64, x.data_ptr(), y.data_ptr()) == -1
        assert bool((y == 7.0).all())
        s.close()
