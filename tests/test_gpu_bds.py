"""Batched bands in diagonal storage against SELL-64: the same bits.

A symmetric band of few distances, all at most 31, with more than 4,096 rows is
kept as its main and upper diagonals.  A stored zero at distance 40 (and its
mirror) changes no sum but puts the matrix out of diagonal storage, so both
forms run the same arithmetic: solutions, counts and residuals agree bit for
bit at slice edges, with holes in the diagonals, and for what diagonal storage
must refuse (an unsymmetric value or pattern, too many distances, diagonals
that are mostly empty)."""

import numpy as np
import pytest
import scipy.sparse as sp

import workloads as W

pytestmark = pytest.mark.gpu


def _band(n, dists, seed, density=1.0):
    rng = np.random.default_rng(seed)
    a = sp.csr_matrix((n, n))
    for d in dists:
        v = rng.uniform(-1.0, -0.1, size=n - d)
        v[rng.uniform(size=n - d) >= density] = 0.0
        a = a + sp.diags([v, v], [d, -d], shape=(n, n))
    a = sp.csr_matrix(a)
    a.eliminate_zeros()
    s = np.asarray(np.abs(a).sum(axis=1)).ravel()
    return sp.csr_matrix(a + sp.diags(s + 0.02))


def _scaled(n, factor):
    a = _band(n, [1, 7], 3)
    a[n // 2, n // 2 + 1] *= factor
    return a


def _one_sided(n):
    a = _band(n, [1, 9], 4).tolil()
    a[n // 3, n // 3 + 9] = 0.0
    a = a.tocsr()
    a.eliminate_zeros()
    return a


def _with_far_zero(a):
    """The same matrix with a stored zero at (i, i + 40) and (i + 40, i)."""
    a = a.tocoo()
    i = a.shape[0] // 2
    rows, cols = np.append(a.row, [i, i + 40]), np.append(a.col, [i + 40, i])
    vals = np.append(a.data, [0.0, 0.0])
    order = np.lexsort((cols, rows))
    rp = np.zeros(a.shape[0] + 1, dtype=np.int32)
    rp[1:] = np.cumsum(np.bincount(rows, minlength=a.shape[0]))
    return W.CSR(a.shape[0], rp, cols[order].astype(np.int32), vals[order])


CASES = {
    "path_4097": lambda: _band(4097, [1], 1),
    "w8_4159": lambda: _band(4159, range(1, 9), 2),
    "w8_4160": lambda: _band(4160, range(1, 9), 2),
    "w8_4161": lambda: _band(4161, range(1, 9), 2),
    "far_31": lambda: _band(5003, [31], 3),
    "mixed_distances": lambda: _band(6400, [3, 17, 31], 4),
    "holes": lambda: _band(6401, [1, 2, 5, 30], 5, density=0.8),
    "nine_distances": lambda: _band(4500, range(1, 10), 6),
    "sparse_diagonals": lambda: _band(4500, [1, 4, 6], 7, density=0.3),
    "unsymmetric_value": lambda: _scaled(4800, 1.0 + 2.0 ** -50),
    "one_sided": lambda: _one_sided(4800),
}


@pytest.mark.parametrize("dot_acc", [0, 1])
@pytest.mark.parametrize("name", list(CASES))
def test_same_bits_as_sell(name, dot_acc):
    import torch
    from paper_2412_08059_amd import BatchSolver, DeviceCSR
    a = CASES[name]()
    a.sort_indices()
    n = a.shape[0]
    b = torch.from_numpy(np.random.default_rng(5).uniform(-1.0, 1.0, n)).cuda()
    out = []
    for m in (W.CSR.from_scipy(a), _with_far_zero(a)):
        A = DeviceCSR.from_host(m)
        systems = [(A, b, torch.full((n,), np.nan, dtype=torch.float64, device="cuda"), e, 1e-10)
                   for e in (-1.0, 1e-3)]
        eng = BatchSolver(4 * 64 * (-(-n // 64)), 4 * 32 * n, 2, dot_acc=dot_acc)
        ids = eng.submit(systems)
        got = eng.wait_all(ids)
        eng.close()
        out.append([((q.status, q.n1, q.n2, q.restarts, q.flags, q.relres_sp, q.relres_restart_true,
                      q.relres_final_true), x.cpu().numpy()) for q, x in (got[i] for i in ids)])
    for (cs, xs), (cz, xz) in zip(*out):
        assert cs == cz, name
        assert np.array_equal(xs.view(np.uint64), xz.view(np.uint64)), name
