"""CG in one workgroup against the two-launch path: the same bits.

Small systems iterate in one workgroup (spmv_variant 0); an explicit variant
keeps the two launches per iteration.  Both add every sum in the same order, so
solutions, iteration counts, flags and Algorithm II's choice agree bit for bit,
wherever a launch ends (graph_iters), at every instance's edges of rows and row
lengths, and when a phase stops at its cap or breaks down."""

import os

import numpy as np
import pytest
import scipy.sparse as sp

import workloads as W
from workloads import paper_family as PF

pytestmark = pytest.mark.gpu
TEST_MODEL = os.path.join(os.path.dirname(__file__), "golden", "knn_model_test.txt")


def _regular(n, deg, seed):
    """Random symmetric pattern, every row of at most deg + 1 entries, one of exactly that."""
    rng = np.random.default_rng(seed)
    have = [set() for _ in range(n)]
    for _ in range(4 * n * deg):
        i, j = rng.integers(0, n, 2)
        if i != j and len(have[i]) < deg and len(have[j]) < deg and j not in have[i]:
            have[i].add(int(j))
            have[int(j)].add(int(i))
    ei = [(i, j) for i in range(n) for j in have[i] if i < j]
    v = rng.uniform(0.1, 1.0, len(ei))
    i, j = np.array(ei).T
    a = sp.coo_matrix((-v, (i, j)), shape=(n, n)).tocsr()
    a = a + a.T
    return W.CSR.from_scipy(a + sp.diags(np.asarray(abs(a).sum(axis=1)).ravel() + 0.05))


def _indefinite(n):
    a = W.poisson2d(int(n ** 0.5)).to_scipy().tolil()
    a[n // 2, n // 2] = -3.0
    return W.CSR.from_scipy(a.tocsr())


CASES = {
    "n1": lambda: W.CSR.from_scipy(sp.csr_matrix(np.array([[3.0]]))),
    "n255": lambda: W.path(255),
    "n257": lambda: W.path(257),
    "n1024": lambda: W.poisson2d(32),
    "n1025": lambda: W.banded(1025, 3, seed=1),
    "n2047_w8": lambda: W.banded(2047, 8, seed=2),
    "n2048_w8": lambda: W.banded(2048, 8, seed=2),
    "n2049_w3": lambda: W.banded(2049, 3, seed=3),
    "n4095": lambda: W.banded(4095, 2, seed=4),
    "n4096": lambda: W.poisson2d(64),
    "n4097": lambda: W.banded(4097, 2, seed=4),                 # one row too many
    "row7": lambda: W.varcoef3d(14, seed=1),
    "row8_4000": lambda: _regular(4000, 7, 1),                  # a row too long for four rows a thread
    "row17": lambda: _regular(1500, 16, 2),
    "row32": lambda: _regular(900, 31, 3),
    "row33": lambda: _regular(900, 32, 4),                      # a row too long
    "tree": lambda: PF.random_sparse(1000, 3.0, 1.1, 7),
    "er": lambda: W.er_laplacian(1000, 10, seed=5),
}


def _solve(a, B, eps1, variant, **kw):
    from paper_2412_08059_amd import DeviceCSR, Solver
    s = Solver(a.n, a.nnz, spmv_variant=variant, model=TEST_MODEL, **kw)
    st, x, q = s.solve(DeviceCSR.from_host(a), B, eps1, 1e-10)
    s.close()
    counts = (st, q.n1, q.n2, q.restarts, q.flags & ~16, q.eps1_class, q.feat.k0_used, q.feat.v, q.relres_sp,
              q.relres_restart_true, q.relres_final_true)
    return counts, x


@pytest.mark.parametrize("name", list(CASES))
def test_same_bits_as_two_launches(name):
    import torch
    a = CASES[name]()
    _, b = W.rhs(a, seed=3)
    B = torch.from_numpy(b).cuda()
    for eps1, kw in ((1e-3, {}), (0.0, {}), (-1.0, {}), (1e-6, {"maxit1": 7, "maxit2": 33}), (1e-2, {"tol_mode": 1})):
        want, xw = _solve(a, B, eps1, 1, **kw)
        for g in (0, 1, 5):
            got, x = _solve(a, B, eps1, 0, graph_iters=g, **kw)
            assert got == want, (name, eps1, kw, g)
            assert torch.equal(x.view(torch.int64), xw.view(torch.int64)), (name, eps1, kw, g)


def test_breakdown_and_zero_rhs():
    import torch
    a = _indefinite(1024)
    _, b = W.rhs(a, seed=5)
    B = torch.from_numpy(b).cuda()
    for eps1 in (1e-4, -1.0, 0.0):
        want, xw = _solve(a, B, eps1, 1)
        got, x = _solve(a, B, eps1, 0)
        assert got == want and want[0] == -2
        assert torch.equal(x.view(torch.int64), xw.view(torch.int64))
    z = W.poisson2d(20)
    got, x = _solve(z, torch.zeros(z.n, dtype=torch.float64, device="cuda"), 1e-4, 0)
    assert got[0] == 0 and float(x.abs().max()) == 0.0
