"""Steps of small systems in one workgroup each: the same bits as the step kernels.

While no listed system has more than 4,096 rows, each advances in a workgroup
of its own; beside a larger one all take the step kernels.  Both keep the same
state and add every sum in the same order, so a set of small systems gives the
same bits alone and beside a larger system, at the edges of rows per thread and
of slices, with rows longer than the registers hold, in every mode, and with
FP32 dot products."""

import os

import numpy as np
import pytest
import scipy.sparse as sp

import workloads as W
from workloads import paper_family as PF

pytestmark = pytest.mark.gpu
TEST_MODEL = os.path.join(os.path.dirname(__file__), "golden", "knn_model_test.txt")


def _indefinite():
    a = W.poisson2d(30).to_scipy().tolil()
    a[450, 450] = -3.0
    return W.CSR.from_scipy(a.tocsr())


def _star(n):
    a = sp.diags([1.0 + (np.arange(n) == 0) * n], [0], shape=(n, n)).tolil()
    a[0, 1:] = -0.5
    a[1:, 0] = -0.5
    return W.CSR.from_scipy(a.tocsr())


SETS = {
    "rows_1": [("n1", lambda: W.CSR.from_scipy(sp.csr_matrix(np.array([[3.0]])))),
               ("n63", lambda: W.path(63)), ("n64", lambda: W.banded(64, 8, seed=1)), ("n65", lambda: W.path(65)),
               ("n1023", lambda: W.banded(1023, 8, seed=2)), ("n1024", lambda: W.poisson2d(32)),
               ("star", lambda: _star(700)), ("tree", lambda: PF.random_sparse(1000, 3.0, 1.1, 7)),
               ("indefinite", _indefinite)],
    "rows_2": [("n1025", lambda: W.banded(1025, 3, seed=1)), ("n2048", lambda: W.banded(2048, 12, seed=2)),
               ("n300", lambda: W.er_laplacian(300, 20, seed=3)), ("n1600", lambda: W.er_laplacian(1600, 8, seed=5))],
    "rows_4": [("n2049", lambda: W.banded(2049, 8, seed=1)), ("n4096", lambda: W.poisson2d(64)),
               ("n3375", lambda: W.varcoef3d(15, seed=1)), ("n4000", lambda: W.er_laplacian(4000, 8, seed=5)),
               ("n100", lambda: W.path(100))],
}


def _solve(torch, small, beside, dot_acc, eps1s):
    from paper_2412_08059_amd import BatchSolver, DeviceCSR
    mats = [DeviceCSR.from_host(a) for a in small]
    gen = np.random.default_rng(11)
    systems, xs = [], []
    for A in mats:
        for e in eps1s:
            b = torch.from_numpy(gen.uniform(-1.0, 1.0, A.n)).cuda()
            xs.append(torch.full((A.n,), np.nan, dtype=torch.float64, device="cuda"))
            systems.append((A, b, xs[-1], e, 1e-10))
    if beside:
        L = DeviceCSR.from_host(W.banded(4161, 8, seed=9))
        systems.append((L, torch.from_numpy(gen.uniform(-1.0, 1.0, L.n)).cuda(),
                        torch.empty(L.n, dtype=torch.float64, device="cuda"), -1.0, 1e-12))
    rows = sum(64 * -(-A.n // 64) for A, *_ in systems)
    eng = BatchSolver(rows, 64 * rows + 64 * 700, len(systems), model=TEST_MODEL, dot_acc=dot_acc)
    ids = eng.submit(systems)
    got = eng.wait_all(ids)
    eng.close()
    out = []
    for k in range(len(xs)):
        q = got[ids[k]][0]
        out.append(((q.status, q.n1, q.n2, q.restarts, q.flags, q.eps1_class, q.relres_sp, q.relres_restart_true,
                     q.relres_final_true, q.feat.k0_used, q.feat.v, q.feat.pdiam), xs[k].cpu().numpy()))
    return out


@pytest.mark.parametrize("dot_acc", [0, 1])
@pytest.mark.parametrize("name", list(SETS))
def test_same_bits_beside_a_larger_system(name, dot_acc):
    import torch
    small = [make() for _, make in SETS[name]]
    eps1s = (-1.0, 1e-4, 0.0) if dot_acc == 0 else (-1.0, 1e-3)
    alone = _solve(torch, small, False, dot_acc, eps1s)
    mixed = _solve(torch, small, True, dot_acc, eps1s)
    for k, ((ca, xa), (cm, xm)) in enumerate(zip(alone, mixed)):
        label = (SETS[name][k // len(eps1s)][0], eps1s[k % len(eps1s)])
        assert ca == cm or (ca[0] != 0 and ca[:4] == cm[:4]), (label, ca, cm)
        assert np.array_equal(xa, xm, equal_nan=True), label
