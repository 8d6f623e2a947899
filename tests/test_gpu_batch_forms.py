"""The batch step's two forms of a decision, at its blocks' heads and in a launch
of one block per system, give the same bits."""

import os

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

TEST_MODEL = os.path.join(os.path.dirname(__file__), "golden", "knn_model_test.txt")
# rows of the system beside which the others' decisions take a launch of their own
LARGE = 400_000


@pytest.fixture(scope="module")
def mats():
    import torch
    from paper_2412_08059_amd import DeviceCSR
    host = {"grid": W.poisson2d(150), "stencil": W.varcoef3d(27, seed=5), "band": W.banded(30_000, 8, seed=6),
            "graph": W.er_laplacian(9000, 8, seed=7), "large": W.banded(LARGE, 3, seed=8)}
    return {k: (DeviceCSR.from_host(a), torch.from_numpy(W.rhs(a, seed=9)[1]).cuda(), a.n) for k, a in host.items()}


@pytest.mark.parametrize("dot_acc", [0, 1])
@pytest.mark.parametrize("eps1", [1e-4, 0.0, -1.0])
def test_forms_give_the_same_bits(mats, eps1, dot_acc):
    import torch
    from paper_2412_08059_amd import BatchSolver
    names = ["grid", "stencil", "band", "graph"]

    def go(which):
        eng = BatchSolver(600_000, 8_000_000, 8, model=TEST_MODEL, dot_acc=dot_acc, maxit1=400, maxit2=400)
        try:
            xs = [torch.empty(mats[k][2], dtype=torch.float64, device="cuda") for k in which]
            ids = eng.submit([(mats[k][0], mats[k][1], x, eps1, 1e-9) for k, x in zip(which, xs)])
            got = eng.wait_all(ids, timeout_s=60)
        finally:
            eng.close()
        out = {}
        for k, rid, x in zip(which, ids, xs):
            s = got[rid][0]
            out[k] = ((s.status, s.n1, s.n2, s.restarts, s.flags, s.eps1_class, s.relres_sp, s.relres_restart_true,
                       s.relres_final_true, s.feat.pdiam, s.feat.v), x.cpu().numpy())
        return out
    alone = {k: go([k])[k] for k in names}      # decisions at the heads
    beside = go(["large"] + names)              # a launch per decision
    for k in names:
        assert alone[k][0] == beside[k][0], k
        assert np.array_equal(alone[k][1].view(np.int64), beside[k][1].view(np.int64)), k
