"""Cancelled Algorithm II systems whose 2BFS runs on the level kernels: what is
cancelled between its sweeps must not go on in a slot that serves another
system by then."""

import os
import time

import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

TEST_MODEL = os.path.join(os.path.dirname(__file__), "golden", "knn_model_test.txt")
# connected, |i - j| > 31: no band sweeps
GRAPHS = [lambda: W.poisson2d(60), lambda: W.er_laplacian(2000, 8, seed=3), lambda: W.varcoef3d(14, seed=4),
          lambda: W.poisson2d(130)]


@pytest.mark.parametrize("delay_ms", [0.0, 0.3, 0.6, 1.0, 1.5, 2.5, 4.0])
def test_cancel_between_sweeps(delay_ms):
    """Eight slots, 24 systems; every other one is cancelled after delay_ms.  The
    others' status, solution check and graph features are the oracle's."""
    import torch
    from paper_2412_08059_amd import BatchSolver, DeviceCSR, capi
    mats = [g() for g in GRAPHS]
    want = [oracle.pseudo_diameter(a) for a in mats]
    eng = BatchSolver(200_000, 2_000_000, 8, model=TEST_MODEL)
    try:
        dev = [DeviceCSR.from_host(a) for a in mats]
        rhs = [torch.from_numpy(W.rhs(a, seed=11)[1]).cuda() for a in mats]
        systems = []
        for k in range(24):
            x = torch.empty(mats[k % 4].n, dtype=torch.float64, device="cuda")
            systems.append((dev[k % 4], rhs[k % 4], x, 0.0, 1e-10))
        ids = eng.submit(systems)
        time.sleep(delay_ms * 1e-3)
        # by graph and by turn, so that each graph is cancelled and kept
        dropped = {rid for k, rid in enumerate(ids) if (k // 4 + k) % 2 == 0}
        for rid in dropped:
            assert eng.cancel(rid) in (0, capi.MPCG_EINVAL)   # EINVAL: already reported
        got = eng.wait_all(ids, timeout_s=60)
    finally:
        eng.close()
    print(f"  delay {delay_ms} ms: {sum(got[r][0].status == capi.MPCG_ECANCELED for r in dropped)} of {len(dropped)} "
          "cancelled", flush=True)
    for k, rid in enumerate(ids):
        st = got[rid][0]
        if rid in dropped and st.status == capi.MPCG_ECANCELED:
            continue
        assert st.status == 0
        assert st.relres_final_true <= 1e-10
        f = st.feat
        assert (f.pdiam, f.bfs_t, f.bfs_u, f.n_components) == want[k % 4]
