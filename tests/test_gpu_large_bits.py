"""Bits of solves large enough for several slices a wave (above 524,288 rows)."""

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _dev(a, seed):
    import torch
    from paper_2412_08059_amd import DeviceCSR
    return DeviceCSR.from_host(a), torch.from_numpy(W.rhs(a, seed=seed)[1]).cuda()


@pytest.mark.parametrize("name,gen", [("cube", lambda: W.varcoef3d(85, seed=1)), ("grid", lambda: W.poisson2d(757)),
                                      ("band", lambda: W.banded(540_001, 8, seed=2))])
def test_diagonals_and_sell_agree(name, gen):
    """Far and near distances, three, two and eight of them; the last waves have
    fewer slices than the others."""
    from paper_2412_08059_amd import Solver
    a = gen()
    dev, b = _dev(a, 3)
    got = []
    for variant in (0, 1):
        s = Solver(a.n, a.nnz, spmv_variant=variant, maxit1=40, maxit2=40, max_restarts=0)
        st, x, S = s.solve(dev, b, 1e-3, 1e-12)
        got.append((st, S.n1, S.n2, S.relres_sp, S.relres_restart_true, S.relres_final_true, x.cpu().numpy().view(np.int64)))
        s.close()
    assert got[0][:6] == got[1][:6]
    assert np.array_equal(got[0][6], got[1][6])


def test_bits_do_not_depend_on_when_the_2bfs_ends():
    """Algorithm II on a band of 600,000 rows with its 2BFS by segments (2 ms) and
    level by level on bits (0.8 s, longer than the whole solve): the same chosen
    class, counts and bits."""
    from paper_2412_08059_amd import DEFAULT_MODEL, Solver
    a = W.banded(600_000, 8, seed=5)
    dev, b = _dev(a, 6)
    got = []
    for tuning in ({}, {"bfs_dia": 2, "bfs_dia_tiles": 0}, {"bfs_dia": 2}, {"bfs_grid_shared": 8}, {}):
        s = Solver(a.n, a.nnz, model=DEFAULT_MODEL)
        if tuning:
            s.set_tuning({**s.tuning_for(a.n, a.nnz, 8), **tuning})
        st, x, S = s.solve(dev, b, 0.0, 1e-10)
        print(f"  {tuning}: n1={S.n1} n2={S.n2} class={S.eps1_class} t_feat={S.t_feat_ms:.1f} ms", flush=True)
        got.append((st, S.n1, S.n2, S.eps1_class, S.feat.pdiam, S.feat.v, x.cpu().numpy().view(np.int64)))
        s.close()
    assert got[0][0] == 0
    for g in got[1:]:
        assert g[:6] == got[0][:6]
        assert np.array_equal(g[6], got[0][6])
