"""The autotuner times its SELL-64 candidates on SELL-64, also for matrices that
a solve would keep as diagonals or iterate in one workgroup."""

import types

import pytest

at = pytest.importorskip("paper_2412_08059_amd.autotune")


@pytest.mark.parametrize("idx16", [0, 1])
def test_candidates_run_their_own_storage(monkeypatch, idx16):
    import paper_2412_08059_amd as P
    seen = []

    class FakeSolver:
        def __init__(self, n, nnz, *, tuning, spmv_variant=0):
            self.ctx = types.SimpleNamespace(variant=spmv_variant, tuning=None)

        def close(self):
            pass

    def time_kernel(ctx, desc, kernel, reps):
        seen.append((ctx.variant, ctx.tuning["sell_split"]))
        return 1.0 + 0.1 * ctx.tuning["sell_batch"] + 0.01 * ctx.tuning["sell_whole_batch"]

    monkeypatch.setattr(P, "Solver", FakeSolver)
    monkeypatch.setattr(P.capi, "mpcg_set_tuning", lambda ctx, t: setattr(ctx, "tuning", t))
    monkeypatch.setattr(P.capi, "mpcg_time_kernel", time_kernel)
    cands = at.sell_candidates(idx16)
    times = at._time_sell(cands, types.SimpleNamespace(n=10, nnz=10), types.SimpleNamespace(desc=None), 1)
    assert set(times) == set(cands)
    assert at.choose_min({c: times[c] for c in cands})[:2] == (4, 0)
    assert {v for v, _ in seen} == ({1} if idx16 else {1, 2})
    assert all((v == 2) == (split == 1) for v, split in seen)
