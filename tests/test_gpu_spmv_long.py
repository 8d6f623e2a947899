"""mpcg_spmv on long rows: the oracle's bits and the checks' verdicts where the
product changes from chunks of entries to a lane per row, and its time."""

import time

import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


def _rows(lens, n, seed=0):
    """CSR with the given row lengths, columns drawn without repetition."""
    assert len(lens) == n
    rng = np.random.default_rng(seed)
    col = np.concatenate([np.sort(rng.choice(n, size=k, replace=False)) for k in lens])
    rp = np.concatenate([[0], np.cumsum(lens)])
    return W.CSR(n, rp.astype(np.int64), col.astype(np.int32), rng.uniform(-1.0, 1.0, len(col)), "rows")


def _lens(n, most, per_slice):
    """Rows of every slice: one of `most` entries, the others sharing the rest of per_slice."""
    out = np.full(n, (per_slice - most) // 63, dtype=np.int64)
    out[::64] = most
    return out


CASES = {
    "all_47": lambda: _rows([47] * 500, 500), "all_48": lambda: _rows([48] * 500, 500), "all_49": lambda: _rows([49] * 513, 513, 1),
    "all_200": lambda: _rows([200] * 300, 300, 2), "one_row": lambda: _rows([60] + [0] * 59, 60, 3),
    "ragged_65": lambda: _rows([60 + i % 9 for i in range(65)] + [0] * 35, 100, 4),
    "empty_between": lambda: _rows([90 if i % 3 else 0 for i in range(1000)], 1000, 5),
    "few_long": lambda: _rows(_lens(640, 300, 300 * 8 - 64), 640, 6), "enough_long": lambda: _rows(_lens(640, 300, 300 * 8 + 64), 640, 7),
    "slices_1024": lambda: _rows([50] * 65536, 65536, 8), "slices_1025": lambda: _rows([50] * 65537, 65537, 9),
    "dense_700": lambda: _rows([700] * 700, 700, 10),
}


@pytest.mark.parametrize("prec", [64, 32])
@pytest.mark.parametrize("name", sorted(CASES))
def test_bits(name, prec):
    import torch
    from paper_2412_08059_amd import DeviceCSR, Solver
    a = CASES[name]()
    x = np.random.default_rng(3).uniform(-1.0, 1.0, a.n)
    if prec == 32:
        x = x.astype(np.float32)
    want = oracle.spmv64(a, x) if prec == 64 else oracle.spmv32(a, x)
    s = Solver(a.n, a.nnz)
    for i64 in (False, True):
        st, y = s.spmv(DeviceCSR.from_host(a, row_ptr_i64=i64), torch.from_numpy(x).cuda(), prec)
        assert st == 0
        assert np.array_equal(y.cpu().numpy(), want)
    s.close()


@pytest.mark.parametrize("where", [0, 77, 13_000, 29_999])
@pytest.mark.parametrize("fault", ["column", "negative", "order", "repeat", "nan", "inf"])
def test_faults_in_long_rows(fault, where):
    import torch
    from paper_2412_08059_amd import DeviceCSR, Solver, capi
    a = _rows([60] * 500, 500, 11)
    k = where - where % 60 + min(where % 60, 58)   # not a row's last entry
    if fault == "column":
        a.col[k] = a.n
    elif fault == "negative":
        a.col[k] = -1
    elif fault == "order":
        a.col[[k, k + 1]] = a.col[[k + 1, k]]
    elif fault == "repeat":
        a.col[k + 1] = a.col[k]
    else:
        a.val[k] = float(fault)
    s = Solver(a.n, a.nnz)
    y = torch.full((a.n,), 7.0, dtype=torch.float64, device="cuda")
    x = torch.ones(a.n, dtype=torch.float64, device="cuda")
    st = capi.mpcg_spmv(s.ctx, DeviceCSR.from_host(a).desc, 64, x.data_ptr(), y.data_ptr())
    assert st == (capi.MPCG_ENONFINITE if fault in ("nan", "inf") else capi.MPCG_EINVAL)
    assert bool((y == 7.0).all())
    s.close()


@pytest.mark.parametrize("n,k", [(2000, 150), (1000, 600), (20000, 300)])
def test_no_slower_than_through_a_copy(n, k):
    """Least of 20 calls: at most a tenth more than with SELL-64 asked for, which
    checks, copies and then multiplies."""
    import torch
    from paper_2412_08059_amd import DeviceCSR, Solver
    rng = np.random.default_rng(12)
    start = rng.integers(0, n - k + 1, size=(n, 1))
    col = start + np.arange(k)   # k consecutive columns
    a = W.CSR(n, np.arange(n + 1, dtype=np.int64) * k, col.astype(np.int32).ravel(), rng.uniform(size=n * k), "rows")
    dev, x = DeviceCSR.from_host(a), torch.ones(n, dtype=torch.float64, device="cuda")
    solvers = [Solver(a.n, a.nnz, spmv_variant=v) for v in (0, 1)]
    best = [np.inf, np.inf]
    for _ in range(20):
        for i, s in enumerate(solvers):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            st, _ = s.spmv(dev, x, 64)
            best[i] = min(best[i], time.perf_counter() - t0)
            assert st == 0
    for s in solvers:
        s.close()
    print(f"  {n} rows of {k}: {1e6 * best[0]:.0f} us, SELL-64 {1e6 * best[1]:.0f} us", flush=True)
    assert best[0] <= 1.1 * best[1]
