"""What the library reports of mpcg_spmv's time is its product's kernel.  Sizes
beyond every cache, so that a launch takes hundreds of microseconds and what
else lies between two events some per cent of them."""

import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _diagonal(n):
    import torch
    from paper_2412_08059_amd import DeviceCSR
    i = torch.arange(n + 1, dtype=torch.int32, device="cuda")
    return DeviceCSR(i, i[:n].clone(), torch.ones(n, dtype=torch.float64, device="cuda"), n)


def _tridiagonal(n):
    import torch
    from paper_2412_08059_amd import DeviceCSR
    i = torch.arange(n, dtype=torch.int64, device="cuda")
    col = i[:, None] + torch.tensor([-1, 0, 1], device="cuda")
    here = (col >= 0) & (col < n)
    val = torch.tensor([-1.0, 3.0, -1.0], dtype=torch.float64, device="cuda").expand(n, 3)
    rp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    rp[1:] = torch.cumsum(here.sum(1), 0)
    return DeviceCSR(rp.to(torch.int32), col[here].to(torch.int32), val[here].contiguous(), n)


def test_timing_hook_times_what_spmv_runs():
    """The product is most of a call: checks and product move 52 bytes a row of a
    tridiagonal matrix, the copy to y 16, the diagonals that a solve would use 32
    in FP64 -- less than three fifths of the call even without its launches."""
    import torch
    from paper_2412_08059_amd import Solver, capi
    a = _tridiagonal(16_000_000)
    x = torch.ones(a.n, dtype=torch.float64, device="cuda")
    s = Solver(a.n, a.nnz)
    call = np.inf
    for _ in range(6):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        st, _ = s.spmv(a, x, 64)
        call = min(call, 1e3 * (time.perf_counter() - t0))
        assert st == 0
    hook = min(capi.mpcg_time_kernel(s.ctx, a.desc, capi.MPCG_KERNEL_SPMV_F64, 10) for _ in range(3))
    s.close()
    print(f"  call {1e3 * call:.0f} us, hook {1e3 * hook:.0f} us", flush=True)
    assert 0.6 * call <= hook <= call


def test_last_kernel_is_the_product_alone():
    """On a diagonal matrix the product moves 32 bytes a row and the copy of the
    result to y 16: both together take half as much again as the product."""
    import torch
    from paper_2412_08059_amd import Solver, capi
    a = _diagonal(32_000_000)
    x = torch.ones(a.n, dtype=torch.float64, device="cuda")
    s = Solver(a.n, a.nnz)
    last = np.inf
    for _ in range(6):
        st, _ = s.spmv(a, x, 64)
        assert st == 0
        last = min(last, capi.mpcg_last_kernel_ms(s.ctx))
    hook = min(capi.mpcg_time_kernel(s.ctx, a.desc, capi.MPCG_KERNEL_SPMV_F64, 10) for _ in range(3))
    s.close()
    print(f"  last kernel {1e3 * last:.0f} us, hook {1e3 * hook:.0f} us", flush=True)
    assert last <= 1.2 * hook
