"""Which kernels a call runs: the tests that compare a path with another one bit
for bit hold as well when a rule refuses everything, so the rules are pinned
here, accepted and refused.  The calls run in a child process under torch's
profiler; the batch's diagonal storage shows in the systems' states instead."""

import json
import os
import re
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

pytestmark = pytest.mark.gpu


def _matrix(spec):
    import numpy as np
    import scipy.sparse as sp

    import workloads as W
    kind, *arg = spec.split(":")
    arg = [int(v) for v in arg]
    if kind == "grid":
        return W.poisson2d(arg[0])
    if kind == "cube":
        return W.varcoef3d(arg[0], seed=1)
    if kind == "band":
        return W.banded(arg[0], arg[1], seed=2)
    if kind == "graph":
        return W.er_laplacian(arg[0], arg[1], seed=3)
    if kind == "unequal":   # a grid with one unequal pair of values
        a = W.poisson2d(arg[0])
        a.val[1] = np.nextafter(a.val[1], 0.0)
        return a
    if kind == "thin":
        w, n = arg[0], arg[0] * arg[1]
        i = np.arange(n)
        r = np.concatenate([i[i % w != w - 1], i[:n - w]])
        c = np.concatenate([i[i % w != w - 1] + 1, i[:n - w] + w])
        m = sp.coo_matrix((-np.ones(len(r)), (r, c)), shape=(n, n))
        m = m + m.T
        return W.CSR.from_scipy((m + sp.diags(np.asarray(-m.sum(axis=1)).ravel() + 0.5)).tocsr())
    raise ValueError(spec)


# name: (call, matrix, options, kernels that run, kernels that do not)
CASES = {
    "grid": ("solve", "grid:100", {}, ["k_ds<0, double, 2, false", "k_ds<0, float, 2, false"], ["k_sell<", "k_wg_cg"]),
    "grid_sell": ("solve", "grid:100", {"spmv_variant": 1}, ["k_sell<0, double"], ["k_ds<", "k_ds_rows"]),
    "grid_csr": ("solve", "grid:100", {"spmv_variant": 3}, ["k_spmv<0, double"], ["k_ds<", "k_sell<"]),
    "cube_large": ("solve", "cube:85", {}, ["k_ds<0, double, 3, false, 2>"], ["k_sell<"]),
    "band_near": ("solve", "band:30000:8", {}, ["k_ds<0, double, 8, true"], ["k_sell<"]),
    "band_nine": ("solve", "band:30000:9", {}, ["k_sell<0, double"], ["k_ds<"]),
    "graph": ("solve", "graph:20000:8", {}, ["k_sell<"], ["k_ds<"]),
    "unequal": ("solve", "unequal:100", {}, ["k_sell<0, double"], ["k_ds<"]),
    "jacobi_pc": ("solve", "grid:40", {"precond": 1}, ["k_ds<0, double"], ["k_wg_cg"]),
    "jacobi": ("jacobi", "band:30000:8", {}, ["k_ds_jac<double", "k_ds_jac<float"], ["k_jac_sell"]),
    "jacobi_nine": ("jacobi", "band:30000:9", {}, ["k_jac_sell<double"], ["k_ds_jac"]),
    "small": ("solve", "grid:64", {}, ["k_wg_cg<double", "k_wg_cg<float"], ["k_ds<0", "k_cg_update"]),
    "small_graph": ("solve", "graph:1000:6", {}, ["k_wg_cg<double"], ["k_sell<0", "k_cg_update"]),
    "small_acc": ("solve", "grid:64", {"dot_acc": 1}, ["k_cg_update"], ["k_wg_cg"]),
    "small_sell": ("solve", "grid:64", {"spmv_variant": 1}, ["k_cg_update"], ["k_wg_cg"]),
    "small_over": ("solve", "band:4097:3", {}, ["k_cg_update"], ["k_wg_cg"]),
    "small_wide": ("solve", "band:3000:8", {}, ["k_cg_update"], ["k_wg_cg"]),
    "spmv": ("spmv", "grid:100", {}, ["k_spmv_checked<double>"], ["k_ds", "k_sell", "k_ingest"]),
    "spmv_sell": ("spmv", "grid:100", {"spmv_variant": 1}, ["k_sell<3, double"], ["k_spmv_checked"]),
    "bfs_segments": ("features", "band:7000:8", {}, ["k_seg_chain", "k_seg_fill"], ["k_bfs_small", "k_dia"]),
    "bfs_band_short": ("features", "band:6000:8", {}, ["k_bfs_small"], ["k_seg", "k_dia"]),
    "bfs_block": ("features", "grid:100", {}, ["k_dia_block"], ["k_bfs_small", "k_dia_offsets"]),
    "bfs_tiles": ("features", "grid:600", {}, ["k_dia_multi"], ["k_bfs_small", "k_dia_block"]),
    "bfs_thin": ("features", "thin:9:8000", {}, ["k_bfs_small"], ["k_dia", "k_seg"]),
    "bfs_graph": ("features", "graph:2000:16", {}, ["k_bfs_small"], ["k_dia", "k_seg"]),
    "batch_small": ("batch", "grid:64", {}, ["k_b_wg<"], ["k_b_product", "k_b_update"]),
    "batch_heavy": ("batch", "band:4000:30", {}, ["k_b_product", "k_b_update"], ["k_b_wg<", "k_b_decide"]),
    "batch": ("batch", "grid:100", {}, ["k_b_product", "k_b_update"], ["k_b_wg<", "k_b_decide"]),
    "batch_large": ("batch", "band:500000:2", {}, ["k_b_product", "k_b_decide", "k_b_close"], ["k_b_wg<"]),
}


def _child():
    """Runs every case under the profiler; prints {name: kernel names}."""
    import torch
    from torch.profiler import ProfilerActivity, profile

    from paper_2412_08059_amd import BatchSolver, DeviceCSR, Solver
    out = {}
    for name, (call, spec, opt, _, _) in CASES.items():
        a = _matrix(spec)
        dev = DeviceCSR.from_host(a)
        b = torch.ones(a.n, dtype=torch.float64, device="cuda")
        x = torch.empty_like(b)
        if call == "batch":
            s = BatchSolver(-(-a.n // 64) * 64, 2 * a.nnz + 64 * a.n, 1, maxit1=30, maxit2=30)
        else:
            s = Solver(a.n, a.nnz, maxit1=30, maxit2=30, max_restarts=0, **opt)
        with profile(activities=[ProfilerActivity.CUDA]) as p:
            if call == "solve":
                s.solve(dev, b, 1e-4, 1e-9, x=x)
            elif call == "jacobi":
                s.solve_jacobi(dev, b, 1e-4, 1e-9, x=x)
            elif call == "spmv":
                s.spmv(dev, b, 64)
            elif call == "features":
                s.features(dev, b)
            else:
                s.wait_all(s.submit([(dev, b, x, 1e-4, 1e-9)]))
            torch.cuda.synchronize()
        s.close()
        out[name] = sorted({re.sub(r"\(.*", "", e.name).replace("void ", "") for e in p.events() if "k_" in e.name})
        print("#", name, flush=True)
    print(json.dumps(out), flush=True)


@pytest.fixture(scope="module")
def kernels():
    import torch
    torch.cuda.synchronize()
    r = subprocess.run([sys.executable, "-u", os.path.abspath(__file__)], cwd=ROOT, stdout=subprocess.PIPE,
                       stderr=subprocess.STDOUT, text=True, timeout=100)
    assert r.returncode == 0, r.stdout[-2000:]
    return json.loads([line for line in r.stdout.splitlines() if line.startswith("{")][-1])


@pytest.mark.parametrize("name", sorted(CASES))
def test_kernels_of_the_call(kernels, name):
    _, _, _, run, not_run = CASES[name]
    names = kernels[name]
    for k in run:
        assert any(k in n for n in names), (k, names)
    for k in not_run:
        assert not any(k in n for n in names), (k, names)


@pytest.mark.parametrize("spec,distances", [
    ("band:30000:8", 8), ("band:30000:3", 3), ("thin:9:1000", 2), ("thin:31:300", 2), ("thin:32:300", 0), ("band:30000:9", 0),
    ("graph:9000:8", 0), ("band:3000:8", 0),   # small systems keep SELL-64
])
def test_batch_diagonal_storage(tmp_path, spec, distances):
    """BSys::ds of the system, left in its slot."""
    import torch

    from paper_2412_08059_amd import BatchSolver, DeviceCSR
    src, exe = tmp_path / "at.cpp", tmp_path / "at"
    src.write_text('#include "batch_internal.hpp"\n#include <cstddef>\n#include <cstdio>\n'
                   'int main() { std::printf("%zu\\n", offsetof(mpcg::batch::BSys, ds)); return 0; }\n')
    subprocess.check_call(["g++", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", f"-I{ROOT}/include",
                           f"-I{ROOT}/paper_2412_08059_amd/csrc", str(src), "-o", str(exe)])
    at = int(subprocess.check_output([str(exe)], text=True))
    a = _matrix(spec)
    dev = DeviceCSR.from_host(a)
    b = torch.ones(a.n, dtype=torch.float64, device="cuda")
    x = torch.empty_like(b)
    eng = BatchSolver(-(-a.n // 64) * 64, 2 * a.nnz + 64 * a.n, 1, maxit1=10, maxit2=10)
    eng.wait_all(eng.submit([(dev, b, x, 1e-4, 1e-9)]))
    eng.close()
    torch.cuda.synchronize()
    assert int(eng.arena[at:at + 4].cpu().view(torch.int32)[0]) == distances


if __name__ == "__main__":
    _child()
