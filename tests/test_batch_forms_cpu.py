"""Which form of the step the batch engine launches for a list of systems: its
host code, compiled for the host, against launch functions that only record."""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HARNESS = r"""
#include "batch_engine.hip"

#include <cstdio>
#include <cstdlib>

using namespace mpcg;
using namespace mpcg::batch;

static int g_form = -1;   // 0: a launch per decision, 1: decisions at the blocks' heads, 2: a workgroup per system

extern "C" hipError_t hipGetLastError() { return hipSuccess; }

namespace mpcg {
namespace batch {
void launch_worklist(hipStream_t, const BArena &, const ListChunk &) {}
void launch_steps(hipStream_t, const BArena &, int32_t, int32_t, int32_t, bool, bool heads) { g_form = heads; }
void launch_wg_steps(hipStream_t, const BArena &, int32_t, int32_t, int32_t) { g_form = 2; }
}  // namespace batch
}  // namespace mpcg

// argv: rows of each listed system and entries of its longest row; prints the form
int main(int argc, char **argv)
{
    Engine e;
    e.graphs_ok = false;
    e.slots.resize((argc - 1) / 2);
    for (int i = 0; 2 * i + 1 < argc; ++i) {
        Slot &sl = e.slots[i];
        sl.used = true;
        sl.adm = 2;
        sl.nslices = (std::atoi(argv[1 + 2 * i]) + 63) / 64;
        sl.padded = (int64_t)sl.nslices * 64 * std::atoi(argv[2 + 2 * i]);
    }
    if (!e.rebuild_list() || !e.launch_group(8)) return 1;
    std::printf("%d\n", g_form);
    return 0;
}
"""


@pytest.fixture(scope="module")
def form(tmp_path_factory):
    d = tmp_path_factory.mktemp("batch_forms")
    src, exe = d / "harness.cpp", d / "harness"
    src.write_text(HARNESS)
    subprocess.check_call(
        ["g++", "-std=c++17", "-O1", "-w", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
         f"-I{ROOT}/include", f"-I{ROOT}/paper_2412_08059_amd/csrc", str(src), "-o", str(exe),
         "-Wl,--unresolved-symbols=ignore-all"])
    return lambda rows, width=17: int(subprocess.check_output(
        [str(exe), *[v for n in rows for v in (str(n), str(width))]], text=True))


@pytest.mark.parametrize("rows,want", [
    ([100_000], 1), ([5000] * 64, 1), ([300_000], 1), ([1000] * 512 + [5000], 1),
    ([500_000], 0), ([1_000_000], 0), ([4_000_000], 0), ([100_000] * 96, 0), ([1000] * 8 + [4_000_000], 0),
])
def test_partials_are_added_in_linear_cost(form, rows, want):
    """Every block adds all of its system's partials only while that is a few
    megabytes of reads a launch; a launch of one block per system otherwise."""
    assert form(rows) == want


@pytest.mark.parametrize("rows,width,want", [
    ([1000], 7, 2), ([1000] * 512, 30, 2), ([4096], 17, 2), ([4096] * 64, 33, 2), ([2000] * 8, 100, 2), ([1000], 300, 2),
    ([4096], 33, 1), ([4096], 400, 1), ([4096] * 64, 101, 1), ([2000], 151, 1), ([3000] * 8, 51, 1), ([1000], 900, 1),
    ([1000] * 8 + [4097], 7, 1),
])
def test_a_workgroup_takes_what_it_reads_in_time(form, rows, width, want):
    assert form(rows, width) == want
