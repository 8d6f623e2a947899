"""Order of the batch engine's launches, on the CPU.

The engine's host code (batch_engine.hip has no kernels) is compiled with the
host compiler against launch functions that only record what they are asked
for, and one pass of its BFS stream is driven from a prepared state copy."""

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

// the device's bfs_mode of every slot after the launches recorded so far
static int g_mode[1024];
static int g_rounds = 0;

extern "C" {
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void *, const void *, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
}

namespace mpcg {
namespace batch {
static void set(const BfsList &l, int mode)
{
    for (int k = 0; k < l.cnt; ++k) g_mode[l.sys[k]] = mode;
}
void launch_bfs_fast_start(hipStream_t, const BArena &, const BfsList &l) { set(l, kBfsRun); }
void launch_bfs_next_sweep(hipStream_t, const BArena &, const BfsList &l) { set(l, kBfsRun); }
void launch_bfs_finish(hipStream_t, const BArena &, const BfsList &l) { set(l, kBfsDone); }
void launch_bfs_start(hipStream_t, const BArena &, int32_t sys, int32_t) { g_mode[sys] = kBfsRun; }
void launch_bfs_cancel(hipStream_t, const BArena &, int32_t sys) { g_mode[sys] = kBfsNone; }
void launch_cancel(hipStream_t, const BArena &, int32_t) {}
void launch_bfs_round(hipStream_t, const BArena &, int32_t, int, int, int64_t, int) { ++g_rounds; }
void launch_band_masks(hipStream_t, const BArena &, const BfsList &) {}
void launch_bfs_band(hipStream_t, const BArena &, const BandList &) {}
}  // namespace batch
}  // namespace mpcg

// argv: slots, then per slot "feat cancel reached": the slot's transition, whether
// its cancel is pending, and how many of its 100 vertices the first sweep reached.
// The copy shows every slot's sweep ended.  Prints "bfs_mode feat" per slot.
int main(int argc, char **argv)
{
    const int n = std::atoi(argv[1]);
    Engine e;
    std::vector<BSys> copy(n);
    e.slots.resize(n);
    e.hi_sys = e.bmirror_n = n;
    e.bmirror = copy.data();
    for (int i = 0; i < n; ++i) {
        Slot &sl = e.slots[i];
        sl.used = sl.autoe = sl.fast = true;
        sl.adm = 2;
        sl.nslices = 2;
        sl.f.n = 100;
        sl.feat = std::atoi(argv[2 + 3 * i]);
        sl.want_bfs_cancel = std::atoi(argv[3 + 3 * i]) != 0;
        std::memset(&copy[i], 0, sizeof(BSys));
        copy[i].bfs_mode = sl.feat == 3 ? kBfsDone : sl.feat ? kBfsSwept : kBfsNone;
        copy[i].reached = std::atoi(argv[4 + 3 * i]);
        if (sl.feat == 0) sl.want_start = !sl.want_bfs_cancel;
        g_mode[i] = copy[i].bfs_mode;
    }
    if (!e.bfs_pump()) return 1;
    for (int i = 0; i < n; ++i) std::printf("%d %d\n", g_mode[i], e.slots[i].feat);
    return 0;
}
"""

NONE, RUN, DONE = 0, 1, 3


@pytest.fixture(scope="module")
def pump(tmp_path_factory):
    d = tmp_path_factory.mktemp("batch_order")
    src, exe = d / "harness.cpp", d / "harness"
    src.write_text(HARNESS)
    subprocess.check_call(
        ["g++", "-std=c++17", "-O1", "-w", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
         f"-I{ROOT}/include", f"-I{ROOT}/paper_2412_08059_amd/csrc", str(src), "-o", str(exe),
         "-Wl,--unresolved-symbols=ignore-all"])

    def run(slots):
        out = subprocess.check_output([str(exe), str(len(slots)), *[str(v) for s in slots for v in s]], text=True)
        return [tuple(int(v) for v in line.split()) for line in out.splitlines()]
    return run


@pytest.mark.parametrize("feat,reached", [(1, 0), (2, 100), (2, 40), (3, 100)])
def test_a_pending_cancel_is_the_last_word_on_its_slot(pump, feat, reached):
    """The copy shows a sweep ended (feat 1: the second one is next, 2: the
    result, or the components where vertices were not reached) and the slot's
    cancel is pending: after the pass its 2BFS is off on the device, and the
    host retires it from the copy behind the cancel (feat 5)."""
    assert pump([(feat, 1, reached)]) == [(NONE, 5)]


def test_cancels_among_many_transitions(pump):
    """More systems than one list holds, every third one cancelled."""
    slots = [(1 + i % 2 if i % 5 else 0, 1 if i % 3 == 0 and i % 5 else 0, 100) for i in range(630)]
    for (feat, cancel, _), (mode, after) in zip(slots, pump(slots)):
        if cancel:
            assert (mode, after) == (NONE, 5)
        else:
            assert (mode, after) == {0: (RUN, 1), 1: (RUN, 2), 2: (DONE, 3)}[feat]
