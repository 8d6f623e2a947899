"""The step of the kernels' walks over a row range's entries, at the largest
entry indices (nnz up to 2^31 - 1), compiled for the host."""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HARNESS = r"""
#include "mpcg_internal.hpp"
#include <cstdio>
#include <cstdlib>
// argv: first and last + 1 entry, chunk length; prints every chunk as "at len"
int main(int, char **argv)
{
    const int b = std::atoi(argv[1]), e = std::atoi(argv[2]), most = std::atoi(argv[3]);
    int chunks = 0;
    for (int at = b, cn; (cn = mpcg::chunk_len(at, e, most)) > 0; at += cn) {
        std::printf("%d %d\n", at, cn);
        if (++chunks > 100) return 1;
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    d = tmp_path_factory.mktemp("entry_walk")
    src, exe = d / "walk.cpp", d / "walk"
    src.write_text(HARNESS)
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-ftrapv", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           f"-I{ROOT}/include", f"-I{ROOT}/paper_2412_08059_amd/csrc", str(src), "-o", str(exe)])

    def run(b, e, most):
        out = subprocess.check_output([str(exe), str(b), str(e), str(most)], text=True)
        return [tuple(int(v) for v in line.split()) for line in out.splitlines()]
    return run


@pytest.mark.parametrize("most", [16, 64, 320])
@pytest.mark.parametrize("end", [2**31 - 1, 2**31 - 2, 2**31 - 319, 1000])
@pytest.mark.parametrize("count", [0, 1, 63, 64, 65, 320, 1000])
def test_chunks_cover_the_entries_and_stay_among_them(walk, most, end, count):
    got = walk(end - count, end, most)
    assert [k for at, cn in got for k in range(at, at + cn)] == list(range(end - count, end))
    assert all(0 < cn <= most for _, cn in got)


@pytest.mark.parametrize("source,fixed_steps", [
    ("kernels_sell.hip", ["c0 += kChkEntries", "kb += 64"]),
    ("kernels_cg.hip", ["c0 += CHUNK"]),
    ("kernels_bfs.hip", ["k0 += kRow", "int j = u.b + l", " int j[kBfsItems]"]),
])
def test_kernel_walks_take_the_step(source, fixed_steps):
    """No walk of the entries adds a fixed length to a signed 32-bit entry index."""
    text = open(os.path.join(ROOT, "paper_2412_08059_amd", "csrc", source)).read()
    assert [s for s in fixed_steps if s in text] == []
