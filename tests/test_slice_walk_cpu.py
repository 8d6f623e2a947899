"""The slice ranges that the SELL products walk, formed from a few numbers, are
those of the definition: XCD x takes the groups floor(b(x) G / B) up to
floor(b(x + 1) G / B), b(x) being the blocks on the XCDs below it."""

import os
import random
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HARNESS = r"""
#include "mpcg_internal.hpp"
#include <cstdio>
int main()
{
    int nslices, grid;
    while (std::scanf("%d %d", &nslices, &grid) == 2) {
        const mpcg::WalkNum t = mpcg::walk_num(nslices, grid);
        for (int x = 0; x < mpcg::kNumXcd; ++x) std::printf("%d %d ", mpcg::walk_first(t, x), mpcg::walk_blocks(t, x));
        std::printf("%d\n", mpcg::walk_first(t, mpcg::kNumXcd));
    }
    return 0;
}
"""


def _ranges(nslices, grid):
    groups, before, out = (nslices + 3) // 4, 0, []
    for x in range(8):
        blocks = grid // 8 + (1 if x < grid % 8 else 0)
        out += [before * groups // grid, blocks]
        before += blocks
    return out + [groups]


def test_ranges_from_numbers(tmp_path):
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(HARNESS)
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           f"-I{ROOT}/include", f"-I{ROOT}/paper_2412_08059_amd/csrc", str(src), "-o", str(exe)])
    rng = random.Random(5)
    asked = [(n, g) for g in (1, 2, 7, 8, 9, 1023, 1792, 2047, 2048) for n in (1, 3, 4, 5, 64, 4 * g - 1, 4 * g + 1, 2**25)]
    asked += [(rng.randrange(1, 2**rng.randrange(2, 26)), rng.randrange(1, 2049)) for _ in range(20000)]
    out = subprocess.run([str(exe)], input="".join(f"{n} {g}\n" for n, g in asked), text=True, check=True,
                         stdout=subprocess.PIPE).stdout.splitlines()
    assert len(out) == len(asked)
    for (n, g), line in zip(asked, out):
        assert [int(v) for v in line.split()] == _ranges(n, g), (n, g)
