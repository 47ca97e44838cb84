"""Grids of kernels that number their workgroups in one run (csrc/launch_grid.hpp, compiled here for the
CPU): every workgroup has a place, no dimension reaches the 2^32 work-items that a launch refuses, and
an ordinary call's grid is one row of exactly its workgroups."""
import subprocess
from pathlib import Path

CSRC = Path(__file__).resolve().parent.parent / "paper_2602_09323_amd" / "csrc"

SOURCE = r"""
#include "launch_grid.hpp"
#include <stdio.h>
using namespace coopt;
int main()
{
    const long long row = kGridRow;
    const long long sizes[] = {1, 8, row - 1, row, row + 1, 2 * row, 2 * row + 1, (1LL << 24) - 1, 1LL << 24,
                               (1LL << 24) + 1, 165191050LL, 0x7fffffffLL};
    for (long long n : sizes) {
        const Grid g = grid_of(n);
        const long long last = grid_index(g.x - 1, g.y - 1);
        bool ok = g.x * 256LL < 1LL << 32 && g.y < 65536 && last >= n - 1 && last - (n - 1) < g.x;
        if (n <= row) ok = ok && g.x == n && g.y == 1;
        for (unsigned y = 1; y < g.y; ++y) ok = ok && grid_index(0, y) == grid_index(g.x - 1, y - 1) + 1;
        if (!ok) printf("%lld workgroups: grid %u x %u\n", n, g.x, g.y);
    }
    return 0;
}
"""


def test_grids_hold_every_workgroup(tmp_path):
    src, exe = tmp_path / "grid.cpp", tmp_path / "grid"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", f"-I{CSRC}", str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout == ""
