"""Slices of calls that need more workgroups than a grid holds (csrc/launch_grid.hpp, compiled here for
the CPU): no slice reaches the 2^32 work-items that a launch refuses, every slice makes progress, a slice
of tokens begins at a whole word of a skip set, and an ordinary call is one launch."""
import subprocess
from pathlib import Path

CSRC = Path(__file__).resolve().parent.parent / "paper_2602_09323_amd" / "csrc"

SOURCE = r"""
#include "launch_grid.hpp"
#include <initializer_list>
#include <stdio.h>
using namespace coopt;
int main()
{
    for (int own : {13, 29, 61})
        for (int heads : {1, 2, 3, 8, 40, 4096})
            for (long long rows : {64LL * 4096, 1LL << 26, 218103807LL, 218103808LL, 0x7fffffffLL}) {
                const long long tokens = rows / heads, n = tokens_per_launch(tokens, own, heads);
                const long long wgs = ((n - 1) / own + 1) * heads, all = ((tokens - 1) / own + 1) * heads;
                bool ok = n > 0 && wgs * 256 < 1LL << 32 && (n >= tokens || n % 32 == 0);
                if (all <= 1 << 23) ok = ok && n == tokens;
                if (!ok) printf("%lld tokens, %d own, %d heads: %lld\n", tokens, own, heads, n);
            }
    for (long long seqs : {1LL, 3LL, 1000LL, 1LL << 20})
        for (long long wgs : {1LL, 30LL, 256LL, 40LL * 512, 1LL << 22}) {
            const long long n = seqs_per_launch(seqs, wgs);
            bool ok = n > 0 && n <= seqs && n * wgs * 256 < 1LL << 32;
            if (seqs * wgs <= 1 << 23) ok = ok && n == seqs;
            if (!ok) printf("%lld sequences of %lld: %lld\n", seqs, wgs, n);
        }
    return 0;
}
"""


def test_slices_fit_a_grid(tmp_path):
    src, exe = tmp_path / "grid.cpp", tmp_path / "grid"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", f"-I{CSRC}", str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout == ""
