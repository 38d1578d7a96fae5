"""The peel's barrier test beyond 2^31 arrivals, on the CPU."""
import os
import subprocess

from conftest import ROOT

SOURCE = r"""
#include "kc_barrier.h"
#include <cstdio>
// Barriers e of `grid` blocks: all of them wait until the last has arrived, and none waits then,
// not even when faster blocks have arrived at the next barrier already.
int main() {
    const unsigned grids[] = {1, 16, 61, 64};
    for (unsigned grid : grids)
        for (unsigned long long at = 1ull << 31; at <= 1ull << 32; at += 1ull << 31)
            for (unsigned long long e = at / grid - 3; e <= at / grid + 3; e++) {
                const unsigned want = static_cast<unsigned>(e) * grid;
                for (unsigned i = 0; i <= 2 * grid - 1; i++) {
                    const unsigned arrived = static_cast<unsigned>((e - 1) * grid + i);
                    if (kc::arrivals_missing(arrived, want) != (i < grid)) {
                        std::printf("grid %u barrier %llu arrived %u\n", grid, e, i);
                        return 1;
                    }
                }
            }
    return 0;
}
"""


def test_barrier_passes_2_to_the_31_arrivals(tmp_path):
    src, exe = tmp_path / "b.cpp", tmp_path / "b"
    src.write_text(SOURCE)
    inc = os.path.join(ROOT, "paper_2104_13209_amd", "csrc")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", inc, str(src), "-o", str(exe)])
    assert subprocess.run([str(exe)]).returncode == 0
