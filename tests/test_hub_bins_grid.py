"""How the hub-list kernel deals out the pieces of a short list in bins: every
piece of every die to one workgroup, for every grid and however unevenly the
dies are filled, and a die's to its own workgroups where all are filled alike
(CPU: the kernel's own index function, compiled for the host)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "ppsp_dev.h"
using namespace ppsp;
int main() {
    const uint32_t lists[][XCDS] = {{1, 1, 1, 1, 1, 1, 1, 1}, {37, 37, 37, 37, 37, 37, 37, 37}, {0, 0, 0, 1, 0, 0, 0, 0},
                                    {0, 0, 0, 0, 0, 0, 0, 2560}, {900, 0, 0, 0, 0, 0, 0, 1}, {1, 0, 5000, 0, 1, 0, 1, 0},
                                    {3, 1, 4, 1, 5, 9, 2, 6}, {0, 700, 0, 0, 20, 0, 0, 0}, {3999999, 1, 0, 0, 0, 0, 0, 0}};
    for (uint32_t grid = XCDS; grid <= 6144; grid++)
        for (const auto &recs : lists) {
            if (recs[0] > 1000000 && grid % 512) continue;
            std::vector<std::vector<uint32_t>> taken(XCDS);
            for (uint32_t x = 0; x < XCDS; x++) taken[x].assign(recs[x], 0);
            for (uint32_t b = 0; b < grid; b++) {
                const DieShare s = die_share(recs, grid, b);
                if (s.x >= XCDS || s.step == 0 || s.first >= s.step) { printf("grid %u block %u: no share\n", grid, b); return 1; }
                for (uint32_t k = s.first; k < recs[s.x]; k += s.step) taken[s.x][k]++;
                if (recs == lists[1] && grid % XCDS == 0 && s.x != b % XCDS) { printf("grid %u: not its own\n", grid); return 1; }
            }
            for (uint32_t x = 0; x < XCDS; x++)
                for (uint32_t k = 0; k < recs[x]; k++)
                    if (taken[x][k] != 1) { printf("grid %u: die %u piece %u %u times\n", grid, x, k, taken[x][k]); return 1; }
        }
    return 0;
}
"""


def test_every_piece_once(tmp_path):
    if not os.path.exists(HIPCC) and shutil.which("hipcc") is None:
        pytest.skip("no hipcc")
    src, exe = tmp_path / "deal.hip", tmp_path / "deal"
    src.write_text(PROGRAM)
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-O2", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                        "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"),
                        "-I", os.path.join(ROOT, "paper_2506_16488_amd", "csrc"), str(src), "-o", str(exe)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
