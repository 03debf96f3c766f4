"""How the hub-list kernel deals out the pieces of a short list in bins: every
piece of every die to one of its workgroups, for every grid (CPU: the kernel's
own index functions, compiled for the host)."""
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
    for (uint32_t grid = XCDS; grid <= 6144; grid++) {
        uint32_t sum = 0;
        for (uint32_t x = 0; x < XCDS; x++) sum += die_blocks(grid, x);
        if (sum != grid) { printf("grid %u: %u workgroups\n", grid, sum); return 1; }
        for (uint32_t pieces : {1u, 37u, 2560u}) {
            std::vector<uint32_t> taken(XCDS * pieces, 0);
            for (uint32_t b = 0; b < grid; b++) {
                const uint32_t x = b % XCDS, step = die_blocks(grid, x);
                for (uint32_t k = b / XCDS; k < pieces; k += step) taken[x * pieces + k]++;
            }
            for (uint32_t k = 0; k < XCDS * pieces; k++)
                if (taken[k] != 1) { printf("grid %u: piece %u of %u %u times\n", grid, k, pieces, taken[k]); return 1; }
        }
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
