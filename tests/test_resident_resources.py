"""Registers and LDS of the resident kernel (CPU: hipcc cross-compiles
gfx950): a workgroup of 1,024 threads fills a compute unit, two of 512 share
one, so every form needs at most 128 registers a lane (16 waves on four SIMDs),
160 KB of LDS for 1,024 threads and half of it for 512, and no scratch."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def test_resident_kernel_fills_a_unit(tmp_path):
    if not os.path.exists(HIPCC) and shutil.which("hipcc") is None:
        pytest.skip("no hipcc")
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-c", "--cuda-device-only",
                        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                        "-Rpass-analysis=kernel-resource-usage", "-I", os.path.join(ROOT, "include"),
                        os.path.join(ROOT, "paper_2506_16488_amd", "csrc", "resident.hip"), "-o", str(tmp_path / "r.o")],
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    kernels, cur = {}, None
    for line in r.stderr.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            cur = kernels.setdefault(m.group(1), {})
            continue
        m = re.search(r"remark:\s+([A-Za-z ]+?)(?: \[[^\]]*\])?: (\d+)", line)
        if m and cur is not None:
            cur[m.group(1).strip()] = int(m.group(2))
    forms = {k: v for k, v in kernels.items() if "k_resident" in k}
    assert len(forms) == 12, list(kernels)
    for name, u in forms.items():
        threads = int(re.search(r"ILi(\d+)E", name).group(1))
        assert threads in (512, 1024)
        assert u["Occupancy"] >= 4 and u["VGPRs Spill"] == 0 and u["ScratchSize"] == 0, (name, u)
        assert u["LDS Size"] <= 160 * threads, (name, u)
