"""The planner of the fp32 products on the bf16 matrix instructions and what its first pass shares with it, compiled for the
host (tests/native/f32_split_host_check.hip)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc to compile the host check")
def test_host_check(tmp_path):
    exe = str(tmp_path / "f32_split_host_check")
    src = os.path.join(ROOT, "tests", "native", "f32_split_host_check.hip")
    cmd = [HIPCC, "-O2", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2202_00774_amd", "csrc"), "-o", exe, src]
    subprocess.run(cmd, check=True, capture_output=True, timeout=300)
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stdout[-2000:]
    assert "total mismatches 0" in run.stdout
