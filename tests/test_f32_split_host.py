"""The planner of the fp32 products on the bf16 matrix instructions and what its first pass shares with it, compiled for the
host (tests/native/f32_split_host_check.hip)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc to compile the host check")


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("native") / "f32_split_host_check")
    src = os.path.join(ROOT, "tests", "native", "f32_split_host_check.hip")
    cmd = [HIPCC, "-O2", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2202_00774_amd", "csrc"), "-o", exe, src]
    subprocess.run(cmd, check=True, capture_output=True, timeout=300)
    return exe


def test_host_check(check):
    run = subprocess.run([check], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stdout[-2000:]
    assert "total mismatches 0" in run.stdout


def tile(check, shape, n, m):
    """Rows and grid positions of the kernel that the planner picks."""
    out = subprocess.run([check, *(str(v) for v in (*shape, n, m))], capture_output=True, text=True, timeout=60, check=True).stdout.split()
    return None if out == ["none"] else (int(out[0]), int(out[1]))


def test_gpu_tests_reach_every_tile(check):
    """The layers of tests/test_gpu_f32_split.py are on the tiles they are there for, compressed and not."""
    import test_gpu_f32_split as gpu
    for layers, patterns in ((gpu.SHAPES, [(n, m) for n, m, _ in gpu.PATTERNS]), (gpu.GROUP_LAYERS, gpu.GROUPS)):
        for n, m in patterns:
            assert {want for _, want in layers} == {(128, 256), (256, 384), (256, 512)}
            for shape, want in layers:
                assert tile(check, shape, n, m) == want, (shape, n, m)
