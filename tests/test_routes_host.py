"""Which kernel takes the layers that the GPU tests are there for: the library's own dispatch on the CPU, with launches that write
the kernel's name instead (tests/native/launch_names.c), so that a test whose layer moves to another kernel says so."""
import os
import re
import shutil
import subprocess
import sys

import pytest

import test_gpu_keepset as keepset

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2202_00774_amd", "libsdgp.so")

pytestmark = pytest.mark.skipif(shutil.which("gcc") is None, reason="needs gcc")

ASK = """
import ctypes, sys
ctypes.CDLL(sys.argv[2], mode=ctypes.RTLD_GLOBAL)   # found in front of the HIP runtime, which the library brings
lib = ctypes.CDLL(sys.argv[1])
i64, i32, vp, sz = ctypes.c_int64, ctypes.c_int, ctypes.c_void_p, ctypes.c_size_t
lib.sdgp_conv_bwd_data.argtypes = [vp] * 3 + [i64] * 5 + [i32] * 8 + [ctypes.c_uint64, vp, sz, vp]
lib.sdgp_conv_bwd_data_workspace.argtypes = [i64] * 5 + [i32] * 7
lib.sdgp_conv_bwd_data_workspace.restype = sz
for line in sys.stdin:
    *geometry, n, m, ranker = map(int, line.split())
    need = lib.sdgp_conv_bwd_data_workspace(*geometry, 1, n, m)
    rc = lib.sdgp_conv_bwd_data(1 << 20, 1 << 20, 1 << 20, *geometry, 1, n, m, ranker, 0, 1 << 20, need, None)
    sys.stderr.write("done %d\\n" % rc)
    sys.stderr.flush()
"""


@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    names = str(tmp_path_factory.mktemp("native") / "launch_names.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-o", names, os.path.join(ROOT, "tests", "native", "launch_names.c"), "-ldl"],
                   check=True, capture_output=True, timeout=60)

    def ask(calls):
        """The kernels of each call (B, H, Wd, C_in, C_out, R, S, stride, pad, n, m, ranker), without template arguments."""
        lines = "\n".join(" ".join(map(str, c)) for c in calls)
        run = subprocess.run([sys.executable, "-c", ASK, LIB, names], input=lines, capture_output=True, text=True, timeout=120)
        found, kernels = [], []
        for line in run.stderr.splitlines():
            if line.startswith("launch "):
                kernel = re.match(r"launch _ZN4sdgp\d+(bwd_[a-z0-9_]+?)I", line)
                kernels.append(kernel.group(1) if kernel else "other")   # (kernels of one source file have no name outside it)
            elif line.startswith("done "):
                assert line == "done 0"
                found.append(kernels)
                kernels = []
        assert len(found) == len(calls), run.stderr[-500:]
        return found
    return ask


def geometry(layer):
    return layer.B, layer.H, layer.Wd, layer.C_in, layer.C_out, layer.R, layer.S, layer.stride, layer.pad


KEPT = {"row512_n64_wide": "bwd_row", "row512_n128_wide_spread": "bwd_row", "row512_n64": "bwd_line", "row512_n128": "bwd_line",
        "row512_n128_spread": "bwd_line", "row256_n64": "bwd_line", "row512_8x8_n128": "bwd_line", "pw_n64": "bwd_pw", "pw_n160": "bwd_pw",
        "pw_s2_n64": "bwd_pw", "stride2_n128_spread": "bwd_stride2", "gather_s2_3x3": "bwd_pw_classes", "gather_s2_4x4": "bwd_pw_classes",
        "conv3_n64": "bwd_line", "conv3_n64_spread": "bwd_line", "conv3_5x5": "bwd_conv3", "tiled_n48": "bwd_line",
        "tiled_n48_spread": "bwd_line", "tiled_s2": "bwd_stride2", "conv3_n64_wide": "bwd_conv3", "conv3_n64_wide_spread": "bwd_conv3",
        "tiled_n48_wide": "bwd_tiled", "tiled_n48_wide_spread": "bwd_tiled", "tiled_5x5s2": "bwd_tiled", "small_n64": "bwd_small",
        "small_n64_spread": "bwd_small", "small_5x5": "bwd_small", "small_n48_spread": "bwd_small", "small_s2": "bwd_small",
        "small_1x1_n160": "bwd_small", "narrow_3x3": "other", "narrow_7x7s2": "other"}
DENSE = {"line_n128": "bwd_line", "line_n96_spread": "bwd_line", "row_n96_wide": "bwd_row", "tiled_n64": "bwd_line",
         "tiled_n64_wide": "bwd_tiled", "tiled_n64_wide_spread": "bwd_tiled", "tiled_s2_n96": "bwd_tiled", "small_n96": "bwd_small",
         "small_s2_n96": "bwd_small"}


def test_kept_set_layers(routes):
    assert [l.name for l, _ in keepset.CASES] == list(KEPT) and [l.name for l, _ in keepset.DENSE_ROWS] == list(DENSE)
    asked = [(l.name, geometry(l) + (n, m, r), KEPT[l.name]) for l, _ in keepset.CASES
             for n, m, r in keepset.nm_settings(tuple(m for m in (4, 8, 16) if l.C_out % m == 0))]
    asked += [(l.name, geometry(l) + (n, m, r), DENSE[l.name]) for l, _ in keepset.DENSE_ROWS
              for n, m in ((3, 4), (4, 8), (4, 16), (2, 32), (16, 32)) for r in keepset.RANKERS]
    for (name, call, want), kernels in zip(asked, routes([call for _, call, _ in asked])):
        assert kernels[-1] == want, (name, call, kernels)


@pytest.mark.parametrize("shape,n,m,kernel", [
    # tests/test_gpu_small.py
    ((12, 20, 70, 64, 96, 3, 3, 1, 1), 2, 4, "bwd_tiled"), ((12, 20, 70, 64, 96, 3, 3, 1, 1), 16, 32, "bwd_tiled"),
    ((140, 17, 19, 64, 96, 5, 5, 2, 2), 2, 16, "bwd_tiled"), ((140, 17, 19, 64, 96, 5, 5, 2, 2), 4, 4, "bwd_tiled"),
    ((4500, 1, 1, 64, 448, 3, 3, 2, 1), 2, 4, "bwd_tiled"), ((2000, 5, 1, 64, 448, 3, 3, 2, 1), 4, 4, "bwd_tiled"),
    ((70, 16, 16, 64, 96, 3, 3, 1, 1), 7, 16, "bwd_line"), ((300, 9, 11, 24, 96, 3, 3, 2, 1), 1, 4, "bwd_stride2"),
    ((300, 9, 11, 24, 96, 3, 3, 2, 1), 7, 16, "bwd_tiled"), ((170, 14, 14, 72, 64, 3, 3, 2, 1), 2, 4, "bwd_pw_classes"),
    # tests/test_gpu_stride2.py
    ((70000, 1, 1, 64, 64, 3, 3, 2, 1), 2, 4, "bwd_stride2"), ((9000, 1, 16, 64, 64, 3, 3, 2, 1), 2, 4, "bwd_stride2"),
    ((1100, 60, 1, 64, 64, 3, 3, 2, 1), 2, 4, "bwd_stride2"), ((20000, 3, 3, 72, 128, 3, 3, 2, 1), 2, 4, "bwd_pw_classes"),
    ((6000, 5, 5, 72, 128, 3, 3, 2, 1), 2, 16, "bwd_pw_classes"),
    # tests/test_gpu_line.py
    ((9, 63, 63, 64, 64, 3, 3, 1, 1), 2, 4, "bwd_line"), ((40, 20, 70, 64, 64, 3, 3, 1, 1), 4, 8, "bwd_row"),
    ((95000, 1, 1, 136, 32, 3, 3, 1, 1), 4, 4, "bwd_line"), ((40000, 2, 2, 72, 64, 3, 3, 1, 1), 4, 8, "bwd_line"),
    ((13000, 3, 3, 72, 32, 3, 3, 1, 1), 4, 4, "bwd_row"), ((13000, 3, 3, 72, 32, 3, 3, 1, 1), 16, 32, "bwd_line"),
    ((600, 300, 1, 72, 64, 3, 3, 1, 1), 5, 16, "bwd_row")])
def test_layers_of_the_kernels_tests(routes, shape, n, m, kernel):
    assert routes([shape + (n, m, 0)])[0][-1] == kernel
