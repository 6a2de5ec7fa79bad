"""The rules by which 3x3 layers find their kernel, compiled for the host without optimisation (tests/native/plan_host_check.hip)."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc to compile the host check")


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("native") / "plan_host_check")
    src = os.path.join(ROOT, "tests", "native", "plan_host_check.hip")
    subprocess.run([HIPCC, "-O0", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2202_00774_amd", "csrc"), "-o", exe, src],
                   check=True, capture_output=True, timeout=300)

    def run(*args):
        done = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, timeout=60)
        assert done.returncode == 0, (args, done.returncode)
        return done.stdout.split()
    return run


@pytest.mark.parametrize("C_out", [256, 512, 1000, 1024])
@pytest.mark.parametrize("H,Wd", [(1, 1), (14, 14), (56, 56), (3, 1023)])
def test_stride2_shapes_beyond_the_lds(ask, C_out, H, Wd):
    """Layers of which no shape, or not every one, fits a CU's LDS: 512 <- 512 at 14x14 wants 240640 bytes for one of them."""
    for lds in (80 * 1024, 132 * 1024):
        got = ask("stride2", 256, H, Wd, 512, C_out, lds)
        assert got == ["none"] or int(got[2]) <= lds
    assert ask("stride2", 256, 14, 14, 512, 1024, 132 * 1024) == ["none"]


def test_stride2_shapes_within_the_lds(ask):
    assert ask("stride2", 256, 56, 56, 128, 128, 80 * 1024) == ["128", "256", "81408", "784"]


@pytest.mark.parametrize("ahead,B,H,Wd,C_in,C_out,taker", [
    (1, 11004, 3, 3, 448, 128, "classes"), (1, 51098, 3, 3, 64, 128, "classes"), (1, 6156, 3, 5, 512, 128, "classes"),
    (1, 20310, 5, 5, 64, 128, "classes"),
    (0, 11004, 3, 3, 448, 128, "stride2"),      # nothing ranked ahead there
    (1, 11004, 3, 3, 448, 64, "stride2"),       # 64 channels
    (1, 6000, 5, 7, 256, 128, "stride2"), (1, 6000, 4, 4, 256, 128, "stride2"), (1, 256, 56, 56, 128, 128, "stride2")])
def test_small_images_of_odd_sides(ask, ahead, B, H, Wd, C_in, C_out, taker):
    """3x3 stride 2, n <= 2: the kernel that computes all four parity classes of every position, and the one that computes what exists
    of them, measured on either side of the line."""
    assert ask("classes", ahead, B, H, Wd, C_in, C_out) == [taker]


RANDOM, GREEDY, RESCALED = 0, 1, 2


@pytest.mark.parametrize("B,H,Wd,C_in,C_out,n,m,ranker,columns", [
    (15, 62, 62, 432, 240, 2, 8, RANDOM, 64), (17, 63, 63, 384, 256, 1, 4, RANDOM, 64),     # one workgroup of 128 columns a CU
    (1038, 2, 33, 352, 256, 2, 16, RANDOM, 64),
    (33, 60, 60, 128, 64, 2, 16, RANDOM, 128),                                              # two
    (512, 16, 16, 128, 256, 2, 4, GREEDY, 128), (82, 34, 34, 224, 192, 2, 8, RESCALED, 128), (301, 9, 9, 128, 96, 2, 4, RESCALED, 64),
    (60, 27, 27, 448, 128, 1, 4, GREEDY, 64)])
def test_line_columns(ask, B, H, Wd, C_in, C_out, n, m, ranker, columns):
    assert ask("columns", B, H, Wd, C_in, C_out, n, m, ranker) == [str(columns)]


def test_line_alone_on_a_cu(ask):
    alone = {(H, Wd) for H in (1, 2, 3, 4, 7, 56, 300) for Wd in (1, 2, 3, 4, 7, 56, 57, 58, 63) if ask("alone", H, Wd) == ["1"]}
    assert {(1, 1), (2, 2), (3, 3), (1, 56), (300, 1), (300, 58), (300, 63)} <= alone
    assert not alone & {(4, 4), (7, 7), (56, 56), (300, 2), (300, 56)}


@pytest.mark.parametrize("mode,m,blocks,rows,bn,line,taker", [
    (0, 4, 746, 512, 128, 2984, "row"),      # 512 <- 64 at 1x1, batch 95360: 57 us against 85
    (0, 4, 202, 256, 64, 202, "line"),       # a round of either
    (1, 8, 494, 512, 128, 988, "line"), (1, 32, 1897, 512, 64, 4332, "row")])
def test_row_kernel_beside_a_lone_line_kernel(ask, mode, m, blocks, rows, bn, line, taker):
    assert ask("row", mode, m, blocks, rows, bn, line) == [taker]


@pytest.mark.parametrize("mode,m,B,H,Wd,C_in,way", [
    (0, 4, 95360, 1, 1, 512, "search"), (1, 8, 63185, 2, 2, 56, "search"),
    (2, 4, 95360, 1, 1, 512, "line"),          # n <= 2: faster there in every layer seen
    (0, 4, 87, 178, 1, 192, "line"),           # one round: a search of 8 us for a call of 7
    (0, 4, 3000, 1, 56, 64, "line"), (0, 4, 13000, 1, 56, 64, "search"),
    (0, 4, 64, 60, 60, 512, "line"), (0, 4, 95360, 4, 4, 512, "line")])     # wide; two workgroups on a CU
def test_what_is_planned_for_the_row_kernel(ask, mode, m, B, H, Wd, C_in, way):
    assert ask("plan", mode, m, B, H, Wd, C_in) == [way]


def test_no_line_kernel_is_built_that_no_layer_gets(ask):
    """The kernels of 128 columns in the library are those that the rule of the columns picks for some layer."""
    lib = os.path.join(ROOT, "paper_2202_00774_amd", "libsdgp.so")
    names = subprocess.run(["nm", "-C", lib], capture_output=True, text=True, check=True).stdout
    built = set(re.findall(r"bwd_line<128, 2, (\d+), (\d+), (true|false), (true|false)>", names))
    picked = set()
    for m in (4, 8, 16):
        for ranker in (RANDOM, GREEDY, RESCALED):
            for n in (1, 2):
                for C_out in (96, 80):
                    if ask("columns", 256, 16, 16, 128, C_out, n, m, ranker) == ["128"]:
                        picked.add((str(m), str(ranker), "true" if n == 1 or C_out % 32 else "false", "true" if n == 2 else "false"))
    assert len(picked) == 18 and built == picked
