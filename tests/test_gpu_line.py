"""The kernel for 3x3 stride-1 layers that takes 256 consecutive pixels of all images at a time (csrc/bwd_line.h): image sizes at
which lines, images and tiles begin in every position to each other, the widest image it takes and the next, column counts around
its tiles, short last chunks, one and two of m, any n of m up to 32 and none pruned, every ranker.  Against the oracle on sampled pixels, image borders included.

Tolerance: the tests of the other bf16 kernels, 1e-2 of sum |a||w| (one rounding to bf16 shows 2^-9)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2202_00774_amd as sdgp
from paper_2202_00774_amd import workloads as wl
from util import rel_error, to_gpu, to_host

pytestmark = pytest.mark.gpu


def check(B, H, Wd, C_in, C_out, n, m, ranker, seed=5):
    layer = wl.ConvLayer("t", B, H, Wd, C_in, C_out, 3, 3, 1, 1)
    dO = wl.laplace_with_zeros(layer.dO_shape, 1e-3, 0.3, seed=seed, dtype=wl.BF16)
    W = wl.normal(layer.W_shape, 0.1, seed + 1, wl.BF16)
    total = B * H * Wd
    ends = np.concatenate([np.arange(min(total, 300)), np.arange(max(0, total - 300), total)])   # the first and the last tile
    pixels = np.unique(np.concatenate([ends, np.random.default_rng(2).choice(total, min(total, 2000), replace=False)]))
    pruned = oracle.prune(dO, n, m, ranker, seed=seed)[0]
    ref, ab = oracle.conv_bwd_data(pruned, W, H, Wd, 1, 1, pixels=pixels)
    out = sdgp.sdgp_conv_bwd_data(to_gpu(dO), to_gpu(W), H, Wd, 1, 1, n, m, ranker, seed)
    got = wl.to_f64(to_host(out.reshape(-1, C_in)[torch.from_numpy(pixels).to(out.device)]))
    assert rel_error(got, ref, ab) <= 1e-2
    assert np.all(got[ab == 0] == 0)


@pytest.mark.parametrize("ranker", (oracle.RANDOM, oracle.GREEDY, oracle.GREEDY_ADJUSTED))
@pytest.mark.parametrize("B,H,Wd", [(33000, 1, 1), (9000, 2, 2), (2100, 1, 16), (600, 60, 1), (1100, 3, 11), (130, 16, 16), (170, 15, 13),
                                    (9, 63, 63), (11, 50, 62), (9, 64, 64), (1, 600, 63)])
def test_image_sizes(B, H, Wd, ranker):
    check(B, H, Wd, 64, 64, 2, 4, ranker)


@pytest.mark.parametrize("n,m,ranker", [(2, 4, oracle.GREEDY), (1, 4, oracle.GREEDY), (1, 4, oracle.GREEDY_ADJUSTED), (2, 8, oracle.RANDOM),
                                        (1, 8, oracle.RANDOM), (2, 16, oracle.GREEDY_ADJUSTED), (2, 16, oracle.GREEDY)])
@pytest.mark.parametrize("C_in,C_out", [(8, 32), (72, 16), (128, 96), (136, 80), (264, 208), (448, 48)])
def test_channels(C_in, C_out, n, m, ranker):
    check(150 if C_in < 264 else 50, 16, 17, C_in, C_out, n, m, ranker)


@pytest.mark.parametrize("C_out", [8, 40, 56, 72])
def test_groups_of_eight_cut_by_the_last_chunk(C_out):
    check(150, 16, 17, 72, C_out, 2, 8, oracle.GREEDY_ADJUSTED)
    check(150, 16, 17, 72, C_out, 1, 4, oracle.RANDOM)


@pytest.mark.parametrize("n,m,ranker", [(3, 4, oracle.GREEDY_ADJUSTED), (4, 8, oracle.RANDOM), (5, 8, oracle.GREEDY), (4, 16, oracle.GREEDY),
                                        (9, 16, oracle.RANDOM), (2, 32, oracle.GREEDY), (4, 32, oracle.RANDOM), (16, 32, oracle.GREEDY_ADJUSTED),
                                        (4, 4, oracle.GREEDY), (8, 8, oracle.RANDOM)])
@pytest.mark.parametrize("B,H,Wd,C_in,C_out", [(150, 16, 17, 8, 32), (150, 16, 17, 72, 96), (50, 16, 17, 264, 160), (9000, 2, 2, 64, 64),
                                               (9, 63, 63, 64, 32), (11, 50, 62, 40, 64)])
def test_whole_gradient(B, H, Wd, C_in, C_out, n, m, ranker):
    check(B, H, Wd, C_in, C_out, n, m, ranker)


@pytest.mark.parametrize("C_out,n,m", [(8, 4, 8), (40, 3, 4), (56, 5, 8), (72, 8, 8), (80, 5, 16), (48, 16, 16)])
def test_whole_gradient_cut_by_the_last_chunk(C_out, n, m):
    check(150, 16, 17, 72, C_out, n, m, oracle.GREEDY_ADJUSTED)
    check(150, 16, 17, 72, C_out, n, m, oracle.RANDOM)


@pytest.mark.parametrize("n,m,ranker", [(2, 4, oracle.GREEDY), (2, 4, oracle.RANDOM), (1, 4, oracle.GREEDY_ADJUSTED), (2, 8, oracle.GREEDY),
                                        (2, 16, oracle.RANDOM), (3, 4, oracle.GREEDY), (4, 8, oracle.RANDOM), (5, 16, oracle.GREEDY_ADJUSTED),
                                        (4, 32, oracle.GREEDY), (4, 4, oracle.GREEDY)])
@pytest.mark.parametrize("B,C_in,C_out", [(40, 64, 64), (20, 136, 96)])
def test_wider_images_stay_on_the_row_kernel(B, C_in, C_out, n, m, ranker):
    check(B, 20, 70, C_in, C_out, n, m, ranker)


def test_infinite_gradient_stays_with_its_pixels():
    """The pixels next to it in the line, but across an image's or a line's end, are not its neighbours."""
    layer = wl.ConvLayer("t", 150, 16, 17, 64, 64, 3, 3, 1, 1)
    dO = wl.laplace_with_zeros(layer.dO_shape, 1e-3, 0.3, seed=3, dtype=wl.BF16)
    for at in ((0, 5, 16), (7, 15, 16), (8, 0, 0), (149, 15, 16), (20, 8, 0)):
        dO[at] = 0x7F80
    W = wl.normal(layer.W_shape, 0.1, 4, wl.BF16)
    out = sdgp.sdgp_conv_bwd_data(to_gpu(dO), to_gpu(W), 16, 17, 1, 1, 2, 4, oracle.GREEDY, 1)
    hit = np.zeros((150, 16, 17), bool)
    for b, y, x in ((0, 5, 16), (7, 15, 16), (8, 0, 0), (149, 15, 16), (20, 8, 0)):
        hit[b, max(0, y - 1):y + 2, max(0, x - 1):x + 2] = True
    assert np.array_equal(~np.isfinite(wl.to_f64(to_host(out))).all(axis=3), hit)


@pytest.mark.parametrize("n,m,ranker", [(4, 4, oracle.GREEDY), (4, 8, oracle.RANDOM), (5, 16, oracle.GREEDY), (16, 32, oracle.GREEDY_ADJUSTED)])
@pytest.mark.parametrize("B,H,Wd,C_in,C_out", [(95000, 1, 1, 136, 32), (40000, 2, 2, 72, 64), (30000, 1, 3, 136, 32), (13000, 3, 3, 72, 32),
                                               (13000, 1, 56, 40, 32), (600, 300, 1, 72, 64)])
def test_whole_gradient_of_images_of_few_lines(B, H, Wd, C_in, C_out, n, m, ranker):
    """One workgroup of the line kernel on a CU, or the row kernel where its rounds are the shorter ones."""
    check(B, H, Wd, C_in, C_out, n, m, ranker)
