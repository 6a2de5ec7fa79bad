"""The kernel for 3x3 layers of stride 2 that computes all four parity classes in one workgroup (csrc/bwd_stride2.h): odd and even
image sizes down to one pixel, where lines, images and tiles begin in every position to each other, the column counts of its three
tile shapes, short last chunks, one and two of m, every ranker.  Against the oracle on sampled pixels.

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
    layer = wl.ConvLayer("t", B, H, Wd, C_in, C_out, 3, 3, 2, 1)
    dO = wl.laplace_with_zeros(layer.dO_shape, 1e-3, 0.3, seed=seed, dtype=wl.BF16)
    W = wl.normal(layer.W_shape, 0.1, seed + 1, wl.BF16)
    total = B * H * Wd
    ends = np.concatenate([np.arange(min(total, 300)), np.arange(max(0, total - 300), total)])   # the first and the last tile
    pixels = np.unique(np.concatenate([ends, np.random.default_rng(2).choice(total, min(total, 2000), replace=False)]))
    pruned = oracle.prune(dO, n, m, ranker, seed=seed)[0]
    ref, ab = oracle.conv_bwd_data(pruned, W, H, Wd, 2, 1, pixels=pixels)
    out = sdgp.sdgp_conv_bwd_data(to_gpu(dO), to_gpu(W), H, Wd, 2, 1, n, m, ranker, seed)
    got = wl.to_f64(to_host(out.reshape(-1, C_in)[torch.from_numpy(pixels).to(out.device)]))
    assert rel_error(got, ref, ab) <= 1e-2
    assert np.all(got[ab == 0] == 0)


@pytest.mark.parametrize("ranker", (oracle.RANDOM, oracle.GREEDY, oracle.GREEDY_ADJUSTED))
@pytest.mark.parametrize("B,H,Wd", [(70000, 2, 2), (40000, 3, 2), (20000, 2, 5), (2100, 2, 31), (1100, 63, 2), (1500, 13, 11),
                                    (300, 28, 28), (300, 27, 29), (30, 100, 112), (70000, 1, 1), (30000, 1, 2), (9000, 1, 16), (2100, 1, 31),
                                    (1100, 60, 1), (12000, 5, 1)])
def test_image_sizes(B, H, Wd, ranker):
    check(B, H, Wd, 64, 64, 2, 4, ranker)


@pytest.mark.parametrize("n,m,ranker", [(2, 4, oracle.GREEDY), (1, 4, oracle.GREEDY), (1, 4, oracle.GREEDY_ADJUSTED), (2, 8, oracle.RANDOM),
                                        (1, 8, oracle.RANDOM), (2, 16, oracle.GREEDY_ADJUSTED), (2, 16, oracle.GREEDY)])
@pytest.mark.parametrize("B,C_in,C_out", [(460, 8, 32), (460, 72, 16), (460, 128, 96), (200, 136, 80), (200, 264, 208), (100, 448, 48),
                                          (20, 40, 288), (20, 232, 352)])
def test_channels(B, C_in, C_out, n, m, ranker):
    check(B, 24, 25, C_in, C_out, n, m, ranker)


@pytest.mark.parametrize("C_out", [8, 40, 56, 72])
def test_groups_of_eight_cut_by_the_last_chunk(C_out):
    check(460, 24, 25, 72, C_out, 2, 8, oracle.GREEDY_ADJUSTED)
    check(460, 24, 25, 72, C_out, 1, 4, oracle.RANDOM)


def test_infinite_gradient_stays_with_its_pixels():
    """The pixels next to it in the line, but across an image's or a line's end, are not its neighbours."""
    layer = wl.ConvLayer("t", 460, 24, 25, 64, 64, 3, 3, 2, 1)
    dO = wl.laplace_with_zeros(layer.dO_shape, 1e-3, 0.3, seed=3, dtype=wl.BF16)
    places = ((0, 5, 12), (7, 11, 12), (8, 0, 0), (459, 11, 12), (20, 8, 0))
    hit = np.zeros((460, 24, 25), bool)
    for b, p, q in places:
        dO[b, p, q] = 0x7F80
        hit[b, max(0, 2 * p - 1):2 * p + 2, max(0, 2 * q - 1):2 * q + 2] = True
    W = wl.normal(layer.W_shape, 0.1, 4, wl.BF16)
    out = sdgp.sdgp_conv_bwd_data(to_gpu(dO), to_gpu(W), 24, 25, 2, 1, 2, 4, oracle.GREEDY, 1)
    assert np.array_equal(~np.isfinite(wl.to_f64(to_host(out))).all(axis=3), hit)


@pytest.mark.parametrize("n,m,ranker", [(2, 4, oracle.RANDOM), (1, 8, oracle.GREEDY), (2, 16, oracle.GREEDY_ADJUSTED)])
@pytest.mark.parametrize("B,H,Wd", [(20000, 3, 3), (9000, 3, 5), (9000, 5, 3), (6000, 5, 5)])
def test_small_images_of_odd_sides(B, H, Wd, n, m, ranker):
    """128 channels: the parity-class kernel with the gradient ranked ahead, which computes only the pixels there are."""
    check(B, H, Wd, 72, 128, n, m, ranker)
