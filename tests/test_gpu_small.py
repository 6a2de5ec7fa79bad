"""The small-problem backward-data kernel against the oracle at the edges of its tiles (rows and columns that end inside
one, channel counts that end inside a reduction step, fewer steps than wavefronts, parity classes without a tap), and the
kernels that take over past its limits at the smallest sizes that still reach them.

Tolerance relative to sum |a||w|: one rounding of the result and one of a rescaled value to bf16 (2^-9 each) and fp32 sums
of K <= 1250 terms (K * 2^-24 = 7.5e-5): 5e-3.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2202_00774_amd as sdgp
from paper_2202_00774_amd import workloads as wl
from util import rel_error, to_gpu, to_host

pytestmark = pytest.mark.gpu

RANKERS = (oracle.RANDOM, oracle.GREEDY, oracle.GREEDY_ADJUSTED)


def check(shape, n, m, ranker, seed=11, linear=False):
    L = wl.ConvLayer("s", *shape)
    dO = wl.laplace_with_zeros(L.dO_shape, 1e-3, 0.3, seed=seed, dtype=wl.BF16)
    W = wl.normal(L.W_shape, 0.1, seed + 1, wl.BF16)
    pruned = oracle.prune(dO, n, m, ranker, seed=seed)[0]
    ref, ab = oracle.conv_bwd_data(pruned, W, L.H, L.Wd, L.stride, L.pad)
    if linear:
        out = sdgp.sdgp_linear_bwd_data(to_gpu(dO).view(L.B, L.C_out), to_gpu(W).view(L.C_out, L.C_in), n, m, ranker, seed).view(L.dD_shape)
    else:
        out = sdgp.sdgp_conv_bwd_data(to_gpu(dO), to_gpu(W), L.H, L.Wd, L.stride, L.pad, n, m, ranker, seed)
    got = wl.to_f64(to_host(out))
    assert rel_error(got, ref, ab) <= 5e-3
    assert np.all(got[ab == 0] == 0)


@pytest.mark.parametrize("ranker", RANKERS)
@pytest.mark.parametrize("n,m", [(2, 4), (3, 4), (1, 8), (5, 8), (2, 16), (7, 16), (1, 32), (16, 32), (4, 4), (5, 5)])
def test_groups(n, m, ranker):
    # C_out 40, 48, 96: reduction steps of 32 or 64 channels end inside the last one
    check((2, 5, 6, 40, 40 if m in (4, 5, 8) else 3 * m, 3, 3, 1, 1), n, m, ranker)


@pytest.mark.parametrize("rows,C_out,C_in", [(1, 8, 8), (33, 1000, 136), (64, 32, 264), (300, 512, 2048), (31, 264, 120)])
def test_linear_edges(rows, C_out, C_in):
    check((rows, 1, 1, C_in, C_out, 1, 1, 1, 0), 2, 4, oracle.RANDOM, linear=True)


@pytest.mark.parametrize("H,Wd,R,S,stride,pad", [(9, 8, 3, 3, 2, 1), (7, 7, 1, 1, 3, 0), (8, 11, 2, 5, 3, 1), (13, 9, 7, 7, 4, 3),
                                                 (5, 5, 3, 3, 1, 0), (9, 9, 3, 1, 2, 0)])
def test_filters(H, Wd, R, S, stride, pad):
    check((3, H, Wd, 24, 24, R, S, stride, pad), 2, 4, oracle.GREEDY)


@pytest.mark.parametrize("n,m", [(2, 4), (4, 4), (5, 8)])
@pytest.mark.parametrize("shape", [
    (2100, 4, 4, 264, 40, 1, 1, 1, 0),      # 1x1, ragged C_out: the pointwise kernel's short last chunk
    (270, 8, 8, 16, 40, 3, 3, 1, 1),        # ragged C_out, more than 512 tiles: the line kernel
    (300, 9, 11, 24, 40, 3, 3, 2, 1),       # the same, strided: bwd_tiled, at 2:4 the stride-2 kernel
    (70, 16, 16, 72, 64, 5, 5, 1, 2),       # a filter neither three wide nor 1x1, more than 512 tiles: bwd_conv3, at 5:8 bwd_tiled
    (65, 16, 16, 72, 64, 2, 2, 1, 1),
    (130, 16, 16, 64, 64, 3, 3, 1, 1),      # the line kernel
    (350, 7, 7, 136, 64, 1, 1, 1, 0),       # the pointwise kernel
    (170, 14, 14, 72, 64, 3, 3, 2, 1),      # its parity classes
])
def test_neighbours(shape, n, m):
    check(shape, n, m, oracle.RANDOM)


@pytest.mark.parametrize("ranker", RANKERS)
@pytest.mark.parametrize("n,m", [(1, 4), (2, 16), (7, 16), (4, 32), (16, 32)])
@pytest.mark.parametrize("shape", [(70, 16, 16, 64, 96, 3, 3, 1, 1), (300, 9, 11, 24, 96, 3, 3, 2, 1)])
def test_tiled_patterns(shape, n, m, ranker):
    """More than 512 tiles of 32 rows and fewer than 128 of 256: the line kernel.  A strided layer of which a parity class has fewer than
    64 tiles of 128: the stride-2 kernel, for general n:m bwd_tiled."""
    check(shape, n, m, ranker)


@pytest.mark.parametrize("ranker", RANKERS)
@pytest.mark.parametrize("n,m", [(2, 4), (1, 4), (2, 8), (2, 16), (7, 16), (4, 32), (16, 32), (4, 4)])
@pytest.mark.parametrize("shape", [(12, 20, 70, 64, 96, 3, 3, 1, 1), (140, 17, 19, 64, 96, 5, 5, 2, 2)])
def test_tiled_on_every_ranker(shape, n, m, ranker):
    """bwd_tiled: an image wider than the line kernel takes, with fewer than 128 tiles of 256 and C_out no multiple of 64; a strided filter
    that is wider than twice its stride."""
    check(shape, n, m, ranker)


@pytest.mark.parametrize("n,m,ranker", [(2, 4, oracle.RANDOM), (2, 16, oracle.GREEDY_ADJUSTED), (5, 8, oracle.GREEDY), (16, 32, oracle.RANDOM),
                                        (4, 4, oracle.GREEDY)])
@pytest.mark.parametrize("shape", [(4500, 1, 1, 64, 448, 3, 3, 2, 1), (3000, 1, 4, 72, 416, 3, 3, 2, 1), (2000, 5, 1, 64, 448, 3, 3, 2, 1),
                                   (1528, 26, 1, 40, 64, 7, 7, 2, 3)])
def test_strided_images_one_pixel_wide_or_high(shape, n, m, ranker):
    """bwd_tiled where some parity classes have no pixel.  The halo such a class would have is larger than what the tile was chosen
    for, and once counted it sent these layers back as not supported."""
    check(shape, n, m, ranker)


@pytest.mark.parametrize("shape,n,m,ranker", [
    ((1, 9, 9, 8, 24, 3, 3, 3, 1), 4, 4, oracle.GREEDY),        # stride 3: no tap reaches row and column 8
    ((2, 9, 10, 136, 24, 3, 3, 3, 1), 2, 8, oracle.GREEDY_ADJUSTED),
    ((2, 13, 9, 24, 40, 7, 7, 4, 3), 2, 4, oracle.GREEDY),
    ((2, 8, 8, 16, 32, 3, 3, 2, 1), 3, 4, oracle.RANDOM),
    ((2, 7, 7, 24, 64, 3, 3, 1, 1), 4, 32, oracle.RANDOM),
    ((1, 9, 9, 8, 16, 9, 9, 1, 4), 2, 16, oracle.GREEDY),       # 81 taps
])
def test_non_finite_weights_outside_the_gradient(shape, n, m, ranker):
    """A tap outside the gradient has no term: a weight there that is infinite or NaN must not reach the pixel.  Every
    gradient value is positive, so the oracle's NaN and infinities are those of the taps inside."""
    L = wl.ConvLayer("i", *shape)
    dO = wl.f32_to_bf16_bits(np.random.default_rng(3).uniform(1, 2, L.dO_shape).astype(np.float32))
    W = wl.normal(L.W_shape, 0.1, 4, wl.BF16)
    W[:, 0, 0, 1::2] = 0x7F80               # +inf: meets dropped values (zeros) too, which is a NaN by definition
    W[:, 0, 0, 4::8] = 0x7FC0               # NaN
    W[L.C_out // 2, L.R - 1, L.S // 2, 0] = 0xFF80
    ref, ab = oracle.conv_bwd_data(oracle.prune(dO, n, m, ranker, seed=9)[0], W, L.H, L.Wd, L.stride, L.pad)
    got = wl.to_f64(to_host(sdgp.sdgp_conv_bwd_data(to_gpu(dO), to_gpu(W), L.H, L.Wd, L.stride, L.pad, n, m, ranker, 9)))
    fin = np.isfinite(ref)
    assert fin.any() and not fin.all()
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(got[~fin & ~np.isnan(ref)], ref[~fin & ~np.isnan(ref)])
    assert np.all(np.abs(got[fin] - ref[fin]) <= 5e-3 * ab[fin])


def test_infinite_weight_outside_the_image_forward():
    """The forward pass of a 9x9 layer (81 taps) goes through the same kernel with the channels exchanged."""
    D = torch.ones(1, 12, 12, 32, dtype=torch.bfloat16, device="cuda")
    W = torch.ones(16, 9, 9, 32, dtype=torch.bfloat16, device="cuda")
    W[5, 0, 0] = float("inf")               # pad 4: outside for the first four output rows and columns
    out = sdgp.sdgp_conv_fwd(D, W, 1, 4).float().cpu()
    inside = torch.isposinf(out[..., 5])
    assert inside[:, 4:, 4:].all() and torch.isfinite(out[:, :4]).all() and torch.isfinite(out[:, :, :4]).all()
    assert out[0, 0, 0, 5] == 32 * 25


@pytest.mark.parametrize("shape", [
    (220, 9, 9, 64, 256, 3, 3, 3, 1),       # stride 3, 558 tiles (a parity class of 62 is too small for the pointwise kernel)
    (36, 16, 16, 8, 128, 9, 9, 1, 4),       # 81 taps, 288 tiles
])
def test_left_by_the_tile_kernels(shape):
    """Strides beyond two and filters beyond 49 taps, which only the plain kernel takes otherwise."""
    check(shape, 2, 4, oracle.GREEDY)
    L = wl.ConvLayer("s", *shape)
    dO, W = to_gpu(wl.laplace_with_zeros(L.dO_shape, 1e-3, 0.3, 5, wl.BF16)), to_gpu(wl.normal(L.W_shape, 0.1, 6, wl.BF16))
    begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    begin.record()
    for _ in range(5):
        sdgp.sdgp_conv_bwd_data(dO, W, L.H, L.Wd, L.stride, L.pad, 2, 4, sdgp.GREEDY)
    end.record()
    end.synchronize()
    assert begin.elapsed_time(end) / 5 < 0.6   # ms; 0.02 and 0.12 here, 1.3 and 6 on the plain kernel
