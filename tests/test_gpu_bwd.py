"""GPU parity of sdgp_linear_bwd_data / sdgp_conv_bwd_data against the CPU oracle.

Tolerance (stated by the benchmark spec): max |gpu - ref| / sum_k |dO_k||W_k| <= 1e-2 for bf16 storage with fp32
accumulation, <= 1e-5 for fp32.  The oracle prunes, then multiplies in fp64.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2202_00774_amd as sdgp
from paper_2202_00774_amd import workloads as wl
from util import rel_error, to_gpu, to_host

pytestmark = pytest.mark.gpu

TOL = {oracle.BF16: 1e-2, oracle.F32: 1e-5}
RANKERS = (oracle.RANDOM, oracle.GREEDY, oracle.GREEDY_ADJUSTED)


def got_f64(t):
    return wl.to_f64(to_host(t))


def check_linear(dO, W, n, m, ranker, seed, dtype):
    pruned = oracle.prune(dO, n, m, ranker, seed=seed)[0]
    ref, ab = oracle.linear_bwd_data(pruned, W)
    d = to_gpu(dO)
    keep = d.clone()
    out = sdgp.sdgp_linear_bwd_data(d, to_gpu(W), n, m, ranker, seed)
    torch.cuda.synchronize()
    assert torch.equal(d.view(torch.uint8), keep.view(torch.uint8))
    err = rel_error(got_f64(out), ref, ab)
    assert err <= TOL[dtype], err
    return err


def check_conv(layer, dO, W, n, m, ranker, seed, dtype, pixels=None):
    pruned = oracle.prune(dO, n, m, ranker, seed=seed)[0]
    ref, ab = oracle.conv_bwd_data(pruned, W, layer.H, layer.Wd, layer.stride, layer.pad, pixels=pixels)
    out = sdgp.sdgp_conv_bwd_data(to_gpu(dO), to_gpu(W), layer.H, layer.Wd, layer.stride, layer.pad, n, m, ranker, seed)
    torch.cuda.synchronize()
    if pixels is not None:
        out = out.reshape(-1, layer.C_in)[torch.from_numpy(pixels).to(out.device)]  # sample before the copy to the host
    got = got_f64(out)
    err = rel_error(got, ref, ab)
    assert err <= TOL[dtype], (layer.name, n, m, ranker, err)
    # pixels that no tap reaches must be exactly zero
    assert np.all(got[ab == 0] == 0)
    return err


# ------------------------------------------------------------------ linear

def test_config1_linear_fp32():
    dO, W = wl.linear_config1()
    for n, m in ((2, 4), (4, 4)):
        check_linear(dO, W, n, m, oracle.GREEDY, 0, oracle.F32)


@pytest.mark.parametrize("ranker", RANKERS)
@pytest.mark.parametrize("dtype", [oracle.BF16, oracle.F32])
@pytest.mark.parametrize("n,m", [(2, 4), (2, 8), (2, 16), (4, 8), (4, 4), (1, 4), (4, 32)])
def test_linear_matches_oracle(ranker, dtype, n, m):
    rows, C_out, C_in = 300, 32 * 5, 136          # several tiles with ragged edges in every dimension
    dO = wl.laplace_with_zeros((rows, C_out), 1e-3, 0.3, seed=5 + m, dtype=dtype)
    W = wl.normal((C_out, C_in), 0.1, 6 + m, dtype)
    check_linear(dO, W, n, m, ranker, 99, dtype)


def test_linear_hand_example():
    dO = torch.tensor([[1.0, 7.0, -3.0, 2.0]], device="cuda")
    W = torch.tensor([[1.0, 0.0], [0.0, 1.0], [1.0, 1.0], [2.0, -1.0]], device="cuda")
    assert sdgp.sdgp_linear_bwd_data(dO, W, 4, 4, sdgp.GREEDY).cpu().tolist() == [[2.0, 2.0]]
    assert sdgp.sdgp_linear_bwd_data(dO, W, 2, 4, sdgp.GREEDY).cpu().tolist() == [[-3.0, 4.0]]


def test_linear_classifier_shape():
    """The 2048 -> 1000 classifier of ResNet-50: 1000 output channels is a multiple of 4 and 8 but not of 16."""
    dO = wl.laplace_with_zeros((64, 1000), 1e-3, 0.3, seed=1, dtype=oracle.BF16)
    W = wl.normal((1000, 2048), 0.03, 2, oracle.BF16)
    for n, m in ((2, 4), (2, 8), (8, 8)):
        check_linear(dO, W, n, m, oracle.RANDOM, 53, oracle.BF16)
    with pytest.raises(sdgp.SdgpError):
        sdgp.sdgp_linear_bwd_data(to_gpu(dO), to_gpu(W), 2, 16, sdgp.GREEDY)


def test_linear_with_few_input_features():
    """A linear layer with three input features takes the first-layer kernel (one-pixel images)."""
    dO = wl.laplace_with_zeros((300, 64), 1e-3, 0.3, seed=31, dtype=oracle.BF16)
    W = wl.normal((64, 3), 0.2, 32, oracle.BF16)
    for n, m, ranker in ((2, 4, oracle.GREEDY), (2, 8, oracle.RANDOM), (4, 4, oracle.GREEDY)):
        check_linear(dO, W, n, m, ranker, 5, oracle.BF16)


# -------------------------------------------------------------------- conv

SMALL_CONVS = [
    wl.ConvLayer("c3x3", 3, 12, 10, 16, 32, 3, 3, 1, 1),
    wl.ConvLayer("c3x3_wide", 2, 9, 9, 72, 64, 3, 3, 1, 1),
    wl.ConvLayer("c3x3_cin3", 2, 16, 16, 3, 64, 3, 3, 1, 1),
    wl.ConvLayer("c1x1", 2, 14, 14, 48, 64, 1, 1, 1, 0),
    wl.ConvLayer("c3x3s2", 2, 14, 14, 32, 32, 3, 3, 2, 1),
    wl.ConvLayer("c1x1s2", 2, 14, 14, 32, 64, 1, 1, 2, 0),
    wl.ConvLayer("c7x7s2", 1, 30, 30, 3, 64, 7, 7, 2, 3),
    wl.ConvLayer("c4x4img", 20, 4, 4, 64, 64, 3, 3, 1, 1),
    wl.ConvLayer("c7x7img", 5, 7, 7, 64, 64, 3, 3, 1, 1),
    wl.ConvLayer("c5x3", 1, 11, 9, 8, 16, 5, 3, 1, 2),
    # few input channels: tap x channel columns on the matrix cores (one and two column tiles), ragged tiles,
    # a channel count that is not a multiple of the 64-channel pass, stride 2, a 1x1 filter
    wl.ConvLayer("c3x3_cin4", 2, 19, 21, 4, 72, 3, 3, 1, 1),
    wl.ConvLayer("c5x5_cin2", 2, 17, 16, 2, 32, 5, 5, 1, 2),
    wl.ConvLayer("c3x3s2_cin3", 2, 32, 32, 3, 136, 3, 3, 2, 1),
    wl.ConvLayer("c1x1_cin1", 3, 16, 16, 1, 16, 1, 1, 1, 0),
]


@pytest.mark.parametrize("layer", SMALL_CONVS, ids=lambda l: l.name)
@pytest.mark.parametrize("ranker", RANKERS)
@pytest.mark.parametrize("dtype", [oracle.BF16, oracle.F32])
def test_conv_matches_oracle(layer, ranker, dtype):
    dO, W = wl.layer_inputs(layer, 1e-3, 0.3, seed=42, dtype=dtype)
    for n, m in ((2, 4), (2, 8), (4, 4)):
        check_conv(layer, dO, W, n, m, ranker, 3, dtype)


@pytest.mark.parametrize("n,m,ranker", [(4, 4, oracle.GREEDY), (4, 8, oracle.GREEDY_ADJUSTED), (2, 4, oracle.RANDOM)])
@pytest.mark.parametrize("B,hw", [(2, 70), (148, 112)])
def test_stem_of_96_channels(B, hw, n, m, ranker):
    """The 7x7 stride-2 first layer with the filter's fragments through LDS (few tiles) and from the L2 (1184)."""
    layer = wl.ConvLayer("c7x7s2_96", B, hw, hw, 3, 96, 7, 7, 2, 3)
    dO, W = wl.layer_inputs(layer, 1e-3, 0.3, seed=44, dtype=oracle.BF16)
    hh = hw * hw
    pixels = np.unique(np.concatenate([np.array([0, hw - 1, hh - 1, B * hh - 1, B * hh - hw]), np.random.default_rng(5).integers(0, B * hh, 3000)]))
    check_conv(layer, dO, W, n, m, ranker, 3, oracle.BF16, pixels=pixels)


def test_conv_2_16_and_dense():
    layer = wl.ConvLayer("c3x3_k64", 2, 8, 8, 32, 64, 3, 3, 1, 1)
    dO, W = wl.layer_inputs(layer, 1e-3, 0.3, seed=43, dtype=oracle.BF16)
    for n, m in ((2, 16), (16, 16), (4, 16), (2, 32)):
        check_conv(layer, dO, W, n, m, oracle.GREEDY, 0, oracle.BF16)


# ------------------------------------------------- many-tile problems (the 512-row stride-1 kernel)
# Enough workgroups (>= 192 tiles of 512 rows) for the dispatcher to pick the eight-wavefront kernel.  The oracle
# prunes the whole gradient and evaluates a seeded sample of output pixels plus the corners of the batch.

MANY_TILE_CONVS = [
    wl.ConvLayer("w16_n64", 400, 16, 16, 64, 64, 3, 3, 1, 1),        # two images per tile, one 64-column tile
    wl.ConvLayer("w16_n136", 392, 16, 16, 136, 32, 3, 3, 1, 1),      # two 128-column tiles, the second one ragged
    wl.ConvLayer("w8", 1608, 8, 8, 16, 32, 3, 3, 1, 1),              # eight images per tile, batch not a multiple
    wl.ConvLayer("w30x28", 100, 30, 28, 8, 32, 3, 3, 1, 1),          # image split into tiles, odd sizes
    wl.ConvLayer("w16_valid", 400, 16, 16, 24, 32, 3, 3, 1, 0),      # no padding: the gradient is 14 x 14
    wl.ConvLayer("w2x2", 400, 16, 16, 8, 32, 2, 2, 1, 1),            # four taps
    wl.ConvLayer("w2x3", 400, 16, 16, 16, 64, 2, 3, 1, 1),           # two filter rows of three taps
    wl.ConvLayer("w16_r256_n64", 200, 16, 16, 64, 64, 3, 3, 1, 1),    # too few 512-row tiles: 256-row tiles, 64 columns
    wl.ConvLayer("w8_r256_n136", 808, 8, 8, 136, 32, 3, 3, 1, 1),     # 256-row tiles of four images, ragged second column tile
    wl.ConvLayer("w1x3", 400, 16, 16, 72, 32, 1, 3, 1, 0),           # one filter row, no padding; 72 columns of a 128-wide tile
]


def sample_pixels(layer, count, seed):
    total = layer.B * layer.H * layer.Wd
    rng = np.random.default_rng(seed)
    hw = layer.H * layer.Wd
    fixed = [0, layer.Wd - 1, hw - layer.Wd, hw - 1, total - hw, total - 1, total - layer.Wd]
    return np.unique(np.concatenate([np.array(fixed, dtype=np.int64), rng.integers(0, total, count)]))


@pytest.mark.parametrize("layer", MANY_TILE_CONVS, ids=lambda l: l.name)
def test_many_tile_conv_matches_oracle(layer):
    dO, W = wl.layer_inputs(layer, 1e-3, 0.3, seed=77, dtype=oracle.BF16)
    pixels = sample_pixels(layer, 700, 5)
    for n, m, ranker in ((4, 4, oracle.GREEDY), (2, 4, oracle.GREEDY), (2, 4, oracle.GREEDY_ADJUSTED),
                         (2, 4, oracle.RANDOM), (1, 4, oracle.GREEDY), (2, 8, oracle.GREEDY_ADJUSTED),
                         (2, 16, oracle.RANDOM), (2, 16, oracle.GREEDY),
                         # more than two survivors per group, or groups of 32: the pruned halo stored dense with zeros
                         (3, 4, oracle.GREEDY), (4, 8, oracle.RANDOM), (4, 16, oracle.GREEDY_ADJUSTED),
                         (16, 32, oracle.GREEDY), (2, 32, oracle.RANDOM)):
        check_conv(layer, dO, W, n, m, ranker, 11, oracle.BF16, pixels=pixels)


def test_many_tile_fused_equals_prune_then_dense():
    """The fused kernel and (standalone prune, then the dense kernel) see the same pruned values."""
    layer = wl.ConvLayer("w16_n128", 400, 16, 16, 128, 64, 3, 3, 1, 1)
    dO, W = wl.layer_inputs(layer, 1e-3, 0.3, seed=78, dtype=oracle.BF16)
    d, w = to_gpu(dO), to_gpu(W)
    for n, m, ranker in ((2, 4, sdgp.GREEDY), (2, 8, sdgp.GREEDY_ADJUSTED), (2, 4, sdgp.RANDOM)):
        pruned = sdgp.sdgp_prune(d, n, m, ranker, 21)[0]
        a = sdgp.sdgp_conv_bwd_data(pruned, w, layer.H, layer.Wd, 1, 1, m, m, sdgp.GREEDY, 0)
        b = sdgp.sdgp_conv_bwd_data(d, w, layer.H, layer.Wd, 1, 1, n, m, ranker, 21)
        torch.cuda.synchronize()
        diff = (a.float() - b.float()).abs().max().item()
        scale = a.float().abs().max().item()
        assert diff <= 2e-2 * scale, (n, m, ranker, diff, scale)


# ------------------------------------------------- 3x3 first layers (C_in <= 4): ragged tiles, one to four channels,
# several passes of 64 output channels, few and many tiles

FIRST_3X3 = [
    wl.ConvLayer("f3_rgb_32", 5, 32, 32, 3, 64, 3, 3, 1, 1),             # CIFAR shape
    wl.ConvLayer("f3_ragged", 2, 20, 36, 4, 128, 3, 3, 1, 1),            # ragged tiles both ways, two passes of 64 channels
    wl.ConvLayer("f3_gray_tiny", 3, 2, 2, 1, 64, 3, 3, 1, 1),            # one block per image
    wl.ConvLayer("f3_two_ch_wide", 1, 6, 70, 2, 192, 3, 3, 1, 1),        # three column tiles, the last ragged
    # 64 output channels on even images: the streaming kernel (a wavefront per strip of 32 columns and range of rows)
    wl.ConvLayer("f3_stream_strips", 2, 20, 36, 4, 64, 3, 3, 1, 1),      # two strips, the second four columns wide
    wl.ConvLayer("f3_stream_wide", 1, 6, 70, 2, 64, 3, 3, 1, 1),         # three strips, three block rows
    wl.ConvLayer("f3_stream_tall", 1, 64, 8, 3, 64, 3, 3, 1, 1),         # one strip, row ranges of four block rows
]
FIRST_3X3_MANY = [
    wl.ConvLayer("f3_rgb_32_many", 300, 32, 32, 3, 64, 3, 3, 1, 1),      # many tiles
    wl.ConvLayer("f3_ragged_many", 90, 40, 44, 4, 128, 3, 3, 1, 1),      # 3 x 2 tiles per image, ragged both ways
    wl.ConvLayer("f3_stream_many", 700, 24, 44, 3, 64, 3, 3, 1, 1),      # more wavefront tasks than the chip holds at once
]


@pytest.mark.parametrize("layer", FIRST_3X3, ids=lambda l: l.name)
@pytest.mark.parametrize("ranker", RANKERS)
def test_first_3x3_matches_oracle(layer, ranker):
    dO, W = wl.layer_inputs(layer, 1e-3, 0.3, seed=91, dtype=oracle.BF16)
    for n, m in ((2, 4), (4, 4), (1, 4), (3, 4), (2, 8), (2, 16), (4, 16)):
        check_conv(layer, dO, W, n, m, ranker, 17, oracle.BF16)


@pytest.mark.parametrize("layer", FIRST_3X3_MANY, ids=lambda l: l.name)
def test_first_3x3_many_tiles_sampled(layer):
    dO, W = wl.layer_inputs(layer, 1e-3, 0.3, seed=92, dtype=oracle.BF16)
    pixels = sample_pixels(layer, 3000, 9)
    for n, m, ranker in ((4, 4, oracle.GREEDY), (2, 4, oracle.GREEDY), (2, 4, oracle.GREEDY_ADJUSTED), (2, 4, oracle.RANDOM),
                         (2, 8, oracle.RANDOM), (4, 8, oracle.GREEDY), (2, 16, oracle.GREEDY_ADJUSTED)):
        check_conv(layer, dO, W, n, m, ranker, 23, oracle.BF16, pixels=pixels)


# ------------------------------------------------- gradient ranked and compressed ahead of the product
# 1x1 layers several column tiles wide and strided filters with C_out a multiple of 64 and n <= 2: a pass of its own
# writes kept values and positions to the workspace, and the product reads them (no ranking in the matrix kernel).

PRE_COMPRESSED = [
    wl.ConvLayer("pre_1x1_wide", 4, 13, 13, 2048, 128, 1, 1, 1, 0),      # ragged last row tile, 16 column tiles
    wl.ConvLayer("small_1x1_wide", 3, 13, 13, 2048, 128, 1, 1, 1, 0),    # a quarter fewer pixels: the small-problem kernel
    wl.ConvLayer("pre_1x1_s2", 5, 27, 27, 1024, 192, 1, 1, 2, 0),        # stride 2: three chunks of 64 channels
    wl.ConvLayer("pre_3x3s2", 44, 40, 40, 64, 128, 3, 3, 2, 1),          # four parity classes, one to four taps (the stride-2 kernel)
    wl.ConvLayer("pre_4x4s2", 44, 40, 40, 72, 64, 4, 4, 2, 1),           # four taps in every class, ragged column tile
]


@pytest.mark.parametrize("layer", PRE_COMPRESSED, ids=lambda l: l.name)
def test_pre_compressed_gradient_matches_oracle(layer):
    assert sdgp.conv_bwd_data_workspace(layer.B, layer.H, layer.Wd, layer.C_in, layer.C_out, layer.R, layer.S, layer.stride,
                                        layer.pad, sdgp.BF16, 2, 4) > 0
    dO, W = wl.layer_inputs(layer, 1e-3, 0.3, seed=61, dtype=oracle.BF16)
    pixels = sample_pixels(layer, 1500, 13)
    for n, m, ranker in ((2, 4, oracle.GREEDY), (2, 4, oracle.GREEDY_ADJUSTED), (2, 4, oracle.RANDOM), (1, 4, oracle.RANDOM),
                         (2, 8, oracle.GREEDY_ADJUSTED), (1, 8, oracle.GREEDY), (2, 16, oracle.RANDOM), (2, 16, oracle.GREEDY),
                         (4, 4, oracle.GREEDY), (3, 4, oracle.GREEDY)):      # the last two: dense and masked kernels, no pass
        check_conv(layer, dO, W, n, m, ranker, 29, oracle.BF16, pixels=pixels)


def test_pre_compressed_equals_fused():
    """With and without room for the compressed gradient the same kept values are multiplied (the entry point without
    a workspace runs the fused kernel when the arrays do not fit its scratch)."""
    layer = wl.ConvLayer("pre_1x1_big", 13, 13, 13, 2048, 128, 1, 1, 1, 0)    # 290 KB of arrays: more than the scratch
    assert sdgp.conv_bwd_data_workspace(13, 13, 13, 2048, 128, 1, 1, 1, 0, sdgp.BF16, 2, 4) > 256 * 1024
    dO, W = wl.layer_inputs(layer, 1e-3, 0.3, seed=62, dtype=oracle.BF16)
    d, w = to_gpu(dO), to_gpu(W)
    for n, m, ranker in ((2, 4, sdgp.RANDOM), (2, 8, sdgp.GREEDY_ADJUSTED)):
        a = sdgp.sdgp_conv_bwd_data(d, w, layer.H, layer.Wd, 1, 0, n, m, ranker, 5)
        b = torch.empty_like(a)
        sdgp.sdgp_conv_bwd_data_noalloc(d, w, layer.H, layer.Wd, 1, 0, n, m, ranker, 5, out=b)
        torch.cuda.synchronize()
        diff = (a.float() - b.float()).abs().max().item()
        assert diff <= 2e-2 * a.float().abs().max().item()


# ------------------------------------------------- full-size workload (the shapes and launches bench.py times)

@pytest.mark.parametrize("index", range(6))
def test_resnet9_batch512_sampled(index):
    """Every ResNet-9 layer at batch 512, in the launches bench.py times: the fused 2:4 kernels of the three rankers,
    2:8 and 2:16 Magnitude (the sparsity sweep on these shapes) and the dense kernel against the oracle on 4096 sampled
    output pixels (plus the corners of the first and last image); the oracle prunes the whole gradient."""
    layer = wl.resnet9_layers(512)[index]
    dO, W = wl.layer_inputs(layer, 1e-3, 0.3, seed=2000 + index, dtype=oracle.BF16)
    pixels = sample_pixels(layer, 4096, 100 + index)
    for n, m, ranker in ((2, 4, oracle.GREEDY), (2, 4, oracle.GREEDY_ADJUSTED), (2, 4, oracle.RANDOM), (2, 8, oracle.GREEDY),
                         (2, 16, oracle.GREEDY), (4, 4, oracle.GREEDY)):
        check_conv(layer, dO, W, n, m, ranker, 0, oracle.BF16, pixels=pixels)


@pytest.mark.parametrize("index", range(6))
def test_resnet50_bottleneck_batch128_sampled(index):
    """The bottleneck convolutions of ResNet-50 at 56x56 and 14x14, batch 128 (gradients of scale 1e-4 with 40 % zeros):
    2:4 greedy and greedy-adjusted, 2:8 and 2:16 greedy, and the dense kernel, on 4096 sampled output pixels."""
    layer = wl.resnet50_bottleneck_layers(128)[index]
    dO, W = wl.layer_inputs(layer, 1e-4, 0.4, seed=3000 + index, dtype=oracle.BF16)
    pixels = sample_pixels(layer, 4096, 200 + index)
    for n, m, ranker in ((2, 4, oracle.GREEDY), (2, 4, oracle.GREEDY_ADJUSTED), (2, 8, oracle.GREEDY),
                         (2, 16, oracle.GREEDY), (4, 4, oracle.GREEDY)):
        check_conv(layer, dO, W, n, m, ranker, 0, oracle.BF16, pixels=pixels)


def _resnet50_distinct_layers():
    """(index, layer) of the first layer of every distinct shape among the 54 layers of ResNet-50 at batch 256."""
    seen = {}
    for index, l in enumerate(wl.resnet50_all_layers(256)):
        seen.setdefault((l.H, l.Wd, l.C_in, l.C_out, l.R, l.S, l.stride, l.pad), (index, l))
    return list(seen.values())


@pytest.mark.parametrize("index,layer", _resnet50_distinct_layers(), ids=lambda v: v.name if hasattr(v, "name") else str(v))
def test_resnet50_batch256_every_layer_shape_sampled(index, layer):
    """Every distinct layer shape of the whole ResNet-50 at batch 256 and 224 x 224 input (stem 7x7 stride 2 with three
    input channels, stride-2 3x3 and 1x1 layers, 1x1 layers up to 2048 channels, 7x7 images, the classifier): random
    ranker seeded with the layer index at 2:4 and 2:8 and the dense kernel, per-layer gradient scale and zero fraction as
    drawn for the whole-network sweep, on 1024 sampled output pixels."""
    scale, zero_frac = wl.resnet50_layer_stats(index)
    dO, W = wl.layer_inputs(layer, scale, zero_frac, seed=5000 + index, dtype=oracle.BF16)
    pixels = sample_pixels(layer, 1024, 300 + index)
    for n, m in ((2, 4), (2, 8), (4, 4)):
        check_conv(layer, dO, W, n, m, oracle.RANDOM, index, oracle.BF16, pixels=pixels)


# ------------------------------------------------- pointwise kernel (1x1 convolutions and linear layers with many rows)

POINTWISE_CONVS = [
    wl.ConvLayer("pw_n264", 64, 23, 23, 264, 64, 1, 1, 1, 0),     # several column tiles, ragged rows and columns
    wl.ConvLayer("pw_n264_few_rows", 32, 16, 16, 264, 96, 1, 1, 1, 0),
    wl.ConvLayer("pw_n128", 128, 32, 32, 128, 32, 1, 1, 1, 0),    # one column tile, one reduction chunk
    wl.ConvLayer("pw_n24", 129, 16, 16, 24, 96, 1, 1, 1, 0),      # 24 live columns of a 64-column tile, ragged rows
    wl.ConvLayer("pw_s2", 64, 31, 29, 72, 64, 1, 1, 2, 0),        # stride 2, odd image: the last row and column stand alone
    wl.ConvLayer("pw_s3_n264", 160, 20, 22, 264, 32, 1, 1, 3, 0),  # stride 3, several column tiles
]


# strided filters wider than 1x1: one pointwise launch per parity class of the input pixels, rows gathered per tap
STRIDED_CONVS = [
    wl.ConvLayer("g_s2_3x3", 64, 30, 28, 72, 64, 3, 3, 2, 1),          # classes of 1, 2, 2 and 4 taps
    wl.ConvLayer("g_s2_3x3_n264", 96, 17, 19, 264, 32, 3, 3, 2, 1),    # odd image, several column tiles
    wl.ConvLayer("g_s2_4x4", 64, 32, 32, 64, 64, 4, 4, 2, 1),          # four taps in every class
    wl.ConvLayer("g_s2_3x3_valid", 64, 31, 31, 40, 32, 3, 3, 2, 0),    # no padding
    wl.ConvLayer("g_s3_3x3", 192, 30, 30, 32, 32, 3, 3, 3, 1),         # stride 3: nine classes of one tap
    wl.ConvLayer("g_s4_5x5", 512, 33, 31, 32, 32, 5, 5, 4, 2),         # stride 4: sixteen classes of 1, 2 or 4 taps, unequal sizes
]


@pytest.mark.parametrize("layer", STRIDED_CONVS, ids=lambda l: l.name)
def test_strided_conv_matches_oracle(layer):
    dO, W = wl.layer_inputs(layer, 1e-3, 0.3, seed=93, dtype=oracle.BF16)
    pixels = sample_pixels(layer, 2000, 9)
    for n, m, ranker in ((4, 4, oracle.GREEDY), (2, 4, oracle.GREEDY), (2, 4, oracle.GREEDY_ADJUSTED),
                         (2, 4, oracle.RANDOM), (2, 8, oracle.RANDOM), (2, 16, oracle.GREEDY),
                         (4, 8, oracle.GREEDY), (4, 8, oracle.RANDOM), (8, 32, oracle.GREEDY_ADJUSTED)):
        check_conv(layer, dO, W, n, m, ranker, 17, oracle.BF16, pixels=pixels)


@pytest.mark.parametrize("layer", POINTWISE_CONVS, ids=lambda l: l.name)
def test_pointwise_conv_matches_oracle(layer):
    dO, W = wl.layer_inputs(layer, 1e-3, 0.3, seed=91, dtype=oracle.BF16)
    pixels = sample_pixels(layer, 1500, 7)
    for n, m, ranker in ((4, 4, oracle.GREEDY), (2, 4, oracle.GREEDY), (2, 4, oracle.GREEDY_ADJUSTED),
                         (2, 4, oracle.RANDOM), (1, 4, oracle.GREEDY), (2, 8, oracle.RANDOM),
                         (2, 16, oracle.GREEDY_ADJUSTED), (2, 16, oracle.GREEDY),
                         # more than two survivors per group, or groups of 32: pruned rows stored dense with zeros
                         (3, 4, oracle.GREEDY), (4, 8, oracle.RANDOM), (4, 16, oracle.GREEDY_ADJUSTED),
                         (16, 32, oracle.GREEDY), (2, 32, oracle.RANDOM)):
        check_conv(layer, dO, W, n, m, ranker, 13, oracle.BF16, pixels=pixels)


def test_pointwise_linear_matches_oracle():
    rows, C_out, C_in = 40001, 64, 136
    dO = wl.laplace_with_zeros((rows, C_out), 1e-3, 0.3, seed=17, dtype=oracle.BF16)
    W = wl.normal((C_out, C_in), 0.1, 18, oracle.BF16)
    sample = np.unique(np.concatenate([np.array([0, rows - 1, rows - 2]), np.random.default_rng(3).integers(0, rows, 3000)]))
    d, w = to_gpu(dO), to_gpu(W)
    for n, m, ranker in ((2, 4, oracle.GREEDY), (2, 8, oracle.GREEDY_ADJUSTED), (2, 4, oracle.RANDOM), (4, 4, oracle.GREEDY)):
        pruned = oracle.prune(dO, n, m, ranker, seed=5)[0]
        ref, ab = oracle.linear_bwd_data(pruned[sample], W)
        out = sdgp.sdgp_linear_bwd_data(d, w, n, m, ranker, 5)
        torch.cuda.synchronize()
        err = rel_error(got_f64(out)[sample], ref, ab)
        assert err <= TOL[oracle.BF16], (n, m, ranker, err)
