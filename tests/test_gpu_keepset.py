"""The kept set and the kept values of the FUSED kernels, bit for bit (Sec. III-B; Alg. 1).

Inside the fused backward-data kernels the pruned gradient exists only in LDS, so a product with a general filter
shows it only through sums of hundreds of terms.  Here the filter is one-hot -- every output channel k of the
gradient feeds exactly one (tap, input channel) with weight 1 -- and, where more than one tap is used, the gradient is
nonzero only on a lattice of pixels whose footprints do not overlap.  Every element of dL/dD is then a single term
x * 1 (or nothing), so it must EQUAL the oracle's pruned value: a wrong survivor, a wrong tie decision, a wrong
position code or a wrong rescaled value changes bits of the output.

Values are finite and normal (signed zeros included; a kept -0 comes out as a zero of either sign, which compares
equal): half the rows Laplace with 30 % zeros, half drawn from a small alphabet so that equal magnitudes meet in
every position of a group.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2202_00774_amd as sdgp
from paper_2202_00774_amd import workloads as wl
from util import to_gpu, to_host

pytestmark = pytest.mark.gpu

RANKERS = (oracle.RANDOM, oracle.GREEDY, oracle.GREEDY_ADJUSTED)
ONE = np.uint16(0x3F80)
# +-0, the smallest normal and its neighbour, +-1, 1.5, +-2, +-2^97: repeats of a magnitude with both signs
ALPHABET = np.array([0x0000, 0x8000, 0x0080, 0x8080, 0x0081, 0x3F80, 0xBF80, 0x3FC0, 0x4000, 0xC000, 0x7000, 0xF000],
                    np.uint16)


def one_hot_filter(layer, spread):
    """W [C_out, R, S, C_in] with a single 1 per output channel.  spread=False: channel k -> (centre tap, k)
    (needs C_in == C_out); spread=True: channel k -> (tap k mod R*S, input channel k div R*S)."""
    W = np.zeros(layer.W_shape, np.uint16)
    T = layer.R * layer.S
    for k in range(layer.C_out):
        if spread:
            tap, c = k % T, k // T
        else:
            tap, c = (layer.R // 2) * layer.S + layer.S // 2, k
        assert c < layer.C_in
        W[k, tap // layer.S, tap % layer.S, c] = ONE
    return W


def gradient(layer, seed, lattice):
    """Half Laplace rows, half alphabet rows; with lattice > 1 only pixels (p, q) = (1, 1) mod lattice are nonzero."""
    shape = layer.dO_shape
    rng = np.random.Generator(np.random.PCG64(seed))
    dO = wl.laplace_with_zeros(shape, 1e-3, 0.3, seed, wl.BF16)
    alpha = rng.choice(ALPHABET, size=shape)
    pick = rng.random(size=shape[:3]) < 0.5
    dO[pick] = alpha[pick]
    if lattice > 1:
        mask = np.zeros(shape[:3], bool)
        mask[:, 1 % shape[1]::lattice, 1 % shape[2]::lattice] = True
        dO[~mask] = 0
    return dO


def sample(layer, count, seed):
    total = layer.B * layer.H * layer.Wd
    if total <= count:
        return np.arange(total, dtype=np.int64)
    hw = layer.H * layer.Wd
    fixed = np.array([0, layer.Wd - 1, hw - layer.Wd, hw - 1, total - hw, total - 1, total - layer.Wd], np.int64)
    return np.unique(np.concatenate([fixed, np.random.default_rng(seed).integers(0, total, count)]))


def check_exact(layer, spread, settings, npix=12000):
    lattice = 1
    if spread:
        lattice = max(-(-layer.R // layer.stride), -(-layer.S // layer.stride))  # footprints must not overlap
    dO = gradient(layer, 4242 + layer.C_out + layer.H, lattice)
    W = one_hot_filter(layer, spread)
    pixels = sample(layer, npix, 17)
    d, w = to_gpu(dO), to_gpu(W)
    for n, m, ranker in settings:
        pruned = oracle.prune(dO, n, m, ranker, seed=29)[0]
        ref, ab = oracle.conv_bwd_data(pruned, W, layer.H, layer.Wd, layer.stride, layer.pad, pixels=pixels)
        # single-term sums: the reference is exactly a stored value
        assert np.array_equal(ref, wl.to_f64(wl.f32_to_bf16_bits(ref.astype(np.float32))))
        out = sdgp.sdgp_conv_bwd_data(d, w, layer.H, layer.Wd, layer.stride, layer.pad, n, m, ranker, 29)
        torch.cuda.synchronize()
        got = wl.to_f64(to_host(out.reshape(-1, layer.C_in)[torch.from_numpy(pixels).to(out.device)]))
        bad = np.argwhere(got != ref)
        assert bad.size == 0, (layer.name, spread, n, m, ranker, len(bad), bad[:4].tolist(),
                               [(got[tuple(i)], ref[tuple(i)]) for i in bad[:4]])
        assert np.count_nonzero(ref) > 0


def nm_settings(ms=(4, 8, 16)):
    return [(2, m, r) for m in ms for r in RANKERS] + [(1, 4, oracle.GREEDY), (1, 8, oracle.RANDOM)]


# (layer, spread): which kernel the dispatcher picks for it is noted per case
CASES = [
    # line kernel: 64 and 128 columns, few and many lines and images a tile (the names are those of the row kernel's tiles, which took
    # these layers before; the wide images are its own)
    (wl.ConvLayer("row512_n64_wide", 30, 20, 70, 64, 64, 3, 3, 1, 1), False),
    (wl.ConvLayer("row512_n128_wide_spread", 30, 20, 70, 128, 128, 3, 3, 1, 1), True),
    (wl.ConvLayer("row512_n64", 400, 16, 16, 64, 64, 3, 3, 1, 1), False),
    (wl.ConvLayer("row512_n128", 400, 16, 16, 128, 128, 3, 3, 1, 1), False),
    (wl.ConvLayer("row512_n128_spread", 400, 16, 16, 128, 128, 3, 3, 1, 1), True),
    (wl.ConvLayer("row256_n64", 200, 16, 16, 64, 64, 3, 3, 1, 1), False),
    (wl.ConvLayer("row512_8x8_n128", 1608, 8, 8, 128, 128, 3, 3, 1, 1), True),
    # pointwise kernel: 256 x 64 tiles, all of C_in (160 of 256 columns) per workgroup
    (wl.ConvLayer("pw_n64", 64, 23, 23, 64, 64, 1, 1, 1, 0), False),
    (wl.ConvLayer("pw_n160", 64, 23, 23, 160, 160, 1, 1, 1, 0), False),
    (wl.ConvLayer("pw_s2_n64", 64, 31, 29, 64, 64, 1, 1, 2, 0), False),
    # pointwise kernel gathering rows per tap, stride-2 3x3 (classes of 1, 2, 2, 4 taps) and 4x4; stride-2 kernel
    (wl.ConvLayer("stride2_n128_spread", 64, 56, 54, 128, 128, 3, 3, 2, 1), True),
    (wl.ConvLayer("gather_s2_3x3", 64, 30, 28, 64, 64, 3, 3, 2, 1), True),
    (wl.ConvLayer("gather_s2_4x4", 64, 32, 32, 64, 64, 4, 4, 2, 1), True),
    # between the small-problem kernel's 256 tiles of 32 rows and the row kernel's 128 of 256: the line kernel, 5x5 the producer/consumer
    # kernel
    (wl.ConvLayer("conv3_n64", 40, 16, 16, 64, 64, 3, 3, 1, 1), False),
    (wl.ConvLayer("conv3_n64_spread", 40, 16, 16, 64, 64, 3, 3, 1, 1), True),
    (wl.ConvLayer("conv3_5x5", 72, 12, 12, 64, 64, 5, 5, 1, 2), True),
    # channel count not a multiple of 32: the line kernel; stride 2 below the pointwise classes' 64 tiles of 128 rows: the stride-2 kernel
    (wl.ConvLayer("tiled_n48", 66, 16, 16, 48, 48, 3, 3, 1, 1), False),
    (wl.ConvLayer("tiled_n48_spread", 66, 16, 16, 48, 48, 3, 3, 1, 1), True),
    (wl.ConvLayer("tiled_s2", 90, 14, 14, 32, 32, 3, 3, 2, 1), True),
    # images wider than the line kernel takes, fewer than 128 tiles of 256: the producer/consumer kernel, and the tiled one where C_out is
    # no multiple of 64; a strided filter wider than twice its stride: the tiled one too
    (wl.ConvLayer("conv3_n64_wide", 12, 20, 70, 64, 64, 3, 3, 1, 1), False),
    (wl.ConvLayer("conv3_n64_wide_spread", 12, 20, 70, 64, 64, 3, 3, 1, 1), True),
    (wl.ConvLayer("tiled_n48_wide", 12, 20, 70, 48, 48, 3, 3, 1, 1), False),
    (wl.ConvLayer("tiled_n48_wide_spread", 12, 20, 70, 48, 48, 3, 3, 1, 1), True),
    (wl.ConvLayer("tiled_5x5s2", 140, 17, 19, 64, 64, 5, 5, 2, 2), True),
    # the small-problem kernel: 3x3, 5x5, stride 2, a channel count that ends inside a reduction step, and 1x1
    (wl.ConvLayer("small_n64", 4, 16, 16, 64, 64, 3, 3, 1, 1), False),
    (wl.ConvLayer("small_n64_spread", 4, 16, 16, 64, 64, 3, 3, 1, 1), True),
    (wl.ConvLayer("small_5x5", 3, 12, 12, 64, 64, 5, 5, 1, 2), True),
    (wl.ConvLayer("small_n48_spread", 4, 16, 16, 48, 48, 3, 3, 1, 1), True),
    (wl.ConvLayer("small_s2", 2, 14, 14, 32, 32, 3, 3, 2, 1), True),
    (wl.ConvLayer("small_1x1_n160", 9, 7, 7, 160, 160, 1, 1, 1, 0), False),
    # first-layer kernel (C_in <= 4): 3x3 on four channels, the 7x7 stride-2 stem on three
    (wl.ConvLayer("narrow_3x3", 2, 19, 21, 4, 32, 3, 3, 1, 1), True),
    (wl.ConvLayer("narrow_7x7s2", 2, 30, 30, 3, 64, 7, 7, 2, 3), True),
]


# The same on patterns that no structured-sparse instruction takes: the ranked rows are multiplied dense.  32 channels a
# group, and more than two survivors.
DENSE_ROWS = [
    (wl.ConvLayer("line_n128", 200, 16, 16, 128, 128, 3, 3, 1, 1), False),
    (wl.ConvLayer("line_n96_spread", 200, 16, 16, 96, 96, 3, 3, 1, 1), True),
    (wl.ConvLayer("row_n96_wide", 30, 20, 70, 96, 96, 3, 3, 1, 1), False),
    (wl.ConvLayer("tiled_n64", 70, 16, 16, 64, 64, 3, 3, 1, 1), False),        # between 512 tiles of 32 rows and 128 of 256: the line kernel
    (wl.ConvLayer("tiled_n64_wide", 12, 20, 70, 64, 64, 3, 3, 1, 1), False),   # the same, wider than the line kernel takes
    (wl.ConvLayer("tiled_n64_wide_spread", 12, 20, 70, 64, 64, 3, 3, 1, 1), True),
    (wl.ConvLayer("tiled_s2_n96", 400, 9, 9, 96, 96, 3, 3, 2, 1), False),      # classes of 25 to 16 pixels: the last has 50 tiles of 128 rows
    (wl.ConvLayer("small_n96", 4, 16, 16, 96, 96, 3, 3, 1, 1), False),
    (wl.ConvLayer("small_s2_n96", 3, 14, 14, 96, 96, 3, 3, 2, 1), False),
]


@pytest.mark.parametrize("layer,spread", DENSE_ROWS, ids=lambda v: v.name if hasattr(v, "name") else "")
def test_pruned_values_multiplied_dense_equal_the_oracle(layer, spread):
    check_exact(layer, spread, [(n, m, r) for n, m in ((3, 4), (4, 8), (4, 16), (2, 32), (16, 32)) for r in RANKERS], npix=4000)


@pytest.mark.parametrize("layer,spread", CASES, ids=lambda v: v.name if hasattr(v, "name") else "")
def test_fused_pruned_values_equal_the_oracle(layer, spread):
    ms = tuple(m for m in (4, 8, 16) if layer.C_out % m == 0)
    check_exact(layer, spread, nm_settings(ms))


def test_linear_identity_equals_the_oracle():
    """dD = prune(dO) @ I for a linear layer: the pointwise kernel on rows of one pixel."""
    rows, C = 40001, 96
    layer = wl.ConvLayer("linear_n96", rows, 1, 1, C, C, 1, 1, 1, 0)
    check_exact(layer, False, nm_settings(), npix=rows)


def test_padded_reduction_identity_equals_the_oracle():
    """C_out = 40 and 1000 are multiples of 8 but not of the kernel's 32-channel chunk: the last chunk's missing channels and
    filter rows are zeros, and the random ranker keeps indexing rows of C_out elements.  (The query still names the size of
    padded copies.)"""
    for rows, C in ((9001, 40), (3100, 1000)):
        layer = wl.ConvLayer("padded_n%d" % C, rows, 1, 1, C, C, 1, 1, 1, 0)
        assert sdgp.conv_bwd_data_workspace(rows, 1, 1, C, C, 1, 1, 1, 0, sdgp.BF16, 2, 4) >= 2 * rows * (-(-C // 32) * 32)
        check_exact(layer, False, [(2, 4, r) for r in RANKERS] + [(2, 8, oracle.RANDOM), (4, 4, oracle.GREEDY), (3, 8, oracle.GREEDY)],
                    npix=600)


def test_ragged_reduction_identity_on_few_tiles_equals_the_oracle():
    """The same channel counts on few rows: 1000 on the small-problem kernel, whose last reduction step ends inside."""
    for rows, C in ((900, 40), (300, 1000)):
        check_exact(wl.ConvLayer("small_n%d" % C, rows, 1, 1, C, C, 1, 1, 1, 0), False,
                    [(2, 4, r) for r in RANKERS] + [(2, 8, oracle.RANDOM), (4, 4, oracle.GREEDY), (3, 8, oracle.GREEDY)], npix=rows)


# The gradient ranked and compressed by a pass of its own, then multiplied without ranking (1x1 layers with several
# column tiles; the strided cases above take the same route): kept values and positions go through global memory.
RANKED_AHEAD = [
    (wl.ConvLayer("ahead_pw_n512", 16, 23, 23, 512, 512, 1, 1, 1, 0), 3000,
     [(2, 4, oracle.RANDOM), (2, 8, oracle.RANDOM), (2, 16, oracle.RANDOM), (1, 4, oracle.RANDOM), (2, 4, oracle.GREEDY_ADJUSTED)]),
    (wl.ConvLayer("ahead_pw_n1024", 8, 16, 16, 1024, 1024, 1, 1, 1, 0), 1000,
     [(2, 4, oracle.GREEDY), (2, 8, oracle.GREEDY_ADJUSTED), (2, 16, oracle.GREEDY), (2, 4, oracle.RANDOM)]),
]


@pytest.mark.parametrize("layer,npix,settings", RANKED_AHEAD, ids=lambda v: v.name if hasattr(v, "name") else "")
def test_ranked_ahead_pruned_values_equal_the_oracle(layer, npix, settings):
    assert sdgp.conv_bwd_data_workspace(layer.B, layer.H, layer.Wd, layer.C_in, layer.C_out, 1, 1, 1, 0, sdgp.BF16, 2, 4) > 0
    check_exact(layer, False, settings, npix=npix)


def test_streaming_first_layer_pruned_values_equal_the_oracle():
    """The streaming 3x3 first-layer kernel (64 output channels, four input channels): output channels 0..35 feed
    (tap k mod 9, input channel k div 9) with weight 1, channels 36..63 carry zeros in the gradient, and only pixels
    (1, 1) mod 3 are nonzero -- every dD element is one kept value or nothing."""
    layer = wl.ConvLayer("stream_3x3", 3, 20, 36, 4, 64, 3, 3, 1, 1)
    dO = gradient(layer, 911, 3)
    dO[..., 36:] = 0
    W = np.zeros(layer.W_shape, np.uint16)
    for k in range(36):
        W[k, (k % 9) // 3, (k % 9) % 3, k // 9] = ONE
    d, w = to_gpu(dO), to_gpu(W)
    for n, m, ranker in nm_settings() + [(4, 8, oracle.GREEDY), (3, 4, oracle.RANDOM), (4, 16, oracle.GREEDY_ADJUSTED)]:
        pruned = oracle.prune(dO, n, m, ranker, seed=29)[0]
        ref, _ = oracle.conv_bwd_data(pruned, W, layer.H, layer.Wd, 1, 1)
        out = sdgp.sdgp_conv_bwd_data(d, w, layer.H, layer.Wd, 1, 1, n, m, ranker, 29)
        torch.cuda.synchronize()
        got = wl.to_f64(to_host(out))
        assert np.array_equal(got, ref), (n, m, ranker, int(np.count_nonzero(got != ref)))
        assert np.count_nonzero(ref) > 0
