"""fp32 backward-data products as sums of bf16 ones, on problems large enough to take that path, against the CPU oracle:
every shape of its tiles (tests/test_f32_split_host.py asks the planner that the layers here reach them), widths and channel
counts that fill none of them, classes without a tap, images laid together in a tile, every product of parts on its own, both
ends of fp32's range, non-finite operands, and the same call without a workspace.

Tolerance, of sum |a||w|: the products left out are within 2^-24 of a term; a sum of S steps (taps times chunks of channels) is
rounded S times by at most 2^-24 of itself, which add like their square root, at most 11 in the layers here; the sum of the
smaller products and the result add one each: 1e-6.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2202_00774_amd as sdgp
from paper_2202_00774_amd import workloads as wl
from util import rel_error, to_gpu, to_host

pytestmark = pytest.mark.gpu


def takes(layer, n, m):
    return sdgp.conv_bwd_data_workspace(layer.B, layer.H, layer.Wd, layer.C_in, layer.C_out, layer.R, layer.S, layer.stride, layer.pad,
                                        sdgp.F32, n, m) > 0


def run(layer, dO, W, n, m, ranker, seed):
    return to_host(sdgp.sdgp_conv_bwd_data(to_gpu(dO), to_gpu(W), layer.H, layer.Wd, layer.stride, layer.pad, n, m, ranker, seed))


# the layer, rows and grid positions of its tiles
SHAPES = [
    ((128, 16, 16, 64, 64, 3, 3, 1, 1), (128, 256)),
    ((30, 21, 19, 72, 36, 3, 3, 1, 1), (128, 256)),       # ragged tiles, columns and channels
    ((30, 16, 16, 256, 64, 3, 3, 1, 1), (128, 256)),
    ((40, 24, 24, 33, 64, 3, 3, 2, 1), (128, 256)),       # classes of one, two and four taps, an odd width
    ((400, 9, 9, 136, 100, 3, 3, 1, 1), (256, 384)),      # three images to a tile
    ((130, 16, 16, 136, 32, 3, 3, 1, 1), (256, 384)),
    ((24, 30, 30, 96, 64, 5, 5, 1, 2), (256, 384)),
    ((62, 29, 29, 33, 128, 1, 1, 2, 0), (256, 384)),      # classes without a tap, one tap: one stage to a chunk
    ((128, 16, 16, 160, 32, 5, 5, 1, 2), (256, 512)),     # compressed: one tap to a stage
    ((240, 8, 8, 200, 36, 3, 3, 1, 1), (256, 512)),       # four images to a tile
]
PATTERNS = [(2, 4, oracle.GREEDY), (1, 4, oracle.RANDOM), (2, 4, oracle.GREEDY_ADJUSTED), (4, 4, oracle.GREEDY), (3, 4, oracle.RANDOM)]


def compare(layer, n, m, ranker, pixels=None):
    """The largest error of the layer's results, of some pixels where the oracle would take long."""
    assert takes(layer, n, m)
    dO = wl.laplace_with_zeros(layer.dO_shape, 1e-3, 0.3, seed=5, dtype=wl.F32)
    W = wl.normal(layer.W_shape, 0.1, 6, wl.F32)
    count = layer.B * layer.H * layer.Wd
    at = np.arange(count) if pixels is None else np.sort(np.random.default_rng(2).choice(count, pixels, replace=False))
    ref, ab = oracle.conv_bwd_data(oracle.prune(dO, n, m, ranker, seed=7)[0], W, layer.H, layer.Wd, layer.stride, layer.pad, pixels=at)
    out = run(layer, dO, W, n, m, ranker, 7).reshape(count, layer.C_in)[at]
    ref, ab = ref.reshape(out.shape), ab.reshape(out.shape)
    assert np.all(out[ab == 0] == 0)
    return rel_error(out, ref, ab)


@pytest.mark.parametrize("n,m,ranker", PATTERNS)
@pytest.mark.parametrize("shape", [s for s, _ in SHAPES])
def test_shapes(shape, n, m, ranker):
    assert compare(wl.ConvLayer("s", *shape), n, m, ranker) <= 1e-6


@pytest.mark.parametrize("n,ranker", [(2, oracle.GREEDY), (1, oracle.RANDOM)])
def test_one_tap(n, ranker):
    """1x1 on several chunks: a grid lands as late as its only stage."""
    assert compare(wl.ConvLayer("o", 120, 17, 17, 448, 128, 1, 1, 1, 0), n, 4, ranker, pixels=6000) <= 1e-6


GROUP_LAYERS = [((64, 16, 16, 128, 96, 3, 3, 1, 1), (128, 256)), ((128, 16, 16, 128, 96, 3, 3, 1, 1), (256, 384)), ((240, 8, 8, 200, 96, 3, 3, 1, 1), (256, 512))]
GROUPS = [(3, 4), (2, 8), (5, 8), (1, 16), (7, 16), (2, 32), (16, 32)]


@pytest.mark.parametrize("ranker", (oracle.RANDOM, oracle.GREEDY, oracle.GREEDY_ADJUSTED))
@pytest.mark.parametrize("n,m", GROUPS)
@pytest.mark.parametrize("shape", [s for s, _ in GROUP_LAYERS])
def test_groups(shape, n, m, ranker):
    assert compare(wl.ConvLayer("g", *shape), n, m, ranker, pixels=4000) <= 1e-6


@pytest.mark.parametrize("n,m", [(2, 4), (4, 8)])
@pytest.mark.parametrize("shape", [s for s, _ in GROUP_LAYERS])
def test_non_finite(shape, n, m):
    """An infinite gradient value times a weight with few bits, dropped channels under an infinite weight, NaN."""
    layer = wl.ConvLayer("i", *shape)
    assert takes(layer, n, m)
    rng = np.random.default_rng(3)
    dO = rng.uniform(1, 2, layer.dO_shape).astype(np.float32)
    W = (rng.integers(1, 4, layer.W_shape) * 0.25).astype(np.float32)
    dO[3, 5, 7, 11] = np.inf
    dO[4, 0, 0, 2] = -np.inf
    dO[5, 1, 1, :4] = np.nan
    W[:, 0, 0, 5] = np.inf
    W[9, 2, 2, 40] = np.nan
    images = 8 * layer.H * layer.Wd
    ref, ab = oracle.conv_bwd_data(oracle.prune(dO, n, m, oracle.GREEDY)[0], W, layer.H, layer.Wd, 1, 1, pixels=np.arange(images))
    got = run(layer, dO, W, n, m, oracle.GREEDY, 0).astype(np.float64).reshape(-1, layer.C_in)[:images]
    ref, ab = ref.reshape(got.shape), ab.reshape(got.shape)
    fin, nan = np.isfinite(ref), np.isnan(ref)
    assert fin.any() and nan.any() and (~fin & ~nan).any()
    assert np.array_equal(np.isnan(got), nan) and np.array_equal(got[~fin & ~nan], ref[~fin & ~nan])
    assert np.all(np.abs(got[fin] - ref[fin]) <= 1e-6 * ab[fin])


def test_without_a_workspace():
    """The library's own entry point takes an fp32 problem without, with too small and with a misaligned workspace."""
    layer = wl.ConvLayer("w", 64, 16, 16, 128, 96, 3, 3, 1, 1)
    dO = to_gpu(wl.laplace_with_zeros(layer.dO_shape, 1e-3, 0.3, seed=1, dtype=wl.F32))
    W = to_gpu(wl.normal(layer.W_shape, 0.1, 2, wl.F32))
    need = sdgp.conv_bwd_data_workspace(64, 16, 16, 128, 96, 3, 3, 1, 1, sdgp.F32, 2, 4)
    want = sdgp.sdgp_conv_bwd_data(dO, W, 16, 16, 1, 1, 2, 4, sdgp.GREEDY)
    room = torch.empty(need + 16, dtype=torch.uint8, device="cuda")
    lib = sdgp.binding.load()
    for ptr, size in ((None, 0), (room.data_ptr(), need - 1), (room.data_ptr() + 4, need), (room.data_ptr(), need)):
        out = torch.empty(64, 16, 16, 128, device="cuda")
        rc = lib.sdgp_conv_bwd_data(dO.data_ptr(), W.data_ptr(), out.data_ptr(), 64, 16, 16, 128, 96, 3, 3, 1, 1, sdgp.F32, 2, 4, sdgp.GREEDY, 0,
                                    ptr, size, torch.cuda.current_stream().cuda_stream)
        assert rc == 0
        assert (out - want).norm() <= 1e-6 * want.norm()


@pytest.mark.parametrize("n,m,ranker", [(2, 4, oracle.GREEDY_ADJUSTED), (3, 4, oracle.RANDOM), (4, 4, oracle.GREEDY)])
@pytest.mark.parametrize("shape", [
    (32, 24, 25, 67, 64, 3, 1, 2, 0), (32, 24, 25, 33, 64, 2, 1, 2, 0), (32, 24, 25, 67, 64, 1, 3, 2, 0), (32, 24, 25, 33, 64, 2, 2, 3, 0),
    (32, 24, 24, 67, 96, 3, 3, 4, 1), (32, 24, 25, 33, 64, 2, 3, 4, 1), (32, 25, 24, 33, 64, 3, 2, 3, 1), (64, 25, 24, 33, 64, 1, 1, 3, 0),
    (64, 2, 97, 33, 64, 1, 2, 2, 0)])   # tiles of one row
def test_classes_without_taps(shape, n, m, ranker):
    """Filters narrower than the stride along one axis or both: classes without taps lie between those that have some."""
    layer = wl.ConvLayer("c", *shape)
    assert takes(layer, n, m)
    dO = wl.laplace_with_zeros(layer.dO_shape, 1e-3, 0.3, seed=15, dtype=wl.F32)
    W = wl.normal(layer.W_shape, 0.1, 16, wl.F32)
    ref, ab = oracle.conv_bwd_data(oracle.prune(dO, n, m, ranker, seed=17)[0], W, layer.H, layer.Wd, layer.stride, layer.pad)
    out = run(layer, dO, W, n, m, ranker, 17)
    assert rel_error(out, ref, ab) <= 1e-6
    assert np.all(out[ab == 0] == 0)


@pytest.mark.parametrize("n,m", [(2, 4), (3, 4), (4, 4)])
def test_every_product_counts(n, m):
    """One term to a result: an error of 2^-24 for the products left out, as much for each of the two sums and the result.  The
    smallest products that count are 2^-17 of the whole, and every result has its own."""
    layer = wl.ConvLayer("p", 128, 32, 32, 33, 32, 1, 1, 1, 0)
    assert takes(layer, n, m)
    rng = np.random.default_rng(31)
    dO = np.zeros(layer.dO_shape, np.float32).reshape(-1, 32)
    pixels = np.arange(dO.shape[0])
    dO[pixels, rng.integers(0, 32, pixels.size)] = rng.choice([-1, 1], pixels.size) * rng.uniform(1, 2, pixels.size)
    dO[::7, 3] += 2.0 ** -9 - 2.0 ** -23           # (some pixels have two terms)
    W = (rng.choice([-1, 1], layer.W_shape) * rng.uniform(1, 2, layer.W_shape)).astype(np.float32)
    W[:, 0, 0, ::3] = np.float32(1 + 2.0 ** -7 - 2.0 ** -23) * np.sign(W[:, 0, 0, ::3])   # the most that truncation loses
    dO = dO.reshape(layer.dO_shape)
    ref, ab = oracle.conv_bwd_data(oracle.prune(dO, n, m, oracle.GREEDY)[0], W, 32, 32, 1, 0)
    assert rel_error(run(layer, dO, W, n, m, oracle.GREEDY, 0), ref, ab) <= 4 * 2.0 ** -24


@pytest.mark.parametrize("n,m", [(2, 4), (4, 4)])
@pytest.mark.parametrize("grad,weight", [(1e-38, 1.0), (1e-36, 1e3), (1.0, 1e-38), (1e-30, 1e-7), (1e34, 1e-20), (1e-20, 1e34), (1e13, 1e13)])
def test_whole_range(grad, weight, n, m):
    """Operands and results next to both ends of fp32's range, subnormal ones among them, have the error of any others (and half
    the smallest step, of the result and of the terms of a sum)."""
    layer = wl.ConvLayer("r", 32, 24, 24, 33, 64, 3, 3, 1, 1)
    assert takes(layer, n, m)
    rng = np.random.default_rng(33)
    dO = (wl.laplace_with_zeros(layer.dO_shape, 1.0, 0.3, seed=33, dtype=wl.F32).astype(np.float64) * grad).astype(np.float32)
    W = (rng.normal(size=layer.W_shape) * weight).astype(np.float32)
    ref, ab = oracle.conv_bwd_data(oracle.prune(dO, n, m, oracle.GREEDY)[0], W, 24, 24, 1, 1)
    got = run(layer, dO, W, n, m, oracle.GREEDY, 0).astype(np.float64)
    assert np.all(np.isfinite(ref)) and np.all(np.abs(got - ref) <= 1e-6 * ab + 2.0 ** -149 * (1 + 9 * 64))


def test_without_room_for_a_workspace():
    """Where the device has no room for the operands' parts the binding makes the call without them, as before there were any."""
    layer = wl.ConvLayer("m", 512, 16, 16, 128, 96, 3, 3, 1, 1)   # 42 MB
    assert takes(layer, 2, 4)
    dO = to_gpu(wl.laplace_with_zeros(layer.dO_shape, 1e-3, 0.3, seed=1, dtype=wl.F32))
    W = to_gpu(wl.normal(layer.W_shape, 0.1, 2, wl.F32))
    want = sdgp.sdgp_conv_bwd_data(dO, W, 16, 16, 1, 1, 2, 4, sdgp.GREEDY)
    out = torch.zeros_like(want)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    torch.cuda.set_per_process_memory_fraction(1e-9)
    try:
        with pytest.raises(torch.OutOfMemoryError):
            torch.empty(1 << 26, dtype=torch.uint8, device="cuda")
        sdgp.sdgp_conv_bwd_data(dO, W, 16, 16, 1, 1, 2, 4, sdgp.GREEDY, out=out)
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert (out - want).norm() <= 1e-6 * want.norm()
