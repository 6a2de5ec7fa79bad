"""fp32 backward-data products on the fp32 matrix instruction against the CPU oracle, at the edges of its tiles:
rows and columns that are no multiple of a tile, an odd number of m-groups (half of the last reduction step is empty),
fewer reduction steps than wavefronts, every tile shape, strides whose parity classes have no tap.

Tolerance: fp32 products summed in fp32 over K terms err by at most K * 2^-24 of sum |a||w| each way; K <= 1152 here
gives 6.9e-5, rounding errors add up like sqrt(K) in practice, and the bound the fp32 tests use is 1e-5.
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


def check(layer, n, m, ranker, seed=11):
    dO = wl.laplace_with_zeros(layer.dO_shape, 1e-3, 0.3, seed=seed, dtype=wl.F32)
    W = wl.normal(layer.W_shape, 0.1, seed + 1, wl.F32)
    pruned = oracle.prune(dO, n, m, ranker, seed=seed)[0]
    ref, ab = oracle.conv_bwd_data(pruned, W, layer.H, layer.Wd, layer.stride, layer.pad)
    out = to_host(sdgp.sdgp_conv_bwd_data(to_gpu(dO), to_gpu(W), layer.H, layer.Wd, layer.stride, layer.pad, n, m, ranker, seed))
    assert rel_error(out, ref, ab) <= 1e-5
    assert np.all(out[ab == 0] == 0)


@pytest.mark.parametrize("ranker", RANKERS)
@pytest.mark.parametrize("n,m", [(2, 4), (1, 8), (5, 8), (2, 16), (7, 16), (1, 32), (16, 32), (4, 4), (7, 7)])
def test_groups(n, m, ranker):
    # three groups (28 channels for m = 7, which only the dense product takes): half of the last step is empty
    check(wl.ConvLayer("g", 2, 5, 6, 36, 28 if m == 7 else 3 * m, 3, 3, 1, 1), n, m, ranker)


@pytest.mark.parametrize("rows,C_in", [(32768 + 5, 132), (32768 + 5, 66), (33, 2), (1, 258), (32, 64)])
def test_tile_shapes(rows, C_in):
    check(wl.ConvLayer("t", rows, 1, 1, C_in, 24, 1, 1, 1, 0), 2, 4, oracle.GREEDY)


@pytest.mark.parametrize("H,Wd,R,S,stride,pad", [(9, 8, 3, 3, 2, 1), (7, 7, 1, 1, 3, 0), (8, 11, 2, 5, 3, 1), (13, 9, 7, 7, 4, 3),
                                                 (5, 5, 3, 3, 1, 0), (9, 9, 3, 1, 2, 0)])
def test_filters(H, Wd, R, S, stride, pad):
    check(wl.ConvLayer("f", 3, H, Wd, 34, 16, R, S, stride, pad), 2, 4, oracle.RANDOM)


@pytest.mark.parametrize("C_in", [70, 66, 3, 1])
def test_unfit_widths(C_in):
    """Widths the 8- and 16-byte weight loads suit and those they do not."""
    check(wl.ConvLayer("w", 2, 6, 6, C_in, 8, 3, 3, 1, 1), 2, 4, oracle.GREEDY)


@pytest.mark.parametrize("C_out,C_in,n,m", [(4, 2, 2, 4), (8, 2, 3, 4), (4, 6, 4, 4), (8, 4, 2, 8), (4, 8, 2, 4)])
def test_a_handful_of_channels(C_out, C_in, n, m):
    check(wl.ConvLayer("h", 3, 9, 9, C_in, C_out, 1, 1, 1, 0), n, m, oracle.GREEDY_ADJUSTED)


def test_unaligned_pointers():
    layer = wl.ConvLayer("u", 2, 4, 4, 8, 8, 1, 1, 1, 0)
    dO = wl.laplace_with_zeros(layer.dO_shape, 1.0, 0.3, seed=3, dtype=wl.F32)
    W = wl.normal(layer.W_shape, 0.1, 4, wl.F32)

    def shifted(a):
        t = torch.empty(a.size + 1, dtype=torch.float32, device="cuda")[1:]
        return t.copy_(torch.from_numpy(a.reshape(-1))).view(a.shape)
    ref, ab = oracle.conv_bwd_data(oracle.prune(dO, 2, 4, oracle.GREEDY)[0], W, 4, 4, 1, 0)
    out = to_host(sdgp.sdgp_conv_bwd_data(shifted(dO), shifted(W), 4, 4, 1, 0, 2, 4, oracle.GREEDY))
    assert rel_error(out, ref, ab) <= 1e-5


@pytest.mark.parametrize("B", [1, 700])
def test_infinite_weight_outside_the_image(B):
    """A tap outside the gradient has no term: an infinite weight there must not reach the pixel."""
    H = 7
    dO = np.ones((B, H, H, 8), dtype=np.float32)
    W = np.ones((8, 3, 3, 68), dtype=np.float32)
    W[:, 0, 0, :] = np.inf            # reaches input pixel (h, w) from gradient pixel (h + 1, w + 1)
    out = to_host(sdgp.sdgp_conv_bwd_data(to_gpu(dO), to_gpu(W), H, H, 1, 1, 8, 8, oracle.GREEDY))
    assert np.all(np.isposinf(out[:, :-1, :-1]))
    assert np.all(out[:, -1, 1:-1] == 8 * 6) and np.all(out[:, 1:-1, -1] == 8 * 6) and np.all(out[:, -1, -1] == 8 * 4)


@pytest.mark.parametrize("B", [8, 128])
def test_nan_gradients_cost_no_more(B):
    """A diverged step's gradient, on the tiles that share the reduction (batch 8) and on those that do not: no weight is
    non-finite, so nothing has to be summed again."""
    W = torch.full((64, 3, 3, 64), 0.01, device="cuda")

    def run(value):
        dO = torch.full((B, 32, 32, 64), value, device="cuda")
        best = 1e9
        for _ in range(3):
            begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            begin.record()
            for _ in range(5):
                out = sdgp.sdgp_conv_bwd_data(dO, W, 32, 32, 1, 1, 2, 4, sdgp.GREEDY)
            end.record()
            end.synchronize()
            best = min(best, begin.elapsed_time(end))
        return best, out

    finite, _ = run(1.0)
    nan, out = run(float("nan"))
    assert out.isnan().all()
    assert nan < 3 * finite, (nan, finite)


@pytest.mark.parametrize("shape,n,m,ranker", [
    ((1, 9, 9, 8, 24, 3, 3, 3, 1), 4, 4, oracle.GREEDY),
    ((2, 13, 9, 24, 40, 7, 7, 4, 3), 2, 8, oracle.GREEDY_ADJUSTED),
    ((2, 8, 8, 132, 32, 3, 3, 2, 1), 3, 4, oracle.RANDOM),
    ((900, 7, 7, 68, 32, 3, 3, 1, 1), 4, 32, oracle.RANDOM),     # one tile per wavefront
])
def test_non_finite_weights_outside_the_gradient(shape, n, m, ranker):
    """Every gradient value is positive, so the oracle's NaN and infinities are those of the taps inside."""
    L = wl.ConvLayer("i", *shape)
    dO = np.random.default_rng(3).uniform(1, 2, L.dO_shape).astype(np.float32)
    W = wl.normal(L.W_shape, 0.1, 4, wl.F32)
    W[:, 0, 0, 1::2] = np.inf
    W[:, 0, 0, 4::8] = np.nan
    W[L.C_out // 2, L.R - 1, L.S // 2, 0] = -np.inf
    ref, ab = oracle.conv_bwd_data(oracle.prune(dO, n, m, ranker, seed=9)[0], W, L.H, L.Wd, L.stride, L.pad)
    got = to_host(sdgp.sdgp_conv_bwd_data(to_gpu(dO), to_gpu(W), L.H, L.Wd, L.stride, L.pad, n, m, ranker, 9)).astype(np.float64)
    fin, nan = np.isfinite(ref), np.isnan(ref)
    assert fin.any() and not fin.all()
    assert np.array_equal(np.isnan(got), nan) and np.array_equal(got[~fin & ~nan], ref[~fin & ~nan])
    assert np.all(np.abs(got[fin] - ref[fin]) <= 1e-5 * ab[fin])
