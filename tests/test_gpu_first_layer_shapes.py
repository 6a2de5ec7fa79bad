"""First layers (up to four input channels) against the CPU oracle: pruned in groups of 32, on the 7x7 stem and on sizes and
filters it does not fit, with and without the workspace, which these calls can do without; the stem on odd image sizes.

Tolerance: the tests of the other bf16 kernels, 1e-2 of sum |a||w|."""
import numpy as np
import pytest
import torch

import oracle
import paper_2202_00774_amd as sdgp
from paper_2202_00774_amd import workloads as wl
from util import rel_error, to_gpu, to_host

pytestmark = pytest.mark.gpu

SHAPES = [(2, 36, 68, 3, 64, 7, 7, 2, 3), (2, 35, 33, 3, 64, 7, 7, 2, 3), (3, 20, 18, 3, 64, 3, 3, 1, 1), (3, 17, 21, 4, 96, 3, 3, 1, 1),
          (2, 12, 12, 1, 32, 5, 5, 1, 2)]


@pytest.mark.parametrize("ranker", (oracle.RANDOM, oracle.GREEDY, oracle.GREEDY_ADJUSTED))
@pytest.mark.parametrize("n", [1, 2, 4, 16, 31])
@pytest.mark.parametrize("shape", SHAPES)
def test_matches_oracle(shape, n, ranker):
    L = wl.ConvLayer("f", *shape)
    dO = wl.laplace_with_zeros(L.dO_shape, 1e-3, 0.3, seed=3 + n, dtype=wl.BF16)
    W = wl.normal(L.W_shape, 0.1, 4, wl.BF16)
    ref, ab = oracle.conv_bwd_data(oracle.prune(dO, n, 32, ranker, seed=11)[0], W, L.H, L.Wd, L.stride, L.pad)
    g, w = to_gpu(dO), to_gpu(W)
    out = sdgp.sdgp_conv_bwd_data(g, w, L.H, L.Wd, L.stride, L.pad, n, 32, ranker, 11)
    got = wl.to_f64(to_host(out))
    assert rel_error(got, ref, ab) <= 1e-2
    assert np.all(got[ab == 0] == 0)
    # none, and one too small to be written to
    small = torch.full((64,), 7, dtype=torch.uint8, device="cuda")
    for ptr, size in ((None, 0), (small.data_ptr(), 16)):
        bare = torch.empty_like(out)
        rc = sdgp.binding.load().sdgp_conv_bwd_data(g.data_ptr(), w.data_ptr(), bare.data_ptr(), L.B, L.H, L.Wd, L.C_in, L.C_out, L.R, L.S, L.stride,
                                                    L.pad, sdgp.BF16, n, 32, ranker, 11, ptr, size, torch.cuda.current_stream().cuda_stream)
        assert rc == 0
        assert rel_error(wl.to_f64(to_host(bare)), ref, ab) <= 1e-2
    assert torch.all(small == 7)
    sdgp.sdgp_conv_bwd_data_noalloc(g, w, L.H, L.Wd, L.stride, L.pad, n, 32, ranker, 11, bare)
    assert rel_error(wl.to_f64(to_host(bare)), ref, ab) <= 1e-2


@pytest.mark.parametrize("n,m,ranker", [(4, 4, oracle.GREEDY), (2, 4, oracle.RANDOM), (4, 8, oracle.GREEDY_ADJUSTED)])
@pytest.mark.parametrize("H,Wd", [(35, 33), (36, 65), (31, 66), (34, 36), (7, 9), (3, 2)])
@pytest.mark.parametrize("C_in", [1, 2, 3, 4])
def test_stem_on_odd_sizes(C_in, H, Wd, n, m, ranker):
    L = wl.ConvLayer("s", 2, H, Wd, C_in, 64, 7, 7, 2, 3)
    dO = wl.laplace_with_zeros(L.dO_shape, 1e-3, 0.3, seed=3 + n, dtype=wl.BF16)
    W = wl.normal(L.W_shape, 0.1, 4, wl.BF16)
    ref, ab = oracle.conv_bwd_data(oracle.prune(dO, n, m, ranker, seed=11)[0], W, H, Wd, 2, 3)
    g, w = to_gpu(dO), to_gpu(W)
    out = torch.full((2, H, Wd, C_in), float("nan"), dtype=torch.bfloat16, device="cuda")
    sdgp.sdgp_conv_bwd_data(g, w, H, Wd, 2, 3, n, m, ranker, 11, out=out)
    assert rel_error(wl.to_f64(to_host(out)), ref, ab) <= 1e-2


@pytest.mark.parametrize("n,m,ranker", [(4, 4, oracle.GREEDY), (2, 4, oracle.GREEDY), (1, 4, oracle.RANDOM), (3, 8, oracle.GREEDY),
                                        (2, 32, oracle.RANDOM), (5, 32, oracle.GREEDY)])
@pytest.mark.parametrize("shape", [(2, 35, 33, 3, 64, 7, 7, 2, 3), (2, 36, 68, 3, 96, 7, 7, 2, 3), (2, 37, 36, 4, 96, 7, 7, 2, 3), (2, 24, 36, 3, 64, 3, 3, 1, 1),
                                   (2, 17, 21, 4, 96, 3, 3, 1, 1)])
def test_non_finite_stay_with_their_taps(shape, n, m, ranker):
    """An infinite or NaN gradient value reaches the pixels that a tap joins to it, a weight those whose tap lies inside the
    gradient, and no others.  Every other value is positive, so the oracle's NaN and infinities are those of these terms."""
    L = wl.ConvLayer("n", *shape)
    rng = np.random.default_rng(5)
    dO = wl.f32_to_bf16_bits(rng.uniform(1, 2, L.dO_shape).astype(np.float32))
    W = wl.f32_to_bf16_bits(rng.uniform(0.5, 1, L.W_shape).astype(np.float32))
    P, Q = L.dO_shape[1:3]
    dO[0, P // 2, Q // 2, 1] = 0x7F80
    dO[0, 1, 2, 40:44] = 0x7FC0
    dO[0, P - 1, Q - 2, 3] = 0xFF80
    dO[0, 0, Q - 1, 5] = 0x7F80
    W[7, 0, 1, 0] = 0x7F80         # meets dropped values (zeros) too, which is a NaN by definition
    W[2, L.R - 1, 0, L.C_in - 1] = 0x7FC0
    ref, ab = oracle.conv_bwd_data(oracle.prune(dO, n, m, ranker, seed=11)[0], W, L.H, L.Wd, L.stride, L.pad)
    fin, nan = np.isfinite(ref), np.isnan(ref)
    assert fin.any() and nan.any() and (~fin & ~nan).any()
    g, w = to_gpu(dO), to_gpu(W)
    got = wl.to_f64(to_host(sdgp.sdgp_conv_bwd_data(g, w, L.H, L.Wd, L.stride, L.pad, n, m, ranker, 11)))
    assert np.array_equal(np.isnan(got), nan) and np.array_equal(got[~fin & ~nan], ref[~fin & ~nan])
    assert np.all(np.abs(got[fin] - ref[fin]) <= 1e-2 * ab[fin])


@pytest.mark.parametrize("n,m,ranker", [(4, 4, sdgp.GREEDY), (2, 4, sdgp.RANDOM), (2, 4, sdgp.GREEDY_ADJUSTED), (4, 32, sdgp.RANDOM), (4, 32, sdgp.GREEDY)])
@pytest.mark.parametrize("shape", [(32, 111, 111, 3, 64, 7, 7, 2, 3), (64, 64, 64, 3, 64, 3, 3, 1, 1)])
def test_nan_gradients_cost_no_more(shape, n, m, ranker):
    """A diverged step's gradient: a NaN under a pixel's own taps leaves nothing to sum again."""
    L = wl.ConvLayer("d", *shape)
    W = torch.full(L.W_shape, 0.01, dtype=torch.bfloat16, device="cuda")

    def run(value):
        dO = torch.full(L.dO_shape, value, dtype=torch.bfloat16, device="cuda")
        best = 1e9
        for _ in range(3):
            begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            begin.record()
            for _ in range(5):
                out = sdgp.sdgp_conv_bwd_data(dO, W, L.H, L.Wd, L.stride, L.pad, n, m, ranker)
            end.record()
            end.synchronize()
            best = min(best, begin.elapsed_time(end))
        return best, out

    finite, _ = run(1.0)
    nan, out = run(float("nan"))
    assert out.isnan().all()
    assert nan < 3 * finite, (nan, finite)
