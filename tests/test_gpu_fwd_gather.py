"""The gathering forward kernel (any filter and stride, bf16, channels multiples of 8) against the oracle at the edges of
its tiles: pixels and output channels that end inside a tile, channel counts that end inside a 32-channel step, one step
in all, images a filter reaches past on every side.

Tolerance relative to sum |a||b|: one rounding of the result to bf16 (2^-9 of the value) and fp32 sums of K <= 1200 terms
(K * 2^-24 = 7e-5): 4e-3.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2202_00774_amd as sdgp
from paper_2202_00774_amd import workloads as wl
from util import to_gpu, to_host

pytestmark = pytest.mark.gpu

LAYERS = [  # B, H, Wd, C_in, C_out, R, S, stride, pad
    (3, 9, 7, 32, 64, 3, 3, 2, 1),
    (2, 17, 13, 40, 136, 3, 3, 2, 1),       # 40 channels: a full step and one of 8; a second column tile of 8
    (1, 1, 1, 8, 8, 1, 1, 1, 0),            # one pixel, one step
    (5, 16, 8, 64, 72, 1, 1, 2, 0),
    (2, 10, 11, 24, 64, 3, 3, 1, 1),        # stride 1 with channels the mirrored path does not take
    (2, 8, 8, 32, 128, 2, 3, 1, 1),
    (1, 9, 9, 48, 8, 5, 5, 3, 2),
    (2, 4, 3, 16, 200, 4, 4, 4, 3),
]


@pytest.mark.parametrize("shape", LAYERS)
def test_matches_oracle(shape):
    L = wl.ConvLayer("f", *shape)
    D, W = wl.normal(L.dD_shape, 1.0, 5, wl.BF16), wl.normal(L.W_shape, 0.1, 6, wl.BF16)
    ref, ab = oracle.conv_fwd(D, W, L.stride, L.pad)
    got = wl.to_f64(to_host(sdgp.sdgp_conv_fwd(to_gpu(D), to_gpu(W), L.stride, L.pad)))
    assert np.all(got[ab == 0] == 0)
    assert np.max(np.abs(got - ref)[ab > 0] / ab[ab > 0]) <= 4e-3


@pytest.mark.parametrize("shape", [
    (12, 113, 113, 40, 120, 3, 3, 2, 1),    # 305 tiles of 128 channels, four LDS buffers
    (12, 113, 113, 40, 136, 3, 3, 2, 1),    # 610, two buffers; a second column tile of 8 channels
    (21, 113, 115, 24, 40, 3, 3, 2, 1),     # 543 tiles of 64 channels, two buffers
    (12, 113, 113, 72, 200, 1, 1, 2, 0),    # three steps, the last of 8 channels
])
def test_larger_grids_match_oracle(shape):
    """The tile shapes and buffer counts that few tiles do not reach, on sampled pixels."""
    L = wl.ConvLayer("f", *shape)
    D, W = wl.normal(L.dD_shape, 1.0, 5, wl.BF16), wl.normal(L.W_shape, 0.1, 6, wl.BF16)
    total = int(np.prod(L.dO_shape[:3]))
    pixels = np.unique(np.concatenate([np.arange(130), np.arange(total - 130, total), np.random.default_rng(3).integers(0, total, 4000)]))
    ref, ab = oracle.conv_fwd(D, W, L.stride, L.pad, pixels=pixels)
    out = sdgp.sdgp_conv_fwd(to_gpu(D), to_gpu(W), L.stride, L.pad).view(total, L.C_out)
    got = wl.to_f64(to_host(out[torch.from_numpy(pixels).cuda()]))
    assert np.max(np.abs(got - ref)[ab > 0] / ab[ab > 0]) <= 4e-3


def test_infinite_weight_outside_the_image():
    """A tap outside the image has no term: an infinite weight there must not reach the pixel."""
    D = torch.ones(2, 7, 7, 8, dtype=torch.bfloat16, device="cuda")
    W = torch.ones(16, 3, 3, 8, dtype=torch.bfloat16, device="cuda")
    W[3, 0, 0] = float("inf")             # stride 2, pad 1: outside for output row 0 and output column 0
    out = sdgp.sdgp_conv_fwd(D, W, 2, 1).float().cpu()
    inside = torch.isposinf(out[..., 3])
    assert inside[:, 1:, 1:].all() and not inside[:, 0].any() and not inside[:, :, 0].any()
    assert out[0, 0, 1, 3] == 48 and out[0, 0, 0, 3] == 32 and torch.isfinite(out[..., :3]).all()


@pytest.mark.parametrize("B,hw,C_in,C_out,stride", [(64, 56, 128, 128, 2), (64, 16, 128, 128, 1)])
def test_nan_activations_cost_no_more(B, hw, C_in, C_out, stride):
    """A diverged step's activations: no weight is non-finite, so nothing has to be summed again."""
    W = torch.full((C_out, 3, 3, C_in), 0.01, dtype=torch.bfloat16, device="cuda")

    def run(value):
        D = torch.full((B, hw, hw, C_in), value, dtype=torch.bfloat16, device="cuda")
        best = 1e9
        for _ in range(3):
            begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            begin.record()
            for _ in range(5):
                out = sdgp.sdgp_conv_fwd(D, W, stride, 1)
            end.record()
            end.synchronize()
            best = min(best, begin.elapsed_time(end))
        return best, out

    finite, _ = run(1.0)
    nan, out = run(float("nan"))
    assert out.isnan().all()
    assert nan < 3 * finite, (nan, finite)
