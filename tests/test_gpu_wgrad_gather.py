"""The gathering weight-gradient kernel (any filter and stride, channels multiples of 8) against the oracle at the edges
of its tiles: every block shape, channel counts that end inside a tile, fewer pixels than a chunk, runs that end inside a
chunk, taps that never meet the image, one split and many.

Tolerance relative to sum |a||b|: products of bf16 values are exact in fp32, runs of at most 128 of them are summed in fp32
(128 * 2^-24 = 7.6e-6 of the run's sum |a||b| at the very worst), the runs and the splits in fp64, and the result is rounded
once to fp32: 8e-6.  (The plain kernel, which takes small filters over few pixels, adds shorter chains.)
"""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2202_00774_amd as sdgp
from paper_2202_00774_amd import binding
from paper_2202_00774_amd import workloads as wl
from util import to_gpu

pytestmark = pytest.mark.gpu

LAYERS = [  # B, H, Wd, C_in, C_out, R, S, stride, pad
    (3, 9, 7, 64, 64, 1, 1, 1, 0),
    (2, 28, 28, 256, 64, 1, 1, 1, 0),       # 64 x 256 blocks, many splits
    (2, 13, 13, 136, 120, 1, 1, 1, 0),      # 128 x 128, ragged on both sides
    (2, 11, 11, 64, 264, 1, 1, 2, 0),       # 64 x 64, five blocks of output channels, the last of 8
    (2, 30, 30, 64, 256, 1, 1, 1, 0),       # 256 x 64
    (2, 30, 30, 56, 248, 2, 2, 1, 1),       # the same, ragged on both sides
    (12, 56, 56, 64, 256, 1, 1, 1, 0),      # 256 x 64, 74 splits: added by sixteen wavefronts
    (12, 56, 56, 64, 64, 1, 1, 1, 0),       # 64 x 64, 74 splits
    (1, 1, 1, 8, 8, 1, 1, 1, 0),            # one pixel
    (5, 8, 9, 72, 40, 3, 3, 2, 1),
    (2, 7, 7, 32, 96, 3, 3, 1, 1),          # stride 1 beside the kernel for multiples of 64
    (1, 3, 2, 16, 24, 2, 2, 1, 1),
    (4, 6, 6, 24, 16, 5, 3, 3, 2),
    (1, 2, 2, 160, 8, 7, 7, 4, 3),          # most taps meet no pixel
]


@pytest.mark.parametrize("shape", LAYERS)
def test_matches_oracle(shape):
    L = wl.ConvLayer("w", *shape)
    D = wl.normal(L.dD_shape, 1.0, 5, wl.BF16)
    G = wl.laplace_with_zeros(L.dO_shape, 1e-3, 0.3, 6, wl.BF16)
    ref, ab = oracle.conv_bwd_weight(D, G, L.R, L.S, L.stride, L.pad)
    out = sdgp.sdgp_conv_bwd_weight(to_gpu(D), to_gpu(G), L.R, L.S, L.stride, L.pad)
    again = sdgp.sdgp_conv_bwd_weight(to_gpu(D), to_gpu(G), L.R, L.S, L.stride, L.pad)
    assert torch.equal(out, again)
    got = out.cpu().numpy().astype(np.float64)
    assert np.all(got[ab == 0] == 0)
    assert np.max(np.abs(got - ref)[ab > 0] / ab[ab > 0]) <= 8e-6


def test_without_workspace():
    """The workspace is an option of these layers: a call without one gives the same sums from the plain kernel."""
    L = wl.ConvLayer("n", 4, 16, 16, 64, 72, 1, 1, 1, 0)
    D, G = to_gpu(wl.normal(L.dD_shape, 1.0, 5, wl.BF16)), to_gpu(wl.laplace_with_zeros(L.dO_shape, 1e-3, 0.3, 6, wl.BF16))
    lib = binding.load()
    geometry = (L.B, L.H, L.Wd, L.C_in, L.C_out, L.R, L.S, L.stride, L.pad, binding.BF16)
    assert lib.sdgp_conv_bwd_weight_workspace(*geometry) > 0
    out = torch.full(L.W_shape, float("nan"), device="cuda")
    assert lib.sdgp_conv_bwd_weight(D.data_ptr(), G.data_ptr(), out.data_ptr(), *geometry, None, 0,
                                    ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
    assert torch.allclose(out, sdgp.sdgp_conv_bwd_weight(D, G, 1, 1, 1, 0), rtol=1e-4, atol=1e-6)


def test_infinite_gradient_stays_with_its_taps():
    """A pixel whose tap falls outside the image adds nothing to that tap, whatever its gradient."""
    D = torch.ones(1, 5, 5, 8, dtype=torch.bfloat16, device="cuda")
    G = torch.ones(1, 3, 3, 8, dtype=torch.bfloat16, device="cuda")
    G[0, 0, 0] = float("inf")            # stride 2, pad 1: its taps (0, .) and (., 0) lie outside
    out = sdgp.sdgp_conv_bwd_weight(D, G, 3, 3, 2, 1)
    assert torch.isinf(out[:, 1:, 1:]).all() and torch.isfinite(out[:, 0]).all() and torch.isfinite(out[:, :, 0]).all()


@pytest.mark.parametrize("shape,asks", [
    ((8, 16, 16, 8, 8, 3, 3, 1, 1), False),     # 576 elements, 2048 pixels: the plain kernel, one workgroup an element
    ((3, 16, 16, 16, 16, 3, 3, 1, 1), False),   # 2304, 768 pixels
    ((2, 16, 16, 40, 40, 1, 1, 1, 0), False),   # 1600 elements of a 1x1 filter, 512 pixels: one split, no room needed
    ((8, 16, 16, 40, 40, 1, 1, 1, 0), True),    # the same, 2048 pixels
])
def test_few_elements_and_pixels(shape, asks):
    L = wl.ConvLayer("p", *shape)
    assert (binding.load().sdgp_conv_bwd_weight_workspace(L.B, L.H, L.Wd, L.C_in, L.C_out, L.R, L.S, L.stride, L.pad, binding.BF16) > 0) == asks
    test_matches_oracle(shape)
