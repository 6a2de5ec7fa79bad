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
    (2100, 4, 4, 264, 40, 1, 1, 1, 0),      # 1x1, ragged C_out, more than 1024 tiles: the padded copies
    (270, 8, 8, 16, 40, 3, 3, 1, 1),        # ragged C_out, more than 511 tiles: bwd_tiled
    (300, 9, 11, 24, 40, 3, 3, 2, 1),       # the same, strided
    (64, 16, 16, 72, 32, 5, 5, 1, 2),       # a filter neither three wide nor 1x1: bwd_conv3
    (65, 16, 16, 72, 32, 2, 2, 1, 1),
    (70, 16, 16, 64, 64, 3, 3, 1, 1),       # the row kernel
    (350, 7, 7, 136, 64, 1, 1, 1, 0),       # the pointwise kernel
    (170, 14, 14, 72, 64, 3, 3, 2, 1),      # its parity classes
])
def test_neighbours(shape, n, m):
    check(shape, n, m, oracle.RANDOM)
