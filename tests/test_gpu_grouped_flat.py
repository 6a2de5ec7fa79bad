"""Grouped 3x3 layers of 16 channels per group on both of their kernels: the one that runs along the padded line of all
grid positions (at the widths where rows and images begin anywhere inside its runs of sixteen, and at the widest it
takes) and the one with tiles of 8 x 32 positions that takes wider images.

Tolerance relative to sum |a||w|: one rounding of the result and one of a rescaled value to bf16 (2^-9 each), fp32 sums of
144 terms: 5e-3.
"""
import numpy as np
import pytest

import oracle
import paper_2202_00774_amd as sdgp
from paper_2202_00774_amd import workloads as wl
from util import to_gpu, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m,ranker", [(2, 4, oracle.RANDOM), (4, 8, oracle.GREEDY_ADJUSTED), (4, 4, oracle.GREEDY)])
@pytest.mark.parametrize("B,H,Wd,groups,stride", [
    (1, 1, 1, 1, 1), (37, 1, 1, 3, 2), (70, 2, 3, 2, 1), (3, 15, 15, 5, 1), (2, 5, 63, 3, 1), (2, 4, 64, 3, 1), (1, 9, 97, 2, 1),
    (36, 63, 63, 4, 1),   # narrow enough, but enough workgroups for the tiles, which rank fewer pixels of it
    (3, 7, 9, 3, 2), (2, 6, 126, 1, 2), (2, 5, 127, 2, 2), (1, 8, 128, 2, 2),
])
def test_matches_oracle(B, H, Wd, groups, stride, n, m, ranker):
    C = 16 * groups
    P, Q = oracle.conv_out_size(H, 3, stride, 1), oracle.conv_out_size(Wd, 3, stride, 1)
    dO = wl.laplace_with_zeros((B, P, Q, C), 1e-3, 0.3, 7 + C, wl.BF16)
    W = wl.normal((C, 3, 3, 16), 0.1, 8 + C, wl.BF16)
    ref, ab = oracle.conv_bwd_data_grouped(oracle.prune(dO, n, m, ranker, seed=5)[0], W, H, Wd, stride, 1, groups)
    got = wl.to_f64(to_host(sdgp.sdgp_conv_bwd_data_grouped(to_gpu(dO), to_gpu(W), H, Wd, stride, 1, groups, n, m, ranker, 5)))
    assert np.all(got[ab == 0] == 0)
    assert np.max(np.abs(got - ref)[ab > 0] / ab[ab > 0]) <= 5e-3
