"""bf16 backward data on C_out that is a multiple of 8 but not of the 32-channel chunk, on problems large enough for the
row, pointwise and parity-class kernels: every remainder, every kind of ranker, and NaN next to the channels that are missing.

Tolerance: the tests of the other bf16 kernels, 1e-2 of sum |a||w| (one rounding to bf16 shows 2^-9)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2202_00774_amd as sdgp
from paper_2202_00774_amd import workloads as wl
from util import rel_error, to_gpu, to_host

pytestmark = pytest.mark.gpu

KINDS = {  # B, H, Wd, C_in and R, S, stride, pad: enough tiles for the kernel named ("row": the line kernel)
    "row_256": ((150, 16, 16, 72), (3, 3, 1, 1)),
    "row_64": ((300, 9, 9, 40), (3, 3, 1, 1)),
    "pointwise": ((1100, 13, 13, 136), (1, 1, 1, 0)),       # (past the limit of the small ones)
    "pointwise_small": ((5, 41, 41, 40), (1, 1, 1, 0)),         # 66 tiles of 64 columns
    "pointwise_small_256": ((20, 41, 41, 248), (1, 1, 1, 0)),   # 263 tiles of 256
    "pointwise_strided": ((300, 20, 20, 64), (1, 1, 2, 0)),
    "classes": ((60, 28, 28, 136), (3, 3, 2, 1)),
}
PATTERNS = [(2, 4, oracle.RANDOM), (1, 4, oracle.GREEDY_ADJUSTED), (2, 8, oracle.GREEDY), (4, 8, oracle.RANDOM), (3, 4, oracle.GREEDY),
            (8, 8, oracle.GREEDY)]


def run(kind, C_out, n, m, ranker, dO=None, seed=21):
    at, rest = KINDS[kind]
    layer = wl.ConvLayer("t", *at, C_out, *rest)
    if dO is None:
        dO = wl.laplace_with_zeros(layer.dO_shape, 1e-3, 0.3, seed=seed, dtype=wl.BF16)
    W = wl.normal(layer.W_shape, 0.1, seed + 1, wl.BF16)
    pixels = np.random.default_rng(2).choice(layer.B * layer.H * layer.Wd, 3000, replace=False)
    pixels.sort()
    pruned = oracle.prune(dO, n, m, ranker, seed=seed)[0]
    ref, ab = oracle.conv_bwd_data(pruned, W, layer.H, layer.Wd, layer.stride, layer.pad, pixels=pixels)
    out = sdgp.sdgp_conv_bwd_data(to_gpu(dO), to_gpu(W), layer.H, layer.Wd, layer.stride, layer.pad, n, m, ranker, seed)
    return layer, wl.to_f64(to_host(out.reshape(-1, layer.C_in)[torch.from_numpy(pixels).to(out.device)])), ref, ab


@pytest.mark.parametrize("n,m,ranker", PATTERNS)
@pytest.mark.parametrize("C_out", [40, 56, 72, 8])
@pytest.mark.parametrize("kind", sorted(KINDS))
def test_remainders(kind, C_out, n, m, ranker):
    _, got, ref, ab = run(kind, C_out, n, m, ranker)
    assert rel_error(got, ref, ab) <= 1e-2
    assert np.all(got[ab == 0] == 0)


@pytest.mark.parametrize("n", [2, 5])
@pytest.mark.parametrize("kind", sorted(KINDS))
def test_half_a_chunk(kind, n):
    """Groups of 16: the last chunk is one group."""
    _, got, ref, ab = run(kind, 80, n, 16, oracle.GREEDY)
    assert rel_error(got, ref, ab) <= 1e-2


@pytest.mark.parametrize("n,m,ranker", PATTERNS + [(1, 4, oracle.GREEDY), (3, 16, oracle.GREEDY_ADJUSTED), (5, 8, oracle.GREEDY)])
def test_one_round_of_wide_tiles(n, m, ranker, monkeypatch):
    """134 tiles of 256 columns, which would be 268 of 128: pruned patterns on the wide ones (whole chunks)."""
    monkeypatch.setitem(KINDS, "wide", ((101, 13, 13, 248), (1, 1, 1, 0)))
    _, got, ref, ab = run("wide", 96, n, m, ranker)
    assert rel_error(got, ref, ab) <= 1e-2
    assert np.all(got[ab == 0] == 0)


@pytest.mark.parametrize("n,m", [(8, 8), (2, 4)])
@pytest.mark.parametrize("kind", sorted(KINDS))
def test_nan_behind_the_last_channel(kind, n, m):
    """What follows a pixel's last channel in memory is the next pixel's first one: a NaN there must stay there."""
    at, rest = KINDS[kind]
    layer = wl.ConvLayer("t", *at, 40, *rest)
    dO = wl.laplace_with_zeros(layer.dO_shape, 1e-3, 0.0, seed=4, dtype=wl.BF16)
    dO[1::2, :, :, 0] = 0x7FC0        # every second image; the images between them stay clean
    _, got, ref, ab = run(kind, 40, n, m, oracle.GREEDY, dO)
    clean = np.isfinite(ref)
    assert clean.any() and not clean.all()
    assert np.array_equal(np.isfinite(got), clean)
    assert np.all(np.abs(got[clean] - ref[clean]) <= 1e-2 * ab[clean])


def test_small_ones_need_no_workspace():
    """The query names one for small 1x1 layers with a short last chunk, and nothing reads it: a call without it, with one that is too
    small and through the binding, which allocates none, gives the same bits."""
    layer = wl.ConvLayer("w", 5, 41, 41, 248, 1000, 1, 1, 1, 0)
    dO, W = to_gpu(wl.laplace_with_zeros(layer.dO_shape, 1e-3, 0.3, seed=1, dtype=wl.BF16)), to_gpu(wl.normal(layer.W_shape, 0.1, 2, wl.BF16))
    geometry = (layer.B, layer.H, layer.Wd, layer.C_in, layer.C_out, 1, 1, 1, 0, sdgp.BF16, 2, 4)
    need = sdgp.conv_bwd_data_workspace(*geometry)
    assert need > 1 << 20
    room = torch.full((need,), 7, dtype=torch.uint8, device="cuda")
    outs = []
    for ptr, size in ((room.data_ptr(), need), (None, 0), (room.data_ptr(), 16)):
        out = torch.empty(layer.dD_shape, dtype=torch.bfloat16, device="cuda")
        rc = sdgp.binding.load().sdgp_conv_bwd_data(dO.data_ptr(), W.data_ptr(), out.data_ptr(), *geometry, sdgp.GREEDY, 0, ptr, size,
                                                    torch.cuda.current_stream().cuda_stream)
        assert rc == 0
        outs.append(out)
    torch.cuda.synchronize()
    assert torch.all(room == 7)
    out = torch.empty_like(out)
    torch.cuda.reset_peak_memory_stats()
    before = torch.cuda.memory_allocated()
    sdgp.sdgp_conv_bwd_data(dO, W, layer.H, layer.Wd, 1, 0, 2, 4, sdgp.GREEDY, 0, out=out)
    assert torch.cuda.max_memory_allocated() == before
    for other in outs:
        assert torch.equal(other.view(torch.int16), out.view(torch.int16))
