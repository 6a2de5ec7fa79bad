"""The calls this library's speed is judged by, over the sizes its users run.

The layers are those of the two networks the repository's workloads describe (ResNet-9 on 32x32 images, ResNet-50 on
224x224 images), RegNetX-400MF's grouped 3x3 layers and the small fp32 linear layer of the tests.  Every case is one
call of a public entry point on tensors that are already on the GPU:

  linear    sdgp_linear_bwd_data                     conv     sdgp_conv_bwd_data
  channel   sdgp_conv_bwd_data_channel_rescaled      grouped  sdgp_conv_bwd_data_grouped
  prune     sdgp_prune                               forward  sdgp_conv_fwd
  wgrad     sdgp_conv_bwd_weight

``listed`` holds one case for each, ``draw`` varies batch, image size, channels, filter, stride, n:m and ranker around
them, ragged sizes included.  ``exact`` is the definition in plain torch, float64.
"""
import math

import torch

import paper_2202_00774_amd as sdgp

_RANKERS = {"random": sdgp.RANDOM, "magnitude": sdgp.GREEDY, "rescaled": sdgp.GREEDY_ADJUSTED}
_DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}


def _conv(name, op, B, hw, C_in, C_out, R, stride, pad, dtype="bf16", n=2, m=4, ranker="magnitude", groups=1):
    return {"name": name, "op": op, "B": B, "hw": hw, "C_in": C_in, "C_out": C_out, "R": R, "stride": stride, "pad": pad,
            "dtype": dtype, "n": n, "m": m, "ranker": ranker, "groups": groups}


def listed():
    return [
        # the smallest call: a linear layer of a small network in fp32; its launch is most of it
        {"name": "linear_f32_256x128x256", "op": "linear", "rows": 256, "C_out": 128, "C_in": 256, "dtype": "f32",
         "n": 2, "m": 4, "ranker": "magnitude"},
        # ResNet-50's classifier, called as the linear layer it is: 1000 outputs are no multiple of a tile
        {"name": "classifier_256x1000x2048", "op": "linear", "rows": 256, "C_out": 1000, "C_in": 2048, "dtype": "bf16",
         "n": 2, "m": 4, "ranker": "random"},
        # ResNet-50, batch 256: the 1x1 layer that takes the largest share of the pass; bound by memory
        _conv("pointwise_64x256_56", "conv", 256, 56, 64, 256, 1, 1, 0, ranker="random"),
        # ResNet-9, batch 512: a 3x3 layer, bound by arithmetic
        _conv("conv3_128x256_16", "conv", 512, 16, 128, 256, 3, 1, 1),
        # ResNet-50, batch 256: the strided 3x3 layer that opens a stage
        _conv("conv3s2_128x128_56", "conv", 256, 56, 128, 128, 3, 2, 1, ranker="random"),
        # ResNet-50, batch 256: the 7x7 stem, three input channels
        _conv("stem7_3x64_224", "conv", 256, 224, 3, 64, 7, 2, 3, ranker="random"),
        # ResNet-9's 3x3 layers in fp32, batch 128
        _conv("conv3_f32_128x128_16", "conv", 128, 16, 128, 128, 3, 1, 1, dtype="f32"),
        # ResNet-9, batch 512: Rescaled Magnitude with one factor per channel, sweep and product in one call
        _conv("channel_64x128_32", "channel", 512, 32, 64, 128, 3, 1, 1),
        # RegNetX-400MF, batch 256: the grouped 3x3 layer of its third stage
        _conv("grouped_160_14", "grouped", 256, 14, 160, 160, 3, 1, 1, groups=10),
        # the pruning function alone on the gradient of ResNet-50's first stage, batch 128
        {"name": "prune_4of8_56", "op": "prune", "rows": 128 * 56 * 56, "C": 256, "dtype": "bf16", "n": 4, "m": 8,
         "ranker": "rescaled", "compact": False},
        # the forward pass of the strided 3x3 layer, batch 128
        _conv("forward3s2_128x128_56", "forward", 128, 56, 128, 128, 3, 2, 1),
        # the weight gradient of ResNet-50's most frequent kind of layer, a 1x1, batch 64
        _conv("wgrad1_256x64_56", "wgrad", 64, 56, 256, 64, 1, 1, 0),
    ]


# ------------------------------------------------------------------------------------------------ drawn cases

_NM = ((2, 4), (2, 4), (2, 8), (2, 16), (1, 4), (4, 8), (4, 16), (4, 32), (4, 4))


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _channels(rng, lo, hi, step):
    return max(step, int(round(_log(rng, lo, hi) / step)) * step)


def _pattern(rng, C):
    return rng.choice([nm for nm in _NM if C % nm[1] == 0])


def _fit(case, most):
    """Halves the batch until the case costs no more than `most` bytes and flops (dense ones)."""
    def over():
        b, f = _size(case)
        return b > most[0] or f > most[1]
    while case["B"] > 1 and over():
        case["B"] = (case["B"] + 1) // 2
    while case["hw"] > 16 and over():
        case["hw"] = case["hw"] * 3 // 4
    return case


def draw(rng):
    base = dict(rng.choice(listed()))
    base.pop("name")
    op, ranker = base["op"], rng.choice(sorted(_RANKERS))
    if op == "linear":
        f32 = base["dtype"] == "f32"
        base.update(rows=_log(rng, 16, 2048), C_out=_channels(rng, 64, 1024, 8), C_in=_channels(rng, 64, 1024 if f32 else 2048, 4 if f32 else 8))
        base["n"], base["m"] = _pattern(rng, base["C_out"])
        base["ranker"] = ranker
        return base
    if op == "prune":
        base.update(C=_channels(rng, 64, 1024, 8), dtype=rng.choice(["bf16", "bf16", "f32"]), compact=rng.random() < 0.3, ranker=ranker)
        base["rows"] = max(1, _log(rng, 1 << 16, 1 << 26) // base["C"])
        base["n"], base["m"] = _pattern(rng, base["C"])
        return base
    most = _size(base)
    base["B"] = _log(rng, max(2, base["B"] // 8), base["B"])
    if op == "grouped":
        groups = rng.randint(2, 24)
        base.update(groups=groups, C_in=16 * groups, C_out=16 * groups, hw=rng.randint(7, 56), stride=rng.choice([1, 1, 2]), ranker=ranker)
        base["n"], base["m"] = _pattern(rng, 16)
        return _fit(base, most)
    if base["C_in"] == 3:  # first layers: the 7x7 stem, and the 3x3 layer of a network for small images
        if rng.random() < 0.6:
            base["hw"] = rng.randint(96, 224)
        else:
            base.update(R=3, stride=1, pad=1, hw=rng.randint(24, 64))
        base["ranker"] = ranker
        base["n"], base["m"] = _pattern(rng, base["C_out"])
        return _fit(base, most)
    step = rng.choice([64, 32, 32, 8])
    base.update(C_in=_channels(rng, 32, 512, step), C_out=_channels(rng, 32, 512, step))
    base["hw"] = _log(rng, 7, 56) if base["dtype"] == "bf16" else _log(rng, 4, 32)
    if op in ("forward", "wgrad"):
        base["R"] = rng.choice([1, 3])
        base["stride"] = rng.choice([1, 2])
    elif base["dtype"] == "f32":
        base["R"] = rng.choice([1, 3, 3])
        base["stride"] = rng.choice([1, 1, 2])
    elif op == "conv" and base["R"] == 1:
        base["stride"] = rng.choice([1, 1, 1, 2])
        if rng.random() < 0.5:  # the wide side of a bottleneck
            base[rng.choice(["C_in", "C_out"])] = _channels(rng, 512, 2048, 64)
    base["pad"] = base["R"] // 2
    if op in ("conv", "channel"):
        base["n"], base["m"] = _pattern(rng, base["C_out"])
        base["ranker"] = ranker
    return _fit(base, most)


# ------------------------------------------------------------------------------------------------ sizes and work

def _out_hw(c):
    return (c["hw"] + 2 * c["pad"] - c["R"]) // c["stride"] + 1


def _size(c):
    """(bytes, dense flops) of a convolution case."""
    elem = 4 if c["dtype"] == "f32" else 2
    pq, nW = _out_hw(c), c["C_out"] * c["R"] ** 2 * c["C_in"] // c["groups"]
    n_out, n_in = c["B"] * pq * pq * c["C_out"], c["B"] * c["hw"] ** 2 * c["C_in"]
    if c["op"] == "wgrad":
        return (n_out + n_in) * elem + nW * 4, 2 * c["B"] * pq * pq * nW
    return (n_out + n_in + nW) * elem, 2 * c["B"] * pq * pq * nW


def work(case):
    c = case
    if c["op"] == "prune":
        elem, total = (4 if c["dtype"] == "f32" else 2), c["rows"] * c["C"]
        out = total * elem + (total // c["m"] * c["n"] * (elem + 1) if c["compact"] else 0)
        return {"bytes": total * elem + out, "flops": 0}
    if c["op"] == "linear":
        elem = 4 if c["dtype"] == "f32" else 2
        b = (c["rows"] * (c["C_out"] + c["C_in"]) + c["C_out"] * c["C_in"]) * elem
        f = 2 * c["rows"] * c["C_out"] * c["C_in"]
    else:
        b, f = _size(c)
    if c["op"] in ("forward", "wgrad"):
        return {"bytes": b, "flops": f}
    return {"bytes": b, "flops": f * c["n"] // c["m"]}  # only the kept values need multiplying


# ------------------------------------------------------------------------------------------------ inputs

def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _gradient(shape, seed, dtype):
    """Laplace values of scale 1e-3, three tenths of them exactly zero: what an output gradient looks like."""
    g = _generator(seed)
    u = torch.rand(shape, generator=g, device="cuda").mul_(2).sub_(1)
    x = torch.log1p(-u.abs().clamp_(max=1 - 1e-7)).mul_(torch.sign(u)).mul_(-1e-3)
    return x.masked_fill_(torch.rand(shape, generator=g, device="cuda") < 0.3, 0.0).to(dtype)


def _normal(shape, std, seed, dtype):
    return torch.randn(shape, generator=_generator(seed), device="cuda").mul_(std).to(dtype)


def prepare(case, seed):
    c, dt = dict(case), _DTYPES[case["dtype"]]
    if c["op"] == "prune":
        return {"c": c, "seed": seed, "dO": _gradient((c["rows"], c["C"]), 4 * seed + 1, dt)}
    if c["op"] == "linear":
        return {"c": c, "seed": seed, "dO": _gradient((c["rows"], c["C_out"]), 4 * seed + 1, dt),
                "W": _normal((c["C_out"], c["C_in"]), math.sqrt(2.0 / c["C_in"]), 4 * seed + 2, dt)}
    pq = _out_hw(c)
    s = {"c": c, "seed": seed}
    if c["op"] != "forward":
        s["dO"] = _gradient((c["B"], pq, pq, c["C_out"]), 4 * seed + 1, dt)
    if c["op"] != "wgrad":
        cig = c["C_in"] // c["groups"]
        s["W"] = _normal((c["C_out"], c["R"], c["R"], cig), math.sqrt(2.0 / (c["R"] ** 2 * cig)), 4 * seed + 2, dt)
    if c["op"] in ("forward", "wgrad"):  # activations behind a ReLU
        s["D"] = _normal((c["B"], c["hw"], c["hw"], c["C_in"]), 1.0, 4 * seed + 3, dt).clamp_(min=0)
    return s


def run(state):
    c, seed = state["c"], state["seed"]
    if c["op"] == "prune":
        return sdgp.sdgp_prune(state["dO"], c["n"], c["m"], _RANKERS[c["ranker"]], seed, compact=c["compact"])
    if c["op"] == "linear":
        return sdgp.sdgp_linear_bwd_data(state["dO"], state["W"], c["n"], c["m"], _RANKERS[c["ranker"]], seed)
    if c["op"] == "forward":
        return sdgp.sdgp_conv_fwd(state["D"], state["W"], c["stride"], c["pad"])
    if c["op"] == "wgrad":
        return sdgp.sdgp_conv_bwd_weight(state["D"], state["dO"], c["R"], c["R"], c["stride"], c["pad"])
    at = (state["dO"], state["W"], c["hw"], c["hw"], c["stride"], c["pad"])
    if c["op"] == "channel":
        return sdgp.sdgp_conv_bwd_data_channel_rescaled(*at, c["n"], c["m"])
    if c["op"] == "grouped":
        return sdgp.sdgp_conv_bwd_data_grouped(*at, c["groups"], c["n"], c["m"], _RANKERS[c["ranker"]], seed)
    return sdgp.sdgp_conv_bwd_data(*at, c["n"], c["m"], _RANKERS[c["ranker"]], seed)


# Measured against `exact` over the listed and forty drawn cases: rounding a result once to bf16 shows 1.7e-3, and
# 2.4e-3 where the pruned and rescaled operand is rounded as well (largest single difference 3.9e-3 and 1.1e-2); fp32
# products 1.4e-7 to 6.1e-7 (4.6e-6), weight gradients with their fp32 sums of up to 2e5 terms 1.4e-7 (5.5e-7) in one
# order of summation, to which a longer chain of additions may add.
def tolerance(case):
    if case["op"] == "prune" and case["ranker"] != "rescaled":
        return "exact"
    if case["dtype"] == "f32":
        return {"rel": 2.5e-6, "max": 2e-5}
    if case["op"] == "wgrad":
        return {"rel": 2e-6, "max": 2e-5}
    return {"rel": 1e-2, "max": 4.5e-2}


# ------------------------------------------------------------------------------------------------ the definition in 64 bits

_M32 = 0xFFFFFFFF


def _hash_keys(lo, hi, seed):
    """The random rule's key of flat elements lo .. hi-1: a 32-bit counter hash of the aligned quad, turned by bytes."""
    e = torch.arange(lo, hi, dtype=torch.int64, device="cuda")
    v = (0xA54FF53A ^ ((seed & _M32) * 0x9E3779B9 & _M32) ^ ((seed >> 32) * 0x510E527F & _M32))
    v = v ^ ((e & _M32) >> 2) ^ ((e >> 32) * 0xBB67AE85 & _M32)
    v = v ^ (v >> 16)
    v = v * 0x6A09E667 & _M32
    v = v ^ (v >> 15)
    v = v * 0xBB67AE85 & _M32
    v = v ^ (v >> 16)
    r = (e & 3) * 8
    return ((v << r) | (v >> (32 - r))) & 0xFFFFFFF0


def _keep(x, n, m, ranker, seed, first):
    """Which elements of x [rows, C] stay: the n of every m with the largest (key, lower position first)."""
    if n == m:
        return torch.ones_like(x, dtype=torch.bool)
    if ranker == "random":
        key = _hash_keys(first, first + x.numel(), seed)
    elif x.dtype == torch.bfloat16:
        key = x.reshape(-1).view(torch.int16).to(torch.int64) & 0x7FFF
    else:
        key = x.reshape(-1).view(torch.int32).to(torch.int64) & 0x7FFFFFFF
    key = key.view(-1, m) * 32 + torch.arange(m - 1, -1, -1, device="cuda")
    kept = torch.zeros_like(key, dtype=torch.bool)
    for _ in range(n):
        top = key == key.amax(1, keepdim=True)
        kept |= top
        key.masked_fill_(top, -1)
    return kept.view(x.shape)


_CHUNK = 1 << 25  # elements at a time


def _pruned(x, c, seed):
    """Alg. 1 on x [rows, C] in 64 bits, and the kept mask."""
    n, m, ranker = c["n"], c["m"], c["ranker"]
    out = torch.empty(x.shape, dtype=torch.float64, device="cuda")
    mask = torch.empty(x.shape, dtype=torch.bool, device="cuda")
    step = max(1, _CHUNK // x.shape[1])
    for at in range(0, x.shape[0], step):
        part = x[at:at + step]
        kept = _keep(part, n, m, ranker, seed, at * x.shape[1])
        v = part.double()
        if ranker == "rescaled" and n < m:
            a = v.abs().view(-1, m)
            t = (a * kept.view(-1, m)).sum(1, keepdim=True)
            v = (v.view(-1, m) * torch.where(t > 0, a.sum(1, keepdim=True) / t.clamp(min=1e-300), torch.ones_like(t))).view(part.shape)
        out[at:at + step] = v * kept
        mask[at:at + step] = kept
    return out, mask


def _back(g, W, hw, stride, pad):
    """dD [B,hw,hw,C] of g [B,P,P,K] and W [K,R,R,C], both float64."""
    B, P, _, K = g.shape
    R, C = W.shape[1], W.shape[3]
    size = max(hw + 2 * pad, (P - 1) * stride + R)
    out = torch.zeros((B, size, size, C), dtype=torch.float64, device="cuda")
    end = (P - 1) * stride + 1
    for r in range(R):
        for s in range(R):
            t = g.reshape(-1, K) @ W[:, r, s, :].contiguous()
            out[:, r:r + end:stride, s:s + end:stride] += t.view(B, P, P, C)
    return out[:, pad:pad + hw, pad:pad + hw].contiguous()


def _in_batches(c, f):
    """f(first, last) over runs of images, laid together."""
    step = max(1, _CHUNK // (c["hw"] ** 2 * max(c["C_in"], c["C_out"])))
    return torch.cat([f(b, min(b + step, c["B"])) for b in range(0, c["B"], step)])


def exact(case, seed):
    s, c = prepare(case, seed), dict(case)
    if c["op"] == "prune":
        out, mask = _pruned(s["dO"], c, seed)
        if not c["compact"]:
            return out, None, None
        at = torch.arange(c["m"], device="cuda").repeat(c["C"] // c["m"]).expand(mask.shape)
        kept = (c["rows"], c["C"] // c["m"] * c["n"])
        return out, out[mask].view(kept), at[mask].view(kept).to(torch.uint8)
    if c["op"] == "linear":
        return _pruned(s["dO"], c, seed)[0] @ s["W"].double()
    R, st, pad, pq = c["R"], c["stride"], c["pad"], _out_hw(c)
    if c["op"] in ("forward", "wgrad"):
        end = (pq - 1) * st + 1

        def tap(d, r, q):
            return d[:, r:r + end:st, q:q + end:st].reshape(-1, c["C_in"])

        def padded(a, b):
            return torch.nn.functional.pad(s["D"][a:b].double(), (0, 0, pad, pad, pad, pad))
        if c["op"] == "forward":
            W = s["W"].double()

            def forward(a, b):
                d = padded(a, b)
                return sum(tap(d, r, q) @ W[:, r, q].t() for r in range(R) for q in range(R)).view(b - a, pq, pq, c["C_out"])
            return _in_batches(c, forward)
        dW = torch.zeros((c["C_out"], R, R, c["C_in"]), dtype=torch.float64, device="cuda")

        def wgrad(a, b):
            d, g = padded(a, b), s["dO"][a:b].double().reshape(-1, c["C_out"]).t().contiguous()
            for r in range(R):
                for q in range(R):
                    dW[:, r, q] += g @ tap(d, r, q)
            return torch.empty(0)
        _in_batches(c, wgrad)
        return dW
    W = s["W"].double()
    if c["op"] == "channel":
        x = s["dO"].view(-1, c["C_out"])
        mag = dict(c, ranker="magnitude")
        g = _pruned(x, mag, seed)[0]
        some, every = g.abs().sum(0), x.double().abs().sum(0)
        g = (g * torch.where(some > 0, every / some.clamp(min=1e-300), torch.ones_like(some))).view(s["dO"].shape)
    else:
        g = _pruned(s["dO"].view(-1, c["C_out"]), c, seed)[0].view(s["dO"].shape)
    if c["op"] == "grouped":
        k, ci = c["C_out"] // c["groups"], c["C_in"] // c["groups"]
        return torch.cat([_back(g[..., i * k:(i + 1) * k].contiguous(), W[i * k:(i + 1) * k], c["hw"], st, pad)
                          for i in range(c["groups"])], dim=3)
    return _in_batches(c, lambda a, b: _back(g[a:b], W, c["hw"], st, pad))
