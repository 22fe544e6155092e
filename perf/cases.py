"""The workloads this library is timed and checked on.

Each case is one call, or one short chain of calls, that a program using the
library makes: a single fused sparse layer (any batch, filter, stride, density),
the chained blocks of the paper's evaluation (VGG-style, ResNet basic block,
Resize-Conv-ReLU-Maxpool), and the plain CSR call of the C interface. Layers are
built once, as a network is, and called on new inputs. ``listed`` holds fixed
cases over the range, ``draw`` more of the same ranges, ``prepare`` and ``run``
what a program holds before a call and the call itself, ``exact`` the result in
float64 from torch alone.

Values: activations are ReLU outputs of a normal distribution (images: U[0, 1)),
weights are normal with variance 2 / (kept taps per output), biases U[-0.1, 0.1),
masks Bernoulli at the case's density, with per-channel densities drawn from
Beta(2, 5) where ``skew`` is set (pruned filters keep very different shares of
their channels).
"""
from __future__ import annotations

import math

import numpy as np
import torch
import torch.nn.functional as F

# kind: "layer"  SparseConvLayer.forward on an unpadded input
#       "chain"  two layers, the first writing the second's padded input
#       "resize" resize_pad_input, then forward_padded
#       "csr"    spconv_pad_input, then spconv_forward (the C call without options)
_DEFAULTS = dict(kind="layer", N=1, C=16, K=16, H=16, W=16, R=3, stride=1, pad=1, density=0.2, skew=False, pool=False,
                 bias=True, residual=False, path="auto", real_channels=0, Hin=0, Win=0)


def _case(name, **kw):
    return {"name": name, **_DEFAULTS, **kw}


def listed():
    return [
        # One small layer on one image: the smallest call, all latency.
        _case("tiny", N=1, C=16, K=16, H=16, W=16, density=0.2),
        # A late, heavily pruned layer in single-image inference.
        _case("single_image_deep", N=1, C=256, K=256, H=14, W=14, density=0.05, skew=True),
        # The deep narrow layer of a pruned network in batched inference, at the
        # three densities of the benchmark (the last one runs the dense path).
        _case("narrow_d005", N=32, C=256, K=256, H=14, W=14, density=0.05, skew=True),
        _case("narrow_d02", N=32, C=256, K=256, H=14, W=14, density=0.2, skew=True),
        _case("narrow_d05", N=32, C=256, K=256, H=14, W=14, density=0.5, skew=True),
        # Conv-ReLU-Maxpool at the density of a lightly pruned layer.
        _case("conv_pool_light", N=32, C=128, K=128, H=28, W=28, density=0.35, pool=True),
        # ResNet basic block: relu(conv2(relu(conv1(x))) + x).
        _case("resnet_block", kind="chain", N=32, C=64, K=64, H=56, W=56, density=0.2, residual=True),
        # VGG-style block, the benchmark's largest configuration: an image of 3
        # channels padded to 64, two layers, the second with the 2x2 max-pool.
        _case("vgg_block", kind="chain", N=32, C=64, K=64, H=224, W=224, density=0.2, pool=True, real_channels=3),
        # Resize-Conv-ReLU-Maxpool: a 42x42 source resized to 28x28.
        _case("resize_block", kind="resize", N=32, C=128, K=128, H=28, W=28, Hin=42, Win=42, density=0.1, pool=True),
        # A downsampling layer (stride 2), as between two stages of a ResNet.
        _case("downsample", N=32, C=64, K=128, H=56, W=56, stride=2, density=0.2),
        # A pointwise layer with the shortcut added (bottleneck block), dense path.
        _case("pointwise", N=32, C=64, K=256, H=28, W=28, R=1, pad=0, density=0.5, residual=True),
        # The plain CSR call on odd sizes: 5x5 filter, odd planes, ragged channels, no bias.
        _case("csr_ragged", kind="csr", N=5, C=37, K=75, H=45, W=61, R=5, pad=2, density=0.15, pool=True, bias=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: batch 1 to 32, 3 to 256 channels, planes of 7 to 224, 1x1 to 5x5
    filters, stride 1 and 2, densities 0.03 to 0.7, odd sizes among them."""
    while True:
        kind = rng.choice(["layer", "layer", "layer", "layer", "chain", "resize", "csr"])
        c = dict(_DEFAULTS)
        c.update(kind=kind, N=_log_int(rng, 1, 32), C=_log_int(rng, 3, 256), K=_log_int(rng, 8, 256),
                 H=_log_int(rng, 7, 224), density=round(math.exp(rng.uniform(math.log(0.03), math.log(0.7))), 3),
                 skew=rng.random() < 0.3, pool=rng.random() < 0.3, bias=rng.random() < 0.9)
        c["W"] = c["H"] if rng.random() < 0.6 else min(224, max(7, int(c["H"] * rng.uniform(0.6, 1.7))))
        if rng.random() < 0.5:  # the round sizes of most networks
            c["C"], c["K"] = max(16, c["C"] // 16 * 16), max(16, c["K"] // 16 * 16)
        if kind == "chain":
            c["K"] = c["C"]
            c["residual"] = rng.random() < 0.5
        elif kind == "resize":
            c["Hin"] = max(7, int(c["H"] * rng.uniform(0.5, 2.0)))
            c["Win"] = max(7, int(c["W"] * rng.uniform(0.5, 2.0)))
        else:
            c["R"] = rng.choice([1, 3, 3, 3, 5])
            c["pad"] = c["R"] // 2
            if kind == "layer":
                c["stride"] = 2 if rng.random() < 0.2 else 1
                c["residual"] = rng.random() < 0.2
                c["path"] = "auto" if rng.random() < 0.7 else "sparse"
        layers = 2 if kind == "chain" else 1
        flops = layers * 2.0 * c["density"] * c["K"] * c["C"] * c["R"] ** 2 * c["N"] * c["H"] * c["W"] / c["stride"] ** 2
        elems = c["N"] * c["H"] * c["W"] * (c["C"] + c["K"])
        if flops <= 5e9 and elems <= 6e7:  # well within the largest listed case
            return c


def _out_side(n, c):
    return (n + 2 * c["pad"] - c["R"]) // c["stride"] + 1


def _weights(c, rng):
    """Masked filter [K, C, R, R], its mask and bias (or None), on the host."""
    K, C, R = c["K"], c["C"], c["R"]
    d = np.full(K, c["density"])
    if c["skew"]:
        d = np.minimum(1.0, rng.beta(2.0, 5.0, size=K) * (c["density"] * 3.5))
    mask = (rng.random((K, C, R, R)) < d[:, None, None, None]).astype(np.uint8)
    std = math.sqrt(2.0 / max(1.0, c["density"] * C * R * R))
    w = np.where(mask != 0, rng.standard_normal((K, C, R, R)) * std, 0.0).astype(np.float32)
    bias = rng.uniform(-0.1, 0.1, K).astype(np.float32) if c["bias"] else None
    return w, mask, bias


def _inputs(c, seed):
    """Filters of each layer, the input and the residual (or None)."""
    rng = np.random.default_rng([seed, 1])
    filters = [_weights(c, rng) for _ in range(2 if c["kind"] == "chain" else 1)]
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 2 + 1)
    H, W = (c["Hin"], c["Win"]) if c["kind"] == "resize" else (c["H"], c["W"])
    shape = (c["N"], c["C"], H, W)
    if c["real_channels"]:
        x = torch.zeros(shape, device="cuda")
        x[:, :c["real_channels"]] = torch.rand((c["N"], c["real_channels"], H, W), generator=g, device="cuda")
    else:
        x = torch.randn(shape, generator=g, device="cuda").relu_()
    res = None
    if c["residual"] and c["kind"] == "layer":
        res = torch.randn((c["N"], c["K"], _out_side(H, c), _out_side(W, c)), generator=g, device="cuda")
    return filters, x, res


def prepare(case, seed):
    from paper_2005_04091_amd import spconv as sp
    c = {**_DEFAULTS, **case}
    filters, x, res = _inputs(c, seed)
    st = {"case": c, "x": x, "residual": res}
    if c["kind"] == "csr":
        w, mask, bias = filters[0]
        host = sp.spconv_pack_csr(w, mask, c["H"] + 2 * c["pad"], c["W"] + 2 * c["pad"])
        st["csr"] = sp.DeviceCSR(host)
        st["bias"] = None if bias is None else torch.from_numpy(bias).cuda()
        return st
    st["layers"] = []
    for i, (w, mask, bias) in enumerate(filters):
        pool = c["pool"] and i + 1 == len(filters)  # a chain pools after its last layer
        layer = sp.SparseConvLayer(w, mask, bias, c["H"], c["W"], c["stride"], c["pad"], True, pool, path=c["path"],
                                   N=c["N"])
        st["layers"].append(layer)
    # A network packs its entry streams before serving.
    first = st["layers"][0]
    unpadded = sp.SPCONV_UNPADDED_INPUT if c["kind"] != "resize" and first.pads_in_kernel(c["N"]) else 0
    first.lowered(c["N"], first.flags | unpadded)
    for layer in st["layers"][1:]:
        layer.lowered(c["N"])
    return st


def run(state):
    from paper_2005_04091_amd import spconv as sp
    c, x = state["case"], state["x"]
    if c["kind"] == "csr":
        xp = sp.spconv_pad_input(x, c["pad"])
        flags = sp.flags_of(True, c["pool"])
        return sp.spconv_forward(xp, c["N"], c["C"], c["H"], c["W"], state["csr"], c["K"], c["R"], c["R"], c["stride"],
                                 c["pad"], state["bias"], flags)
    first = state["layers"][0]
    if c["kind"] == "resize":
        return first.forward_padded(first.resize_pad_input(x))
    if c["kind"] == "chain":
        second = state["layers"][1]
        y = first.forward(x, out_pad=second.pad)
        return second.forward_padded(y, residual=x if c["residual"] else None)
    return first.forward(x, residual=state["residual"])


def work(case):
    c = {**_DEFAULTS, **case}
    layers = 2 if c["kind"] == "chain" else 1
    Ho, Wo = _out_side(c["H"], c), _out_side(c["W"], c)
    nnz = c["density"] * c["K"] * c["C"] * c["R"] ** 2
    H, W = (c["Hin"], c["Win"]) if c["kind"] == "resize" else (c["H"], c["W"])
    stored = c["N"] * c["K"] * ((Ho // 2) * (Wo // 2) if c["pool"] else Ho * Wo)
    elems = c["N"] * c["C"] * H * W + stored
    if c["residual"] and c["kind"] == "layer":
        elems += c["N"] * c["K"] * Ho * Wo
    return {"bytes": 4.0 * elems + layers * (8.0 * nnz + 8.0 * c["K"]), "flops": layers * 2.0 * nnz * c["N"] * Ho * Wo}


def tolerance(case):
    # Sums of up to a few thousand fp32 products: against float64 the listed cases
    # measure 7e-8 (tiny) to 3.1e-7 (256 channels at density 0.5).
    return {"rel": 1.2e-6, "max": 1e-5}


def _conv64(x, w, bias, c):
    """Cross-correlation in float64, one matrix product per filter tap."""
    xp = F.pad(x, (c["pad"],) * 4)
    N, C = x.shape[:2]
    K, _, R, S = w.shape
    st = c["stride"]
    Ho, Wo = (xp.shape[2] - R) // st + 1, (xp.shape[3] - S) // st + 1
    out = torch.zeros((N, K, Ho * Wo), dtype=torch.float64, device=x.device)
    for r in range(R):
        for s in range(S):
            tap = xp[:, :, r:r + (Ho - 1) * st + 1:st, s:s + (Wo - 1) * st + 1:st].reshape(N, C, Ho * Wo)
            for n in range(N):
                out[n].addmm_(w[:, :, r, s].contiguous(), tap[n])
    out = out.view(N, K, Ho, Wo)
    return out if bias is None else out + bias.view(1, K, 1, 1)


def exact(case, seed):
    c = {**_DEFAULTS, **case}
    filters, x, res = _inputs(c, seed)
    y = x.double()
    if c["kind"] == "resize":
        y = F.interpolate(y, size=(c["H"], c["W"]), mode="bilinear", align_corners=False)
    for i, (w, mask, bias) in enumerate(filters):
        wd = torch.from_numpy(w).cuda().double()
        bd = None if bias is None else torch.from_numpy(bias).cuda().double()
        y = _conv64(y, wd, bd, c)
        if res is not None:
            y = y + res.double()
        elif c["residual"] and c["kind"] == "chain" and i == 1:
            y = y + x.double()
        y = torch.relu(y)
    return F.max_pool2d(y, 2) if c["pool"] else y
