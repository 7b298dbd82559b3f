"""The work that performance is judged by: what a user of this package has it do, through its public entry points.

Six kinds of call, over the sizes and options they are used with:

  gemm      a linear layer on quantised activations: `apnn_pack` of the activation codes (one per byte), then `apnn_gemm`
            with weights packed once, to int32 (the step of `bench.py`)
  fc        a fully connected layer inside a packed network: `apnn_layer(is_gemm=True)`, planes in, planes out
  conv      a convolution layer inside a packed network: `apnn_layer`, planes in, planes out, with or without the fused
            2 x 2 max pooling
  conv2d    a convolution on its own: `apnn_pack_fmap` of N x C x H x W codes, then `apnn_conv2d`, to int32
  network   `PackedNet.forward`: an 8-bit image batch in, int32 logits out
  quantize  `apnn_quantize`: fp32 activations to packed planes

A case is a dict of plain values.  All results are whole numbers and exact.
"""
import math

import torch

from paper_2106_12169_amd import binding as B
from paper_2106_12169_amd import workloads as wl
from paper_2106_12169_amd.network import PackedNet

_U, _PM1 = B.ENC_UNSIGNED, B.ENC_PM1
_NETS = {"resnet18": wl.resnet18_layers, "alexnet": wl.alexnet_layers, "vgg16": wl.vgg16_layers}

# (weight bits, activation bits) of the precision sweep and of the fully connected shapes in workloads.py
_BITS = tuple(sorted(set(wl.SWEEP_BITS) | set(wl.PAPER_FC_BITS)))


def listed():
    return [
        # benchmark configuration 0: the smallest product, a call whose time is launches and host work
        dict(name="gemm_w1a2_128", kind="gemm", M=128, N=128, K=128, p=1, q=2, encW=_PM1, encX=_U),
        # benchmark configuration 1, the headline: a large product whose int32 result alone is 64 MiB
        dict(name="gemm_w1a2_4096", kind="gemm", M=4096, N=4096, K=4096, p=1, q=2, encW=_PM1, encX=_U),
        # benchmark configuration 2 at its widest weights: more than two bits on both sides
        dict(name="gemm_w3a5_2048", kind="gemm", M=2048, N=2048, K=2048, p=3, q=5, encW=_U, encX=_U),
        # a 1000-class layer on a batch and a feature count that divide into no tile or vector
        dict(name="gemm_w2a2_ragged", kind="gemm", M=1000, N=777, K=1999, p=2, q=2, encW=_U, encX=_U),
        # the fully connected shape of the paper's latency table: batch 64, 1024 x 1024, serving latency
        dict(name="fc_w1a2_64x1024", kind="fc", N=64, Cin=1024, Cout=1024, p=1, q=2, encW=_U, encX=_U, q_out=2),
        # benchmark configuration 3: one layer of a residual network at batch 8
        dict(name="conv_w1a2_28x28", kind="conv", N=8, H=28, W=28, Cin=128, Cout=128, R=3, stride=1, pad=1,
             p=1, q=2, encW=_PM1, encX=_U, q_out=2, pool=0),
        # a stand-alone convolution with multi-bit operands, an odd frame and a channel count that is no power of two
        dict(name="conv2d_w2a4_ragged", kind="conv2d", N=4, H=27, W=31, Cin=96, Cout=160, R=3, stride=1, pad=1,
             p=2, q=4, encW=_U, encX=_U),
        # benchmark configuration 4: network latency at a small batch
        dict(name="resnet18_b8", kind="network", net="resnet18", batch=8, hw=224),
        # the same network at the batch of the paper's throughput column
        dict(name="resnet18_b128", kind="network", net="resnet18", batch=128, hw=224),
        # one image at a time: the latency of a chain of small launches and of reading wide fully connected weights
        dict(name="alexnet_b1", kind="network", net="alexnet", batch=1, hw=224),
        # the network with the largest convolutions and the fused pooling
        dict(name="vgg16_b8", kind="network", net="vgg16", batch=8, hw=224),
        # the quantisation layer in front of the headline product: memory traffic only
        dict(name="quantize_a2_4096", kind="quantize", rows=4096, K=4096, bits=2),
    ]


def _log_int(rng, lo, hi):
    """An integer from lo to hi, uniform over the logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_enc(rng, p, q):
    """Weights of one bit are -1/+1 or 0/1; activations of one bit join -1/+1 weights in a binary network."""
    encW = rng.choice((_PM1, _U)) if p == 1 else _U
    encX = _PM1 if q == 1 and encW == _PM1 and rng.random() < 0.5 else _U
    return encW, encX


def draw(rng):
    kind = rng.choice(("gemm", "gemm", "fc", "conv", "conv2d", "network", "quantize"))
    if kind == "gemm":
        p, q = rng.choice(_BITS)
        encW, encX = _draw_enc(rng, p, q)
        return dict(kind=kind, M=_log_int(rng, 64, 4096), N=_log_int(rng, 64, 4096), K=_log_int(rng, 64, 4096),
                    p=p, q=q, encW=encW, encX=encX)
    if kind == "fc":
        p, q = rng.choice(wl.PAPER_FC_BITS)
        encW, encX = _draw_enc(rng, p, q)
        return dict(kind=kind, N=_log_int(rng, 1, 256), Cin=_log_int(rng, 128, 4096), Cout=32 * _log_int(rng, 4, 128),
                    p=p, q=q, encW=encW, encX=encX, q_out=2)
    if kind in ("conv", "conv2d"):
        while True:
            p, q = rng.choice(((1, 1), (1, 2), (2, 2), (1, 4), (2, 4)))
            encW, encX = _draw_enc(rng, p, q)
            R = rng.choice((1, 3, 3, 5))
            c = dict(kind=kind, N=_log_int(rng, 1, 32), H=_log_int(rng, 7, 64), W=_log_int(rng, 7, 64),
                     Cin=32 * _log_int(rng, 1, 16), Cout=32 * _log_int(rng, 1, 16), R=R, stride=rng.choice((1, 1, 2)),
                     pad=R // 2, p=p, q=q, encW=encW, encX=encX)
            if c["N"] * c["H"] * c["W"] * c["Cin"] * c["Cout"] * R * R <= 30e9:
                break
        if kind == "conv":
            c.update(q_out=2, pool=rng.choice((0, 0, 1)))
        return c
    if kind == "network":
        net = rng.choice(sorted(_NETS))
        hw = rng.randint(128, 256)
        macs = sum(_macs(L, 1) for L in _NETS[net](hw))
        return dict(kind=kind, net=net, batch=_log_int(rng, 1, max(1, min(128, int(230e9 / macs)))), hw=hw)
    return dict(kind="quantize", rows=_log_int(rng, 64, 4096), K=_log_int(rng, 64, 4096), bits=rng.choice((1, 2, 4, 8)))


# ---- inputs -----------------------------------------------------------------------------------------------------

def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _codes(g, shape, bits, enc):
    """Uniform codes, one per byte; -1/+1 as signed bytes (the distributions of workloads.py)."""
    if enc == _PM1:
        return torch.randint(0, 2, shape, generator=g, device="cuda", dtype=torch.int8) * 2 - 1
    return torch.randint(0, 1 << bits, shape, generator=g, device="cuda", dtype=torch.uint8)


def _levels(bits, enc):
    """Mean and variance of one operand value."""
    if enc == _PM1:
        return 0.0, 1.0
    return ((1 << bits) - 1) / 2.0, (4.0 ** bits - 1.0) / 12.0


def _affine(g, c, K):
    """Per-channel scale and bias that spread the layer's results over the four codes."""
    (mw, vw), (mx, vx) = _levels(c["p"], c["encW"]), _levels(c["q"], c["encX"])
    var = K * (vw * vx + vw * mx * mx + vx * mw * mw)
    scale = (1.0 + 0.1 * torch.randn(c["Cout"], generator=g, device="cuda")) / math.sqrt(var)
    centre = 1.0 if c.get("pool") else 2.0
    bias = centre - scale * (K * mw * mx) + 0.1 * torch.randn(c["Cout"], generator=g, device="cuda")
    return scale.contiguous(), bias.contiguous()


def _net_params(layers, g):
    """The recipe of `workloads.network_params` (fair -1/+1 weights, folded batch-norm constants from the closed-form
    statistics of their sums), drawn on the GPU: the largest of these networks has 138 million weights."""
    by_name = {L.name: L for L in layers}
    out = {}
    for L in layers:
        if L.kind not in ("conv", "fc"):
            continue
        K = L.Cin * L.R * L.S
        src = by_name.get(L.src)
        if src is None:
            mu, v = 127.5, (256.0 ** 2 - 1.0) / 12.0
        elif src.kind == "maxpool" or (src.kind == "conv" and src.pool):
            mu, v = 1.41, 0.5
        elif src.kind == "sumpool":
            mu, v = 1.5 * src.H * src.W, 1.0 * src.H * src.W
        else:
            mu, v = 1.5, 1.0
        w = torch.randint(0, 2, (L.Cout, L.Cin, L.R, L.S), generator=g, device="cuda", dtype=torch.int8) * 2 - 1
        wsum = w.view(L.Cout, -1).sum(1, dtype=torch.int32).double()
        a = (1.0 + 0.1 * torch.randn(L.Cout, generator=g, device="cuda").double()) / math.sqrt(K * v)
        pooled = L.pool or any(M.kind == "maxpool" and M.src == L.name for M in layers)
        centre = (0.5 if src is None or pooled else 2.0) - (1.5 * L.res_scale if L.res else 0.0)
        b = centre - a * mu * wsum + 0.1 * torch.randn(L.Cout, generator=g, device="cuda").double()
        out[L.name] = (w.cpu().numpy(), a.float().cpu().numpy(), b.float().cpu().numpy())
    return out


def _conv(c):
    return B.Conv(c["N"], c["H"], c["W"], c["Cin"], c["Cout"], c["R"], c["R"], c["stride"], c["pad"],
                  c["p"], c["q"], c["encW"], c["encX"])


def prepare(case, seed):
    g, c, kind = _generator(seed), case, case["kind"]
    s = {"case": c, "kind": kind}
    empty = lambda n: torch.empty(n, dtype=torch.int32, device="cuda")  # noqa: E731
    if kind == "gemm":
        s["W"] = B.apnn_pack(_codes(g, (c["M"], c["K"]), c["p"], c["encW"]), c["p"], c["encW"])
        s["x"] = _codes(g, (c["N"], c["K"]), c["q"], c["encX"])
        s["X"] = empty(B.apnn_packed_words(c["N"], c["K"], c["q"]))
        s["Y"] = torch.empty((c["M"], c["N"]), dtype=torch.int32, device="cuda")
    elif kind == "fc":
        s["d"] = B.Conv(c["N"], 1, 1, c["Cin"], c["Cout"], p=c["p"], q=c["q"], encW=c["encW"], encX=c["encX"])
        s["W"] = B.apnn_pack(_codes(g, (c["Cout"], c["Cin"]), c["p"], c["encW"]), c["p"], c["encW"])
        s["X"] = B.apnn_pack(_codes(g, (c["N"], c["Cin"]), c["q"], c["encX"]), c["q"], c["encX"])
        s["scale"], s["bias"] = _affine(g, c, c["Cin"])
        s["Y"] = empty(B.apnn_fmap_words(c["N"], c["Cout"], c["q_out"]))
    elif kind in ("conv", "conv2d"):
        s["d"] = d = _conv(c)
        s["W"] = B.apnn_pack_conv_weights(_codes(g, (c["Cout"], c["Cin"], c["R"], c["R"]), c["p"], c["encW"]), c["p"], c["encW"])
        x = _codes(g, (c["N"], c["Cin"], c["H"], c["W"]), c["q"], c["encX"])
        if kind == "conv":
            s["X"] = B.apnn_pack_fmap(x, B.LAYOUT_NCHW, c["q"], c["encX"])
            s["scale"], s["bias"] = _affine(g, c, c["Cin"] * c["R"] ** 2)
            s["Y"] = empty(B.apnn_fmap_words(_pixels(c), c["Cout"], c["q_out"]))
        else:
            s["x"] = x
            s["X"] = empty(B.apnn_fmap_words(c["N"] * c["H"] * c["W"], c["Cin"], c["q"]))
            s["Y"] = torch.empty((c["N"], d.Ho, d.Wo, c["Cout"]), dtype=torch.int32, device="cuda")
    elif kind == "network":
        layers = _NETS[c["net"]](c["hw"])
        s["net"] = PackedNet(layers, _net_params(layers, g), c["batch"])
        s["image"] = torch.randint(0, 256, (c["batch"], 3, c["hw"], c["hw"]), generator=g, device="cuda", dtype=torch.uint8)
    else:
        # activations as a normalised layer leaves them; the step spreads them over the codes
        s["x"] = torch.randn((c["rows"], c["K"]), generator=g, device="cuda")
        s["zero"], s["step"] = -2.0, 4.0 / (1 << c["bits"])
        s["Y"] = empty(B.apnn_packed_words(c["rows"], c["K"], c["bits"]))
    return s


def run(s):
    c, kind = s["case"], s["kind"]
    if kind == "gemm":
        B.apnn_pack(s["x"], c["q"], c["encX"], out=s["X"])
        return B.apnn_gemm(s["W"], s["X"], c["M"], c["N"], c["K"], c["p"], c["q"], c["encW"], c["encX"], out=s["Y"])
    if kind == "fc":
        return B.apnn_layer(s["d"], s["W"], s["X"], is_gemm=True, q_out=c["q_out"], scale=s["scale"], bias=s["bias"], out=s["Y"])
    if kind == "conv":
        return B.apnn_layer(s["d"], s["W"], s["X"], q_out=c["q_out"], scale=s["scale"], bias=s["bias"], out=s["Y"],
                            pool=B.POOL_MAX2 if c["pool"] else B.POOL_NONE)
    if kind == "conv2d":
        B.apnn_pack_fmap(s["x"], B.LAYOUT_NCHW, c["q"], c["encX"], out=s["X"])
        return B.apnn_conv2d(s["d"], s["W"], s["X"], out=s["Y"])
    if kind == "network":
        return s["net"].forward(s["image"])
    return B.apnn_quantize(s["x"], s["zero"], s["step"], c["bits"], out=s["Y"])


# ---- what a pass cannot do without ------------------------------------------------------------------------------

def _pixels(c):
    Ho, Wo = ((c[k] + 2 * c["pad"] - c["R"]) // c["stride"] + 1 for k in ("H", "W"))
    return c["N"] * ((Ho // 2) * (Wo // 2) if c.get("pool") else Ho * Wo)


def _macs(L, batch):
    return batch * L.Ho * L.Wo * L.Cout * L.Cin * L.R * L.S if L.kind in ("conv", "fc") else 0


def work(case):
    c, kind = case, case["kind"]
    if kind == "gemm":      # activation codes and weight planes in, int32 out
        return {"bytes": c["N"] * c["K"] + c["M"] * c["K"] * c["p"] / 8 + 4 * c["M"] * c["N"], "flops": 2 * c["M"] * c["N"] * c["K"]}
    if kind == "fc":        # planes in, planes out
        return {"bytes": c["Cin"] * (c["N"] * c["q"] + c["Cout"] * c["p"]) / 8 + 8 * c["Cout"] + c["N"] * c["Cout"] * c["q_out"] / 8,
                "flops": 2 * c["N"] * c["Cin"] * c["Cout"]}
    if kind in ("conv", "conv2d"):
        pix = c["N"] * c["H"] * c["W"] * c["Cin"]
        weights = c["Cout"] * c["Cin"] * c["R"] ** 2
        flops = 2 * weights * _pixels(dict(c, pool=0))
        if kind == "conv":
            return {"bytes": (pix * c["q"] + weights * c["p"] + _pixels(c) * c["Cout"] * c["q_out"]) / 8 + 8 * c["Cout"], "flops": flops}
        return {"bytes": pix + weights * c["p"] / 8 + 4 * _pixels(c) * c["Cout"], "flops": flops}
    if kind == "network":   # image, weight planes and per-channel constants in, logits out
        layers = _NETS[c["net"]](c["hw"])
        bytes_ = c["batch"] * 3 * c["hw"] ** 2 + 4 * c["batch"] * layers[-1].Cout
        bytes_ += sum(L.Cout * L.Cin * L.R * L.S / 8 + 8 * L.Cout for L in layers if L.kind in ("conv", "fc"))
        return {"bytes": bytes_, "flops": 2 * sum(_macs(L, c["batch"]) for L in layers)}
    return {"bytes": c["rows"] * c["K"] * (4 + c["bits"] / 8), "flops": 0}


def tolerance(case):
    """Codes, planes and int32 sums: whole numbers, the same for every correct implementation."""
    return "exact"
