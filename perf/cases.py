"""What a user of this library has it compute, as cases to time and to compare.

Each case is a layer, or a short run of layers, through the public Python entry points, with the sizes of the
library's own workloads and layer table or generic ones beside them.  `listed()` names twelve; `draw(rng)` gives
more of the same ranges: batches of 1 to 32 images, planes of 7 to 224 pixels a side (odd ones among them), few to
many channels, strides 1 and 2, the four element formats in channel-first and channel-last layout.

All tensors are dense; inputs are N(0, 1) as after a normalisation layer, weights N(0, 2 / fan-in), quantised
tensors uniform over int8, requantisation scales such that results fill the int8 range.
"""
import math

import torch

import paper_2310_05218_amd as sw


def listed():
    return [
        # one single-channel image under one small filter (edge or blur filters): the smallest call, all latency
        {"name": "image_3x3", "kind": "image", "N": 1, "H": 256, "W": 256, "R": 3, "pad": 0},
        # 64 long signals: a nine-tap filter, moving average and moving maximum (three calls on one input)
        {"name": "signals_64x65536", "kind": "signals", "N": 64, "L": 65536, "k": 9, "window": 8},
        # the standard 3x3 layer of a residual network's first stage, training-size batch
        {"name": "conv3x3_64", "kind": "conv", "N": 32, "C": 64, "H": 56, "W": 56, "K": 64, "R": 3, "stride": 1, "pad": 1, "dil": 1, "relu": False},
        # the first layers of an image network: 7x7 stride 2 over RGB with bias and rectifier, then 3x3 stride-2 max pooling
        {"name": "stem_rgb_7x7_pool", "kind": "stem", "N": 32, "H": 224, "W": 224, "K": 64},
        # the channel-reducing 1x1 layer of a bottleneck, bias and rectifier fused
        {"name": "conv1x1_256to64", "kind": "conv", "N": 32, "C": 256, "H": 56, "W": 56, "K": 64, "R": 1, "stride": 1, "pad": 0, "dil": 1, "relu": True},
        # the same kind of 3x3 layer late in the network for a single image: what a latency-bound server runs
        {"name": "conv3x3_256_one_image", "kind": "conv", "N": 1, "C": 256, "H": 14, "W": 14, "K": 256, "R": 3, "stride": 1, "pad": 1, "dil": 1, "relu": True},
        # odd planes and channel counts off the powers of two, a small batch
        {"name": "conv3x3_ragged", "kind": "conv", "N": 5, "C": 96, "H": 35, "W": 35, "K": 136, "R": 3, "stride": 1, "pad": 1, "dil": 1, "relu": True},
        # depthwise layers, 3x3 and 7x7, of separable and large-kernel networks (two calls on one input)
        {"name": "depthwise_3x3_7x7", "kind": "depthwise2", "N": 32, "C": 256, "H": 56, "W": 56},
        # a down-sampling depthwise layer on an odd plane, bias and rectifier fused
        {"name": "depthwise_5x5_s2_ragged", "kind": "depthwise", "N": 8, "C": 144, "H": 75, "W": 75, "R": 5, "stride": 2, "dtype": "f32"},
        # the quantised 3x3 layer with exact int32 sums, channel first
        {"name": "conv3x3_s8", "kind": "conv_s8", "N": 32, "C": 128, "H": 28, "W": 28, "K": 128, "R": 3, "stride": 1, "pad": 1, "requant": False},
        # the first-stage 3x3 layer as inference engines run it: bf16, channel last
        {"name": "conv3x3_bf16_nhwc", "kind": "conv_nhwc", "N": 32, "C": 64, "H": 56, "W": 56, "K": 64, "R": 3, "stride": 1, "pad": 1, "dtype": "bf16"},
        # a quantised bottleneck, channel last, int8 between its layers: 1x1, 3x3, 1x1 (three dependent calls)
        {"name": "bottleneck_s8_nhwc", "kind": "bottleneck_s8", "N": 32, "H": 28, "W": 28, "C": 512, "K": 128},
    ]


def _log(rng, lo, hi):
    """A whole number between lo and hi, spread over its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case.  Caps on the work keep a drawn case below the largest listed one."""
    while True:
        kind = rng.choice(["image", "signals", "conv", "conv", "conv", "stem", "depthwise", "depthwise",
                           "conv_s8", "conv_nhwc", "conv_nhwc", "bottleneck_s8"])
        c = {"kind": kind}
        n = _log(rng, 1, 32)
        side = _log(rng, 7, 112)
        side2 = side if rng.random() < 0.7 else _log(rng, 7, 112)
        if kind == "image":
            c.update(N=_log(rng, 1, 8), H=_log(rng, 64, 512), W=_log(rng, 64, 512), R=rng.choice([3, 5, 7]))
            c["pad"] = rng.choice([0, c["R"] // 2])
        elif kind == "signals":
            c.update(N=_log(rng, 1, 128), L=_log(rng, 4096, 131072), k=_log(rng, 2, 33), window=_log(rng, 2, 33))
            if c["N"] * c["L"] > 8 << 20:
                continue
        elif kind == "conv":
            r = rng.choice([1, 1, 3, 3, 3, 5])
            ch = lambda: 8 * _log(rng, 2, 64) if rng.random() < 0.85 else _log(rng, 9, 200)
            c.update(N=n, C=ch(), H=side, W=side2, K=ch(), R=r, stride=rng.choice([1, 1, 2]), dil=rng.choice([1, 1, 1, 2]) if r == 3 else 1,
                     relu=rng.random() < 0.5)
            c["pad"] = c["dil"] * (r // 2)
            if c["dil"] > 1:
                c["relu"] = False
            if min(side, side2) < c["dil"] * (r - 1) + 1 or not 1e7 < work(c)["flops"] < 4e9 or work(c)["bytes"] > 1.2e8:
                continue
        elif kind == "stem":
            c.update(N=n, H=_log(rng, 96, 256), W=_log(rng, 96, 256), K=rng.choice([32, 48, 64]))
            if c["N"] * c["H"] * c["W"] * c["K"] > 32 * 224 * 224 * 64:
                continue
        elif kind == "depthwise":
            c.update(N=n, C=8 * _log(rng, 4, 96), H=side, W=side2, R=rng.choice([3, 3, 5, 7]), stride=rng.choice([1, 1, 2]),
                     dtype=rng.choice(["f32", "f32", "bf16"]))
            if c["R"] ** 2 * n * c["C"] * side * side2 > 1.5e8 * (1 if c["dtype"] == "bf16" else 3):
                continue
        elif kind == "conv_s8":
            r = rng.choice([1, 3, 3])
            c.update(N=n, C=16 * _log(rng, 2, 24), H=side, W=side2, K=16 * _log(rng, 2, 24), R=r, stride=rng.choice([1, 1, 2]), pad=r // 2,
                     requant=rng.random() < 0.5)
            if not 1e7 < work(c)["flops"] < 4e9:
                continue
        elif kind == "conv_nhwc":
            r = rng.choice([1, 3, 3, 5])
            c.update(N=n, C=16 * _log(rng, 1, 32), H=side, W=side2, K=16 * _log(rng, 1, 32), R=r, stride=rng.choice([1, 1, 2]), pad=r // 2,
                     dtype=rng.choice(["bf16", "bf16", "f16", "f32"]))
            if rng.random() < 0.15:     # the first layer of such a network: three channels
                c.update(N=min(n, 4), C=3, H=_log(rng, 64, 224), W=_log(rng, 64, 224), K=rng.choice([32, 64]), R=3, stride=2, pad=1)
            if not 1e7 < work(c)["flops"] < 4e9 or work(c)["bytes"] > 1.2e8:
                continue
        else:
            c.update(N=n, H=side, W=side2, K=32 * _log(rng, 1, 8))
            c["C"] = 4 * c["K"]
            if work(c)["flops"] > 6e9:
                continue
        return c


def _out(n, k, stride, pad, dil=1):
    return (n + 2 * pad - dil * (k - 1) - 1) // stride + 1


def work(case):
    """Bytes (each input once, each output once) and operations (two a multiply-add) of one pass."""
    k = case["kind"]
    if k == "image":
        ho, wo = _out(case["H"], case["R"], 1, case["pad"]), _out(case["W"], case["R"], 1, case["pad"])
        return {"bytes": 4 * case["N"] * (case["H"] * case["W"] + ho * wo), "flops": 2 * case["R"] ** 2 * case["N"] * ho * wo}
    if k == "signals":
        n, lo, lp = case["N"], case["L"] - case["k"] + 1, case["L"] - case["window"] + 1
        return {"bytes": 4 * n * (case["L"] + lo + 2 * lp), "flops": n * (2 * case["k"] * lo + (2 * case["window"] - 1) * lp)}
    if k == "stem":
        ho, wo = _out(case["H"], 7, 2, 3), _out(case["W"], 7, 2, 3)
        hp, wp = _out(ho, 3, 2, 1), _out(wo, 3, 2, 1)
        return {"bytes": 4 * case["N"] * (3 * case["H"] * case["W"] + case["K"] * (ho * wo + hp * wp)) + 4 * 148 * case["K"],
                "flops": case["N"] * case["K"] * (2 * 147 * ho * wo + 8 * hp * wp)}
    if k == "depthwise2":
        px = case["N"] * case["C"] * case["H"] * case["W"]
        return {"bytes": 4 * 3 * px + 4 * 58 * case["C"], "flops": 2 * 58 * px}
    if k == "bottleneck_s8":
        px, c, m = case["N"] * case["H"] * case["W"], case["C"], case["K"]
        return {"bytes": px * (2 * c + 2 * m) + 2 * c * m + 9 * m * m + 8 * (c + 2 * m), "flops": 2 * px * (2 * c * m + 9 * m * m)}
    r, st = case["R"], case["stride"]
    if k == "depthwise":
        ho, wo, e = _out(case["H"], r, st, r // 2), _out(case["W"], r, st, r // 2), 2 if case["dtype"] == "bf16" else 4
        planes = case["N"] * case["C"]
        return {"bytes": e * planes * (case["H"] * case["W"] + ho * wo) + 4 * case["C"] * (r * r + 1), "flops": 2 * r * r * planes * ho * wo}
    dil = case.get("dil", 1)
    ho, wo = _out(case["H"], r, st, case["pad"], dil), _out(case["W"], r, st, case["pad"], dil)
    outs = case["N"] * case["K"] * ho * wo
    if k == "conv_s8":
        e_in, e_out = 1, 1 if case["requant"] else 4
    elif k == "conv_nhwc":
        e_in = e_out = 4 if case["dtype"] == "f32" else 2
    else:
        e_in = e_out = 4
    return {"bytes": e_in * (case["N"] * case["C"] * case["H"] * case["W"] + case["K"] * case["C"] * r * r) + e_out * outs,
            "flops": 2 * outs * case["C"] * r * r}


_DT = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}


def prepare(case, seed):
    """Inputs and weights on the GPU, from the seed alone."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    nrm = lambda *s, std=1.0: torch.randn(s, generator=g, device="cuda") * std
    s8 = lambda *s: torch.randint(-128, 128, s, generator=g, device="cuda", dtype=torch.int8)
    s = dict(case)
    k = case["kind"]
    if k == "image":
        s["x"] = nrm(case["N"], 1, case["H"], case["W"])
        s["w"] = nrm(1, 1, case["R"], case["R"], std=1.0 / case["R"])
    elif k == "signals":
        s["x"] = nrm(case["N"], case["L"])
        s["w"] = nrm(case["k"], std=case["k"] ** -0.5)
    elif k == "stem":
        s["x"] = nrm(case["N"], 3, case["H"], case["W"])
        s["w"] = nrm(case["K"], 3, 7, 7, std=(2.0 / 147) ** 0.5)
        s["b"] = nrm(case["K"], std=0.5)
    elif k == "depthwise2":
        s["x"] = nrm(case["N"], case["C"], case["H"], case["W"])
        s["w3"], s["w7"] = nrm(case["C"], 1, 3, 3, std=1 / 3), nrm(case["C"], 1, 7, 7, std=1 / 7)
    elif k == "depthwise":
        s["x"] = nrm(case["N"], case["C"], case["H"], case["W"]).to(_DT[case["dtype"]])
        s["w"] = nrm(case["C"], 1, case["R"], case["R"], std=1 / case["R"])
        s["b"] = nrm(case["C"], std=0.5)
    elif k == "conv":
        s["x"] = nrm(case["N"], case["C"], case["H"], case["W"])
        s["w"] = nrm(case["K"], case["C"], case["R"], case["R"], std=(2.0 / (case["C"] * case["R"] ** 2)) ** 0.5)
        s["b"] = nrm(case["K"], std=0.5)
    elif k == "conv_nhwc":
        s["x"] = nrm(case["N"], case["H"], case["W"], case["C"]).to(_DT[case["dtype"]])
        s["w"] = nrm(case["K"], case["R"], case["R"], case["C"], std=(2.0 / (case["C"] * case["R"] ** 2)) ** 0.5).to(_DT[case["dtype"]])
        s["b"] = nrm(case["K"], std=0.5)
    elif k == "conv_s8":
        s["x"], s["w"] = s8(case["N"], case["C"], case["H"], case["W"]), s8(case["K"], case["C"], case["R"], case["R"])
        s["b"], s["s"] = _requant(g, case["K"], case["C"] * case["R"] ** 2, 74.0)
    else:
        c, m = case["C"], case["K"]
        s["x"] = s8(case["N"], case["H"], case["W"], c)
        s["w1"], s["w2"], s["w3"] = s8(m, 1, 1, c), s8(m, 3, 3, m), s8(c, 1, 1, m)
        # a rectified int8 input has about the root mean square 32 that these scales give it
        (s["b1"], s["s1"]), (s["b2"], s["s2"]), (s["b3"], s["s3"]) = _requant(g, m, c, 74.0), _requant(g, m, 9 * m, 32.0), _requant(g, c, m, 32.0)
    return s


def _requant(g, n, terms, rms_x):
    """Biases and scales of n channels whose sums have `terms` products: results spread over the int8 range."""
    rms = rms_x * 74.0 * terms ** 0.5
    bias = (torch.randn(n, generator=g, device="cuda") * 0.3 * rms).to(torch.int32)
    return bias, (torch.rand(n, generator=g, device="cuda") * 0.5 + 0.75) * (45.0 / rms)


def run(s):
    k = s["kind"]
    if k == "image":
        return sw.sw_conv2d(s["x"], s["w"], 1, s["pad"])
    if k == "signals":
        return (sw.sw_conv1d(s["x"], s["w"]), sw.sw_pool1d(s["x"], s["window"], 1, sw.SW_POOL_AVG),
                sw.sw_pool1d(s["x"], s["window"], 1, sw.SW_POOL_MAX))
    if k == "stem":
        y = sw.sw_conv2d_bias_relu(s["x"], s["w"], s["b"], 2, 3, True)
        return y, sw.sw_pool2d(y, 3, 3, 2, 1, sw.SW_POOL_MAX)
    if k == "depthwise2":
        return sw.sw_conv2d_depthwise(s["x"], s["w3"], 1, 1), sw.sw_conv2d_depthwise(s["x"], s["w7"], 1, 3)
    if k == "depthwise":
        if s["dtype"] == "bf16":
            return sw.sw_conv2d_depthwise_bf16(s["x"], s["w"], s["stride"], s["R"] // 2)
        return sw.sw_conv2d_depthwise_bias_relu(s["x"], s["w"], s["b"], s["stride"], s["R"] // 2, True)
    if k == "conv":
        if s["dil"] > 1:
            return sw.sw_conv2d_dilated(s["x"], s["w"], s["stride"], s["pad"], s["dil"])
        if s["relu"]:
            return sw.sw_conv2d_bias_relu(s["x"], s["w"], s["b"], s["stride"], s["pad"], True)
        return sw.sw_conv2d(s["x"], s["w"], s["stride"], s["pad"])
    if k == "conv_nhwc":
        return sw.sw_conv2d_nhwc(s["x"], s["w"], s["stride"], s["pad"], 1, s["b"], True)
    if k == "conv_s8":
        if s["requant"]:
            return sw.sw_conv2d_s8_requant(s["x"], s["w"], s["b"], s["s"], s["stride"], s["pad"], True)
        return sw.sw_conv2d_s8(s["x"], s["w"], s["stride"], s["pad"])
    y1 = sw.sw_conv2d_s8_nhwc(s["x"], s["w1"], 1, 0, s["b1"], s["s1"], True)
    y2 = sw.sw_conv2d_s8_nhwc(y1, s["w2"], 1, 1, s["b2"], s["s2"], True)
    return y1, y2, sw.sw_conv2d_s8_nhwc(y2, s["w3"], 1, 0, s["b3"], s["s3"], False)


def _conv64(x, w, stride, pad, dil=1):
    """The convolution of x [N,C,H,W] under w [K,C,R,S] (or [C,1,R,S]: one filter a channel) in float64, tap by tap."""
    x, w = x.double(), w.double()
    n, c, h, wd = x.shape
    k, cw, r, s = w.shape
    ho, wo = _out(h, r, stride, pad, dil), _out(wd, s, stride, pad, dil)
    xz = torch.zeros((n, c, h + 2 * pad, wd + 2 * pad), dtype=torch.float64, device=x.device)
    xz[:, :, pad:pad + h, pad:pad + wd] = x
    y = torch.zeros((n, k, ho, wo), dtype=torch.float64, device=x.device)
    for i in range(r):
        for j in range(s):
            win = xz[:, :, i * dil:i * dil + (ho - 1) * stride + 1:stride, j * dil:j * dil + (wo - 1) * stride + 1:stride]
            if cw == 1 and k == c:
                y += win * w[:, 0, i, j].view(1, k, 1, 1)
            else:
                for b in range(n):
                    y[b] += (w[:, :, i, j].contiguous() @ win[b].reshape(c, ho * wo)).view(k, ho, wo)
    return y


def _sums(x, w, stride, pad):
    """Exact integer sums: float64 holds them below 2^53."""
    return _conv64(x, w, stride, pad).to(torch.int64)


def _quant(acc, bias, scale, relu, shape):
    """clamp(round-to-even(scale * float32(acc + bias))), the float32 steps the entry points define."""
    v = (acc + bias.to(torch.int64).view(shape)).to(torch.float32) * scale.view(shape)
    return torch.clamp(torch.round(v), 0 if relu else -128, 127).to(torch.int8)


def exact(case, seed):
    """What run() returns for these inputs, in 64 bits and plain torch."""
    s = prepare(case, seed)
    k = case["kind"]
    if k == "image":
        return _conv64(s["x"], s["w"], 1, s["pad"])
    if k == "signals":
        x = s["x"].double()
        lo, lp = x.shape[1] - s["k"] + 1, x.shape[1] - s["window"] + 1
        w = s["w"].double()
        conv = sum(w[j] * x[:, j:j + lo] for j in range(s["k"]))
        avg = sum(x[:, j:j + lp] for j in range(s["window"])) / s["window"]
        mx = x[:, :lp]
        for j in range(1, s["window"]):
            mx = torch.maximum(mx, x[:, j:j + lp])
        return conv, avg, mx
    if k == "stem":
        y = torch.relu(_conv64(s["x"], s["w"], 2, 3) + s["b"].double().view(1, -1, 1, 1))
        return y, torch.nn.functional.max_pool2d(y, 3, 2, 1)
    if k == "depthwise2":
        return _conv64(s["x"], s["w3"], 1, 1), _conv64(s["x"], s["w7"], 1, 3)
    if k == "depthwise":
        y = _conv64(s["x"], s["w"], s["stride"], s["R"] // 2)
        return y if s["dtype"] == "bf16" else torch.relu(y + s["b"].double().view(1, -1, 1, 1))
    if k == "conv":
        y = _conv64(s["x"], s["w"], s["stride"], s["pad"], s["dil"])
        return torch.relu(y + s["b"].double().view(1, -1, 1, 1)) if s["relu"] else y
    if k == "conv_nhwc":
        y = _conv64(s["x"].permute(0, 3, 1, 2), s["w"].permute(0, 3, 1, 2), s["stride"], s["pad"])
        return torch.relu(y + s["b"].double().view(1, -1, 1, 1)).permute(0, 2, 3, 1).contiguous()
    if k == "conv_s8":
        acc = _sums(s["x"], s["w"], s["stride"], s["pad"])
        return _quant(acc, s["b"], s["s"], True, (1, -1, 1, 1)) if s["requant"] else acc.to(torch.int32)
    p = lambda t: t.permute(0, 3, 1, 2)
    y1 = _quant(_sums(p(s["x"]), p(s["w1"]), 1, 0), s["b1"], s["s1"], True, (1, -1, 1, 1))
    y2 = _quant(_sums(y1, p(s["w2"]), 1, 1), s["b2"], s["s2"], True, (1, -1, 1, 1))
    y3 = _quant(_sums(y2, p(s["w3"]), 1, 0), s["b3"], s["s3"], False, (1, -1, 1, 1))
    return tuple(t.permute(0, 2, 3, 1).contiguous() for t in (y1, y2, y3))


def tolerance(case):
    """Whole numbers are exact.  The rest: about four times what the library showed against `exact` (32-bit sums of up
    to 25 x 200 products; one rounding to 16 bits)."""
    k = case["kind"]
    if k in ("conv_s8", "bottleneck_s8"):
        return "exact"
    dt = case.get("dtype", "f32")
    if dt == "bf16":
        return {"rel": 7e-3, "max": 2e-2}
    if dt == "f16":
        return {"rel": 9e-4, "max": 3e-3}
    return {"rel": 2e-6, "max": 2e-5}
