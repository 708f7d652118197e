"""The work this library is timed on: whole quantised layers of a diffusion UNet through the public calls.

A case is one layer (or the nine-layer sweep of the benchmark): the activations are transformed and
quantised and the integer product is taken, as the layer of a sampler does once per denoising step.  The
weights are prepared beforehand, as a program that loads a model does once.

kind      calls of one pass
linear    hq_act_hadamard_quant + hq_int_linear                     (dynamic scales; also 1x1 layers)
fused     hq_act_quant_int_linear                                   (the same layer in one launch)
single    hq_act_hadamard_quant + hq_int_linear_single              (un-transformed weights, digit planes)
conv      hq_act_hadamard_quant + hq_int_conv2d                     (3x3, stride 1 or 2)
static    hq_act_hadamard_quant_static + hq_int_conv2d_static       (one scale for the tensor)
width     hq_act_hadamard_quant_width + hq_int_conv2d_width         (transform along the image width)
i8        hq_act_hadamard_quant / _i8 + hq_int_conv2d_i8            (8-bit weights, 8- or 4-bit activations)
sweep     every layer of benchmark configuration 5, in order
"""
import math

import numpy as np
import torch

import paper_2512_05746_amd as hq
import workloads

_DTYPE = {"f16": torch.float16, "f32": torch.float32}
_LINEAR = ("linear", "fused", "single")


def _linear(kind, m, k, n, a_bits=4, dtype="f16", bias=False, had_block=64):
    return {"kind": kind, "m": m, "k": k, "n": n, "a_bits": a_bits, "w_bits": 4, "dtype": dtype, "bias": bias,
            "had_block": had_block}


def _conv(kind, nb, h, w, cin, cout, stride=1, a_bits=4, w_bits=4, dtype="f16", bias=False, had_block=64):
    return {"kind": kind, "nb": nb, "h": h, "w": w, "cin": cin, "cout": cout, "stride": stride, "a_bits": a_bits,
            "w_bits": w_bits, "dtype": dtype, "bias": bias, "had_block": had_block}


def listed():
    cases = [
        # the smallest layer of the benchmark configurations (configuration 1): fp32, with a bias; latency counts
        ("linear_256_f32", _linear("linear", 256, 256, 256, dtype="f32", bias=True)),
        # the query/key/value projection of an attention block (configuration 2)
        ("linear_qkv", _linear("linear", 8192, 384, 1152)),
        # the widest feed-forward layer, 3-bit activations (configuration 4)
        ("linear_ffn_a3", _linear("linear", 2048, 960, 3840, a_bits=3)),
        # a 1x1 layer at the highest resolution, where the one-launch form is the faster one
        ("linear_one_launch", _linear("fused", 16 * 64 * 64, 192, 192)),
        # an attention projection in the scheme that leaves the weights un-transformed
        ("linear_single", _linear("single", 4096, 576, 1728)),
        # 3x3 layer with many channels on a small image, 3-bit activations (configuration 4)
        ("conv_a3_16x16x960", _conv("conv", 8, 16, 16, 960, 960, a_bits=3)),
        # 3x3 layer with one scale per tensor and timestep
        ("conv_static_32x32x384", _conv("static", 16, 32, 32, 384, 384)),
        # the downsampling convolution between the first two resolutions
        ("conv_down_64x64x192", _conv("conv", 16, 64, 64, 192, 192, stride=2)),
        # 3x3 layer transformed along the image width
        ("conv_width_16x16x576", _conv("width", 16, 16, 16, 576, 576, had_block=16)),
        # 3x3 layer at 8 bits
        ("conv_w8a8_32x32x384", _conv("i8", 16, 32, 32, 384, 384, a_bits=8, w_bits=8)),
        # an image that is no power of two, channel counts that are not multiples of a tile, a bias
        ("conv_ragged", _conv("conv", 3, 45, 27, 320, 200, bias=True)),
        # the benchmark itself: 3x3, 1x1 and attention layers at four resolutions, batch 16
        ("sweep_b16", {"kind": "sweep", "config": 5}),
    ]
    return [dict(case, name=name) for name, case in cases]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _sweep_ops(config):
    return sum(layer.ops for layer in workloads.config_layers(config))


def _channels(rng, lo, hi, ragged):
    """A channel count in [lo, hi]: a multiple of 64 (of 192 half of the time, the UNet's own unit), or, for
    the calls that take it, now and then any multiple of 8."""
    if ragged and rng.random() < 0.15:
        return 8 * _log_int(rng, lo // 8, hi // 8)
    unit = 192 if hi >= 192 and rng.random() < 0.5 else 64
    return unit * max(1, _log_int(rng, max(1, lo // unit), hi // unit))


def _block(rng, k):
    """The transform's block: 64, or the largest power of two that divides the channels."""
    return math.gcd(k, 64)


def draw(rng):
    kind = rng.choice(["linear", "linear", "fused", "single", "conv", "conv", "conv", "static", "width", "i8"])
    bias = rng.random() < 0.5
    limit = _sweep_ops(5) // 2      # well below the largest listed case
    if kind in _LINEAR:
        k = _channels(rng, 64, 960, kind == "linear")
        n = 8 * _log_int(rng, 8, 480)
        top = limit // (3 if kind == "single" else 2) // 2
        m = _log_int(rng, 64, max(64, min(65536, top // (k * n))))
        dtype = "f32" if kind == "linear" and rng.random() < 0.2 else "f16"
        if k % 64:                  # the few-channel form
            m = min(m, 8192)
        return _linear(kind, m, k, n, a_bits=rng.choice([4, 4, 3]), dtype=dtype, bias=bias, had_block=_block(rng, k))
    stride = 2 if kind in ("conv", "i8") and rng.random() < 0.25 else 1
    cin = _channels(rng, 64, 960, kind == "conv" and stride == 1)
    cout = 8 * _log_int(rng, 8, 120) if rng.random() < 0.4 else cin
    side = _log_int(rng, 8, 64)
    h, w = (side, side) if rng.random() < 0.6 else (side, _log_int(rng, 8, 64))
    had_block = _block(rng, cin)
    if kind == "width":             # the block lies along the image width
        w = 8 * max(1, w // 8)
        had_block = rng.choice([b for b in (8, 16, 32, 64) if w % b == 0])
    top = limit // (3 if kind == "width" else 1)
    if cin % 64:
        top //= 8
    nb = max(1, min(_log_int(rng, 1, 32), top // (18 * h * w * cin * cout)))
    a_bits, w_bits = rng.choice([4, 4, 3]), 4
    if kind == "i8":
        a_bits, w_bits = rng.choice([8, 8, 4]), 8
    return _conv(kind, nb, h, w, cin, cout, stride, a_bits, w_bits, "f16", bias, had_block)


# ---- inputs ------------------------------------------------------------------------------------------------

def _activations(gen, shape, dtype):
    """N(0, 1) with one channel in a hundred twenty times as large, as the activations of a UNet have."""
    x = torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32)
    k = shape[-1]
    channels = torch.randperm(k, generator=gen, device="cuda")[: max(1, round(0.01 * k))]
    x[..., channels] *= 20.0
    return x.to(dtype)


def _layer_state(case, gen):
    """Inputs of one layer: the activations, the prepared weights, the bias and a given scale."""
    kind, dtype = case["kind"], _DTYPE[case["dtype"]]
    if kind in _LINEAR:
        x_shape, k, n, taps = (case["m"], case["k"]), case["k"], case["n"], 1
    else:
        x_shape = (case["nb"], case["h"], case["w"], case["cin"])
        k, n, taps = case["cin"], case["cout"], 9
    x = _activations(gen, x_shape, dtype)
    w = (torch.randn((n, taps, k), generator=gen, device="cuda", dtype=torch.float32) * 0.02).to(dtype)
    bias = (torch.randn(n, generator=gen, device="cuda", dtype=torch.float32) * 0.01).to(dtype) if case["bias"] else None
    if kind == "single":
        wq, sw = hq.hq_quantize_weights_single(w[:, 0, :].contiguous(), case["had_block"], case["w_bits"])
    else:
        wq, sw = hq.hq_quantize_weights(w, 1 if kind == "width" else case["had_block"], case["w_bits"])
    if kind == "linear" or kind == "fused":
        wq = wq[:, 0, :]
    state = {"case": case, "x": x, "wq": wq, "sw": sw, "bias": bias}
    if kind in ("static", "width"):   # a learned scale: somewhat below the abs-max one, so that the clamp is at work
        state["scale"] = torch.full((1,), 1.0, device="cuda") * (x.float().std() * 3.0 / (2 ** (case["a_bits"] - 1) - 1))
    return state


def _sweep_cases(config):
    out = []
    for layer in workloads.config_layers(config):
        if layer.ksize == 3:
            nb, h, w, cin = layer.x_shape
            out.append(_conv("conv", nb, h, w, cin, layer.n_out, a_bits=layer.a_bits, dtype=layer.dtype))
        else:
            out.append(_linear("linear", layer.m, layer.k_in, layer.n_out, a_bits=layer.a_bits, dtype=layer.dtype))
    return out


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    if case["kind"] == "sweep":
        return {"case": case, "layers": [_layer_state(c, gen) for c in _sweep_cases(case["config"])]}
    return _layer_state(case, gen)


# ---- one pass ------------------------------------------------------------------------------------------------

def _run_layer(s):
    c, x, wq, sw, bias = s["case"], s["x"], s["wq"], s["sw"], s["bias"]
    kind, dtype = c["kind"], _DTYPE[c["dtype"]]
    if kind == "fused":
        return hq.hq_act_quant_int_linear(x, wq, sw, bias, c["had_block"], c["a_bits"], y_dtype=dtype)
    if kind == "static":
        xq = hq.hq_act_hadamard_quant_static(x, s["scale"], c["had_block"], c["a_bits"])
        return hq.hq_int_conv2d_static(xq, s["scale"], wq, sw, bias, ksize=3, stride=c["stride"], y_dtype=dtype)
    if kind == "width":
        xu3 = hq.hq_act_hadamard_quant_width(x, s["scale"], c["had_block"], c["a_bits"])
        return hq.hq_int_conv2d_width(xu3, s["scale"], wq, sw, bias, c["had_block"], y_dtype=dtype, stride=c["stride"])
    if kind == "i8":
        quant = hq.hq_act_hadamard_quant if c["a_bits"] == 8 else hq.hq_act_hadamard_quant_i8
        xq, sx = quant(x, c["had_block"], c["a_bits"])
        return hq.hq_int_conv2d_i8(xq, sx, wq, sw, bias, ksize=3, y_dtype=dtype, stride=c["stride"])
    xq, sx = hq.hq_act_hadamard_quant(x, c["had_block"], c["a_bits"])
    if kind == "single":
        return hq.hq_int_linear_single(xq, sx, wq, sw, bias, c["had_block"], y_dtype=dtype)
    if kind == "linear":
        return hq.hq_int_linear(xq, sx, wq, sw, bias, y_dtype=dtype)
    return hq.hq_int_conv2d(xq, sx, wq, sw, bias, ksize=3, stride=c["stride"], y_dtype=dtype)


def run(state):
    if state["case"]["kind"] == "sweep":
        return [_run_layer(s) for s in state["layers"]]
    return _run_layer(state)


# ---- what a pass cannot do without ---------------------------------------------------------------------------

def _layer_work(c):
    size = 2 if c["dtype"] == "f16" else 4
    if c["kind"] in _LINEAR:
        pixels = outputs = c["m"]
        k, n, taps = c["k"], c["n"], 1
    else:
        pixels = c["nb"] * c["h"] * c["w"]
        ho, wo = (c["h"] - 1) // c["stride"] + 1, (c["w"] - 1) // c["stride"] + 1
        outputs = c["nb"] * ho * wo
        k, n, taps = c["cin"], c["cout"], 9
    w_bytes = n * taps * k * c["w_bits"] // 8 * (3 if c["kind"] == "single" else 1) + 4 * n
    data = pixels * k * size + w_bytes + outputs * n * size + (n * size if c["bias"] else 0)
    # the product, and the transform of every activation (log2 of the block additions each)
    flops = 2 * outputs * n * taps * k + pixels * k * int(np.log2(c["had_block"]))
    return data, flops


def work(case):
    layers = _sweep_cases(case["config"]) if case["kind"] == "sweep" else [case]
    parts = [_layer_work(c) for c in layers]
    return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}


def tolerance(case):
    # Against the same layers in 64 bits the 2-norm error is 2.1e-4 (the rounding of fp16 results; 7e-8 for
    # fp32 ones) plus what flipped codes add: a value within one fp32 rounding of a tie moves its products by one
    # step, which brought single layers to 3e-4 .. 9e-4 (most where fp16 inputs put many values on ties).
    return {"rel": 2e-3}
