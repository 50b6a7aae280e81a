"""Performance cases: the update phase of a training step as programs run it through this package.

A case is a dict of plain values.  `listed()` names the ones that are always timed, `draw(rng)` gives further cases of
the same families over their whole range of sizes, `prepare` makes what a program holds before the call, `run` is one
pass through the public entry points, `work` the bytes and operations one pass cannot do without, `tolerance` how far
another correct implementation of the same precision may differ.

Families
  update   prune + compress of g [T x O], then dW = theta(g)^T h, through the two library calls of the package
  block    the same for the four linear layers of a transformer block, one after the other
  linear   an NMLinear / NMLinearReLU layer, forward and backward
  conv     the weight gradient of an NMConv2d layer (the backward pass of the first layer, or of one whose input
           gradient is taken elsewhere): the forward pass and the input gradient are the vendor library's
"""
from __future__ import annotations

import torch

import paper_2203_10991_amd as nm
from paper_2203_10991_amd import synth
from paper_2203_10991_amd.autograd import NMConfig, NMConv2d, NMLinear, NMLinearReLU

DEVICE = "cuda:0"
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
Q8_G_TOP = {"2:4": 57344.0 / 4.0, "1:2": 57344.0 / 2.0}     # e5m2: a kept value is at most the sum of its block
Q8_H_TOP = 448.0                                            # e4m3


def _update(name, T, O, I, dtype="bf16", pattern="2:4", mode=0, precision="native", transposed=False, sigma=2.5, zeros=0.1):
    return {"name": name, "family": "update", "T": T, "O": O, "I": I, "dtype": dtype, "pattern": pattern, "mode": mode,
            "precision": precision, "transposed": transposed, "sigma": sigma, "zeros": zeros}


def _linear(name, tokens, fin, fout, pattern="2:4", mode=0, precision="native", relu=False):
    return {"name": name, "family": "linear", "tokens": tokens, "in": fin, "out": fout, "pattern": pattern, "mode": mode,
            "precision": precision, "relu": relu, "sigma": 2.0, "zeros": 0.2}


def _conv(name, batch, cin, cout, side, precision="native", channels_last=False):
    return {"name": name, "family": "conv", "batch": batch, "cin": cin, "cout": cout, "side": side, "precision": precision,
            "channels_last": channels_last, "sigma": 3.0, "zeros": 0.5}


def listed():
    return [
        # a small layer (the smoke check's size): launches and host time are what counts
        _update("small_2of4", 512, 512, 256),
        # binary32 tensors at a small size, MVUE 1:2 (1024 tokens of a 1024 x 1024 layer)
        _update("fp32_1of2", 1024, 1024, 1024, dtype="f32", pattern="1:2", sigma=2.0, zeros=0.3),
        # transformer MLP: hidden 1024, FFN 4096, 32 x 512 tokens, MVUE 1:2
        _update("transformer_mlp_1of2", 16384, 4096, 1024, pattern="1:2", zeros=0.4),
        # one ViT-Base block, batch 64 at 197 positions: qkv, proj, fc1, fc2
        {"name": "vit_block_2of4", "family": "block", "tokens": 64 * 197, "width": 768, "pattern": "2:4", "sigma": 2.0, "zeros": 0.2},
        # fine-tuning batch of 8 images: a token count that is no multiple of 16, the paper's approximate estimator
        _linear("linear_ragged_approx", 8 * 197, 768, 3072, mode=1),
        # Linear + ReLU of the transformer MLP: the activation's backward is fused with the prune
        _linear("linear_relu", 16384, 1024, 4096, relu=True),
        # 8-bit update phase of ViT-Base fc2 inside a layer (scales, cast, prune, 8-bit product)
        _linear("linear_q8", 64 * 197, 3072, 768, precision="q8"),
        # ResNet-50 stage-1 3x3 convolution at batch 256, bf16
        _conv("conv3x3_64", 256, 64, 64, 56),
        # ResNet-50 14 x 14 stage, 8-bit
        _conv("conv3x3_256_q8", 256, 256, 256, 14, precision="q8"),
        # binary32 tensors through three bf16 terms, the gradient stored transposed, odd sizes
        _update("fp32_x3_transposed", 9328, 2960, 1976, dtype="f32", precision="bf16x3", transposed=True),
        # large decoder MLP layer: 32768 tokens, hidden 8192, FFN 28672
        _update("decoder_2of4", 32768, 28672, 8192),
        # the same layer on the 8-bit path
        _update("decoder_q8", 32768, 28672, 8192, precision="q8"),
    ]


def _log_int(rng, lo, hi, step):
    """A multiple of `step` in [lo, hi], spread over the logarithm of the range."""
    v = lo * (hi / lo) ** rng.random()
    return max(lo, min(hi, int(round(v / step)) * step))


def draw(rng):
    family = rng.choice(["update", "update", "update", "block", "linear", "linear", "conv"])
    if family == "update":
        form = rng.choice(["bf16", "bf16", "q8", "f32", "x3"])
        hi_t, hi_w, most = {"bf16": (32768, 28672, 4e12), "q8": (32768, 28672, 4e12), "f32": (16384, 8192, 1e11), "x3": (16384, 8192, 4e11)}[form]
        while True:
            T = _log_int(rng, 256, hi_t, 32 if form == "q8" else 16)
            O, I = _log_int(rng, 64, hi_w, 8), _log_int(rng, 64, hi_w, 16 if form == "q8" else 8)
            if T * O * I <= most:
                break
        pattern = rng.choice(["2:4", "2:4", "1:2"])
        c = _update("", T, O, I, dtype="f32" if form in ("f32", "x3") else "bf16", pattern=pattern,
                    mode=rng.choice([0, 0, 0, 1]) if pattern == "2:4" else 0,
                    precision={"q8": "q8", "x3": "bf16x3"}.get(form, "native"), transposed=rng.random() < 0.25,
                    sigma=rng.choice([2.0, 2.5]), zeros=rng.choice([0.1, 0.2, 0.3, 0.4]))
    elif family == "block":
        c = {"family": "block", "tokens": 16 * _log_int(rng, 32, 1024, 1), "width": _log_int(rng, 256, 1536, 8), "pattern": rng.choice(["2:4", "1:2"]),
             "sigma": 2.0, "zeros": 0.2}
    elif family == "linear":
        precision = rng.choice(["native", "native", "q8"])
        c = _linear("", _log_int(rng, 197, 16384, 1), _log_int(rng, 256, 4096, 16), _log_int(rng, 256, 4096, 8),
                    pattern=rng.choice(["2:4", "2:4", "1:2"]), mode=rng.choice([0, 0, 1]), precision=precision,
                    relu=precision == "native" and rng.random() < 0.5)
        if c["pattern"] == "1:2":
            c["mode"] = 0
    else:
        side = rng.choice([56, 28, 14, 7])
        batch = rng.choice([24, 32, 50, 64, 96, 128, 200, 256])
        ch = 64 * 56 // side
        c = _conv("", batch, rng.choice([ch, ch // 2]), ch, side, precision=rng.choice(["native", "q8"]), channels_last=rng.random() < 0.5)
    c.pop("name", None)
    return c


def _gh(case, T, O, I, seed, h_kind="normal"):
    """(g, h): gradients with lognormal magnitudes and exact zeros, activations normal or half-normal after a ReLU."""
    w = synth.Workload("case", T, O, I, case.get("dtype", "bf16"), case.get("pattern", "2:4"), 0.0, case["sigma"], case["zeros"], h_kind)
    return synth.make_device(w, seed, DEVICE)


def _layers(case):
    w = case["width"]
    return [(3 * w, w), (w, w), (4 * w, w), (w, 4 * w)]        # (out, in) of qkv, proj, fc1, fc2


def prepare(case, seed):
    s = {"case": case, "seed": int(seed) % (1 << 31)}
    if case["family"] == "update":
        g, h = _gh(case, case["T"], case["O"], case["I"], seed)
        s["g"], s["h"] = (g.t().contiguous() if case["transposed"] else g), h
    elif case["family"] == "block":
        s["gh"] = [_gh(case, case["tokens"], o, i, seed + 1000 * k) for k, (o, i) in enumerate(_layers(case))]
    elif case["family"] == "linear":
        cfg = NMConfig(nm=case["pattern"], mode=case["mode"], seed=s["seed"], precision=case["precision"])
        torch.manual_seed(int(seed))
        layer = (NMLinearReLU if case["relu"] else NMLinear)(case["in"], case["out"], cfg=cfg, device=DEVICE, dtype=torch.bfloat16)
        g, h = _gh(case, case["tokens"], case["out"], case["in"], seed)
        s["layer"], s["gy"], s["x"] = layer, g, h.requires_grad_()
    else:
        n, side, cin, cout = case["batch"], case["side"], case["cin"], case["cout"]
        cfg = NMConfig(seed=s["seed"], precision=case["precision"])
        torch.manual_seed(int(seed))
        layer = NMConv2d(cin, cout, 3, padding=1, bias=False, cfg=cfg, device=DEVICE, dtype=torch.bfloat16)
        g, h = _gh(case, n * side * side, cout, cin, seed, "relu")
        fmt = torch.channels_last if case["channels_last"] else torch.contiguous_format
        x = h.view(n, side, side, cin).permute(0, 3, 1, 2).contiguous(memory_format=fmt)
        s["gy"] = g.view(n, side, side, cout).permute(0, 3, 1, 2).contiguous(memory_format=fmt)
        s["layer"], s["y"] = layer, layer(x)
    return s


def _update_step(case, g, h, seed):
    """One layer's update phase: the compressed gradient and dW."""
    two, t = case["pattern"] == "2:4", case.get("transposed", False)
    kw = {"mode": case.get("mode", 0)} if two else {}
    if case.get("precision", "native") == "q8":
        sg, sh = nm.nm_q8_scale(g, Q8_G_TOP[case["pattern"]]), nm.nm_q8_scale(h, Q8_H_TOP)
        h8 = nm.nm_cast_e4m3(h, sh)
        prune = (nm.mvue_prune_2of4_q8_t if t else nm.mvue_prune_2of4_q8) if two else (nm.mvue_prune_1of2_q8_t if t else nm.mvue_prune_1of2_q8)
        vals, meta = prune(g, seed=seed, scale=sg, **kw)
        return vals, meta, nm.nm_update_gemm_q8(vals, meta, h8, alpha=(sg, sh))
    if t:
        vals, meta = (nm.mvue_prune_2of4_t if two else nm.mvue_prune_1of2_t)(g, seed=seed, **kw)
    else:
        vals, meta, _ = (nm.mvue_prune_2of4 if two else nm.mvue_prune_1of2)(g, seed=seed, **kw)
    return vals, meta, nm.nm_update_gemm(vals, meta, h, f32_as_bf16x3=case.get("precision") == "bf16x3")


def run(s):
    case = s["case"]
    if case["family"] == "update":
        return _update_step(case, s["g"], s["h"], s["seed"])
    if case["family"] == "block":
        return [_update_step(case, g, h, s["seed"] + k) for k, (g, h) in enumerate(s["gh"])]
    if case["family"] == "linear":
        layer = s["layer"]
        y = layer(s["x"])
        return (y.detach(),) + torch.autograd.grad(y, (s["x"], layer.weight, layer.bias), s["gy"])
    return torch.autograd.grad(s["y"], (s["layer"].weight,), s["gy"], retain_graph=True)


def _update_work(T, O, I, e, q8=False, products=1):
    """g and h read once, kept values, index words and dW written once; half of the products are executed."""
    kept = 1 if q8 else e
    return T * O * e + T * O // 2 * kept + T * O // 8 + T * I * e + O * I * 4, products * T * O * I


def work(case):
    if case["family"] == "update":
        q8, x3 = case["precision"] == "q8", case["precision"] == "bf16x3"
        e = 4 if case["dtype"] == "f32" else 2
        # binary32 has no sparse matrix instruction (every product is executed); three bf16 terms make six sparse products
        b, f = _update_work(case["T"], case["O"], case["I"], e, q8, 6 if x3 else 2 if e == 4 else 1)
    elif case["family"] == "block":
        parts = [_update_work(case["tokens"], o, i, 2) for o, i in _layers(case)]
        b, f = sum(p[0] for p in parts), sum(p[1] for p in parts)
    elif case["family"] == "linear":
        T, I, O = case["tokens"], case["in"], case["out"]
        # x, W, gy in; y, dx, dW, db out (bf16): forward and input gradient dense, the weight gradient half of the products
        b, f = 2 * (T * I + O * I + T * O) + 2 * (T * O + T * I + O * I + O), 5 * T * O * I
    else:
        T = case["batch"] * case["side"] ** 2
        b, f = 2 * (T * case["cin"] + T * case["cout"] + 9 * case["cin"] * case["cout"]), 9 * T * case["cin"] * case["cout"]
    return {"bytes": b, "flops": f}


def tolerance(case):
    """About four times the distance of today's results from binary64 sums of the same operands; index words and 8-bit
    codes are exact."""
    if case["family"] in ("linear", "conv"):
        return {"rel": 6e-3, "max": 1.6e-2}    # bf16 results: half a unit in the last place is 1.7e-3 in the 2-norm, 2^-8 at most
    if case.get("precision") == "q8":
        return {"rel": 3e-4, "max": 1.4e-2}    # the 8-bit matrix instruction adds a step's products in a window of its own: 7e-5
    return {"rel": 1.5e-6, "max": 1.5e-4}      # binary32 sums: 3e-7 in the 2-norm at 32768 tokens, 4e-5 at most
