"""The work a user of this library has it do, as cases that can be timed.

A case is one pass through a public entry point of paper_2412_19867_amd.wq with everything a
program keeps between passes (plan, prepared weights, workspace, output buffer) in hand:

  conv      Plan.forward            one quantized Winograd convolution, F(2,3), F(4,3) or F(6,3)
  stack     Plan.forward, chained   the ResNet-block convolutions of a diffusion UNet: three
                                    resolutions, each conv reads the previous one's output
  direct    DirectPlan.forward      the group-quantized standard 3x3 convolution, W8A8 or W4A8
  linear    DirectPlan.forward      the group-quantized linear layer, W8A8 or W4A8
  weights   Plan.weight_prepare     the offline weight stage (run when a model is loaded)

Sizes, distributions and options are those of the layer sets in workloads.py, of the tests and of
bench.py; draw() spreads over the ranges between and around them.
"""
import math

import numpy as np
import torch

from paper_2412_19867_amd import wq


def _conv(name, N, H, W, Cin, Cout, m, g, acts="latent", scaled=False, integer=0):
    return {"name": name, "kind": "conv", "N": N, "H": H, "W": W, "Cin": Cin, "Cout": Cout, "m": m, "g": g,
            "acts": acts, "scaled": scaled, "integer": integer}


def listed():
    return [
        # the smallest layer in use: one image, few channels; launches and host work count
        _conv("conv_32x32_64", 1, 32, 32, 64, 64, 4, 32, acts="normal"),
        # first and last 3x3 stage of a ResNet-18 at batch 32: many tiles and a short reduction,
        # then 7x7 images (ragged for F(6,3)) and a long one
        _conv("resnet_56x56_64", 32, 56, 56, 64, 64, 6, 32, acts="relu"),
        _conv("resnet_7x7_512", 32, 7, 7, 512, 512, 6, 32, acts="relu"),
        # deep layer of a UNet at 512 px: few tiles, 59 MB of weights
        _conv("unet_16x16_1280", 2, 16, 16, 1280, 1280, 4, 64),
        # skip-concat layer of the same UNet with F(6,3), small groups and learned row scales
        _conv("unet_skip_64x64_960", 2, 64, 64, 960, 320, 6, 32, scaled=True),
        # nothing divides anything: an image of odd size, output channels that need padding
        _conv("ragged_45x61_192", 3, 45, 61, 192, 200, 4, 64),
        # fully-integer input and output transforms, one scale per transform matrix
        _conv("integer_64x64_640", 2, 64, 64, 640, 640, 4, 64, integer=1),
        # SDXL-scale UNet at 1024 px: 12 convolutions one after the other, the largest case
        {"name": "sdxl_stack", "kind": "stack", "N": 2, "size": 128, "base": 320, "depth": 4, "m": 4, "g": 64},
        # the standard convolution the paper compares against
        {"name": "direct_32x32_640", "kind": "direct", "N": 2, "H": 32, "W": 32, "Cin": 640, "Cout": 640, "g": 64,
         "bits": 8},
        # a transformer block's projection over an image's tokens, with 4-bit weights
        {"name": "linear_4096_1280_w4", "kind": "linear", "rows": 4096, "Cin": 1280, "Cout": 1280, "g": 64, "bits": 4},
        # a wide projection of a few rows (decode): its weights are all that is read
        {"name": "linear_16_5120", "kind": "linear", "rows": 16, "Cin": 5120, "Cout": 5120, "g": 64, "bits": 8},
        # loading a model: the weights of one deep UNet layer
        {"name": "weights_1280", "kind": "weights", "Cin": 1280, "Cout": 1280, "m": 4, "g": 64, "scaled": False},
    ]


# ---- drawn cases ----

def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _channels(rng, lo, hi, step):
    return max(step, (_log(rng, lo, hi) + step // 2) // step * step)


def _outputs(rng, lo, hi):   # mostly multiples of 32, sometimes any number
    return _log(rng, lo, hi) if rng.random() < 0.25 else _channels(rng, lo, hi, 32)


def _image(rng, lo, hi):
    h = _log(rng, lo, hi)
    return h, (h if rng.random() < 0.5 else min(hi, max(lo, int(h * rng.uniform(0.6, 1.7)))))


def draw(rng):
    while True:
        kind = rng.choices(("conv", "integer", "stack", "direct", "linear", "weights"), (50, 8, 10, 10, 14, 8))[0]
        if kind in ("conv", "integer"):
            m, g = rng.choice((4, 4, 4, 4, 6, 6, 6, 6, 2)), rng.choice((32, 32, 64, 64, 64, 128, 256))
            H, W = _image(rng, 6, 128)
            c = _conv(None, _log(rng, 1, 32), H, W, _channels(rng, 64, 2560, g), _outputs(rng, 32, 1280), m, g,
                      acts=rng.choice(("latent", "relu", "normal")), scaled=rng.random() < 0.25)
            del c["name"]
            if kind == "integer":
                c["integer"], c["scaled"] = rng.choice((1, 2)), rng.random() < 0.5
        elif kind == "stack":
            c = {"kind": "stack", "N": rng.choice((1, 2, 2, 3)), "size": _log(rng, 24, 128),
                 "base": 64 * rng.randint(1, 5), "depth": rng.choice((2, 3, 4)), "m": rng.choice((4, 4, 6)),
                 "g": rng.choice((32, 64, 64))}
        elif kind == "direct":
            H, W = _image(rng, 6, 64)
            g = rng.choice((32, 64, 64, 128))
            c = {"kind": "direct", "N": _log(rng, 1, 16), "H": H, "W": W, "Cin": _channels(rng, 64, 1280, g),
                 "Cout": _outputs(rng, 32, 1280), "g": g, "bits": rng.choice((8, 8, 4))}
        elif kind == "linear":
            g = rng.choice((32, 64, 64, 128, 256))
            c = {"kind": "linear", "rows": _log(rng, 1, 8192), "Cin": _channels(rng, 320, 5120, g),
                 "Cout": _outputs(rng, 320, 5120), "g": g, "bits": rng.choice((8, 4))}
        else:
            g = rng.choice((32, 64, 64, 128, 256))
            c = {"kind": "weights", "Cin": _channels(rng, 64, 1280, g), "Cout": _outputs(rng, 64, 1280),
                 "m": rng.choice((4, 4, 6, 6, 2)), "g": g, "scaled": rng.random() < 0.25}
        w = work(c)
        if w["bytes"] <= 300e6 and w["flops"] <= (250e9 if c["kind"] == "stack" else 120e9):
            return c


# ---- what a case needs ----

def _levels(c):   # the resolutions of a stack: halved edge, doubled channels
    return [(max(1, c["size"] >> k), c["base"] << k) for k in range(3)]


def _conv_work(N, H, W, Cin, Cout, m, g):
    n2, groups = (m + 2) ** 2, Cin // g
    tiles = N * H * W / m ** 2
    return (4 * N * H * W * (Cin + Cout) + n2 * Cout * (Cin + 4 * groups) + 4 * Cout, 2 * n2 * tiles * Cin * Cout)


def work(case):
    """Inputs and prepared weights read once, outputs written once; the multiply-adds of the
    Winograd-domain (or plain) integer products."""
    c = case
    if c["kind"] == "conv":
        b, f = _conv_work(c["N"], c["H"], c["W"], c["Cin"], c["Cout"], c["m"], c["g"])
    elif c["kind"] == "stack":
        b = f = 0
        for s, ch in _levels(c):
            lb, lf = _conv_work(c["N"], s, s, ch, ch, c["m"], c["g"])
            b, f = b + c["depth"] * lb, f + c["depth"] * lf
    elif c["kind"] == "weights":
        n2 = (c["m"] + 2) ** 2
        b = 36 * c["Cin"] * c["Cout"] + n2 * c["Cout"] * (c["Cin"] + 4 * (c["Cin"] // c["g"])) + 8 * c["Cout"]
        f = 2 * c["Cin"] * c["Cout"] * 3 * (c["m"] + 2) * (c["m"] + 5)
    else:
        taps = 9 if c["kind"] == "direct" else 1
        P = c["N"] * c["H"] * c["W"] if taps == 9 else c["rows"]
        b = 4 * P * (c["Cin"] + c["Cout"]) + 4 * c["Cout"] + \
            taps * c["Cout"] * (c["Cin"] * c["bits"] // 8 + 4 * (c["Cin"] // c["g"]))
        f = 2 * taps * P * c["Cin"] * c["Cout"]
    return {"bytes": float(b), "flops": float(f)}


def tolerance(case):
    """Single layers: codes, scales and integer sums are exact and only the order of the fp32 sums
    behind them is free; F(6,3)'s output transform cancels (sum of magnitudes over result: about
    100).  Chained layers and the integer output transform quantize such fp32 sums again: a
    rounding difference moves a few values by one code of 127, and with F(6,3) and F(4,3) an
    output code counts up to 32 x 32 (8 x 8) in the integer output transform."""
    if case["kind"] == "weights":
        return "exact"
    if case["kind"] == "stack":
        return {"rel": 1e-2, "max": 0.5}
    if case.get("integer"):
        return {"rel": 5e-3, "max": 0.9}
    return {"rel": 3e-5 if case.get("m") == 6 else 1e-5}


# ---- inputs ----

def _activations(gen, shape, acts):
    """NHWC activations (channels last): half-normal after a ReLU; normal with two loud channels;
    heavy-tailed UNet latents, Student-t with 3 degrees of freedom and 1 % loud channels."""
    x = torch.randn(shape, generator=gen, device="cuda")
    ch = shape[-1]
    if acts == "relu":
        return x.abs_()
    loud, by = (2, 20.0) if acts == "normal" else (max(1, round(0.01 * ch)), 30.0)
    if acts == "latent":
        chi2 = torch.zeros(shape, device="cuda")
        for _ in range(3):
            chi2 += torch.randn(shape, generator=gen, device="cuda").square_()
        x = x.mul_(2.0).div_(chi2.div_(3.0).sqrt_())
    gain = torch.ones(ch, device="cuda")
    gain[torch.randperm(ch, generator=gen, device="cuda")[:loud]] = by
    return x.mul_(gain).contiguous()


def _weights(gen, shape, std):
    return torch.randn(shape, generator=gen, device="cuda").mul_(std)


def _plan(c, N, H, W, Cin, Cout, seed):
    mats = {}
    if c.get("scaled"):   # learned per-row scales of the transform matrices
        rng = np.random.default_rng(seed)
        n = c["m"] + 2
        mats = dict(zip(("AT", "BT", "G"), wq.scaled_transforms(c["m"], rng.uniform(0.5, 2.0, n), rng.uniform(0.5, 2.0, n))))
    plan = wq.Plan(N, H, W, Cin, Cout, c["m"], c["g"], **mats)
    return plan.set_integer_transforms(c["integer"]) if c.get("integer") else plan


def _weight_std(acts, fan_in):
    return 0.02 if acts == "latent" else math.sqrt(2.0 / fan_in)


def prepare(case, seed):
    c = case
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    if c["kind"] == "weights":
        plan = _plan(c, 1, 16, 16, c["Cin"], c["Cout"], seed)
        return {"kind": "weights", "plan": plan, "w": _weights(gen, (c["Cout"], c["Cin"], 3, 3), 0.02),
                "bias": _weights(gen, (c["Cout"],), 0.1),
                "blob": torch.zeros(plan.layout.blob_bytes, dtype=torch.uint8, device="cuda")}
    if c["kind"] == "stack":
        calls, ends, need = [], [], 0
        for s, ch in _levels(c):
            plan = _plan(c, c["N"], s, s, ch, ch, seed)
            need = max(need, plan.layout.ws_bytes)
            x = _activations(gen, (c["N"], s, s, ch), "latent")
            for _ in range(c["depth"]):
                blob, y = plan.alloc_blob(), plan.alloc_output()
                plan.weight_prepare(_weights(gen, (ch, ch, 3, 3), 0.02), _weights(gen, (ch,), 0.1), blob)
                calls.append((plan, x, blob, y))
                x = y
            ends.append(x)
        # one workspace for all layers: they run one after the other
        ws = torch.empty(need, dtype=torch.uint8, device="cuda")
        calls = [(plan, x, blob, ws[:plan.layout.ws_bytes], y) for plan, x, blob, y in calls]
        return {"kind": "stack", "calls": calls, "ends": ends}
    if c["kind"] == "conv":
        plan = _plan(c, c["N"], c["H"], c["W"], c["Cin"], c["Cout"], seed)
        x = _activations(gen, (c["N"], c["H"], c["W"], c["Cin"]), c["acts"])
        w = _weights(gen, (c["Cout"], c["Cin"], 3, 3), _weight_std(c["acts"], 9 * c["Cin"]))
    elif c["kind"] == "direct":
        plan = wq.DirectPlan(c["N"], c["H"], c["W"], c["Cin"], c["Cout"], c["g"], weight_bits=c["bits"])
        x = _activations(gen, (c["N"], c["H"], c["W"], c["Cin"]), "latent")
        w = _weights(gen, (c["Cout"], c["Cin"], 3, 3), 0.02)
    else:
        plan = wq.DirectPlan(c["rows"], 1, 1, c["Cin"], c["Cout"], c["g"], linear=True, weight_bits=c["bits"])
        x = _activations(gen, (c["rows"], c["Cin"]), "latent")
        w = _weights(gen, (c["Cout"], c["Cin"]), 0.02)
    blob = plan.alloc_blob()
    plan.weight_prepare(w, _weights(gen, (c["Cout"],), 0.1), blob)
    return {"kind": c["kind"], "plan": plan, "x": x, "blob": blob, "ws": plan.alloc_workspace(),
            "y": plan.alloc_output()}


def run(state):
    s = state
    if s["kind"] == "weights":
        s["plan"].weight_prepare(s["w"], s["bias"], s["blob"])
        return s["blob"]
    if s["kind"] == "stack":
        for plan, x, blob, ws, y in s["calls"]:
            plan.forward(x, blob, ws, y)
        return s["ends"]
    s["plan"].forward(s["x"], s["blob"], s["ws"], s["y"])
    return s["y"]
