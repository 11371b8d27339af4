"""The workloads by which this library's speed is judged.

A program that uses the library does one of four things with it: it runs a 3x3
convolution layer (``Plan.conv2d``), a 1D convolution (``Plan.conv1d``), a whole
stack of layers (``VggStack.forward``), or, in an error study or a search for a
plan, the float64 direct convolution that results are held against
(``layer_ops.direct_conv_f64``).  ``listed`` names one case for each real use;
``draw`` gives more of the same ranges.  The library has no backward pass.
"""
import math

import numpy as np
import torch

TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}

# modulus set -> (output tile m, domain points alpha' per dimension)
F2 = "0,1,-1,inf"
F4 = "0,1,-1,1/2,-1/2,inf"
F4Q = "0,1,-1,a^2+1,inf"
F6 = "0,-1,1,-1/2,2,1/2,-2,inf"
F6Q = "0,-1,1,-1/2,2,a^2+1,inf"
F6QQ = "0,-1,1,a^2+1,a^2-2,inf"
F8Q = "0,-1,1,-1/2,2,1/2,-2,a^2+1,inf"
F10Q = "0,-1,1,-1/2,2,1/2,-2,-1/4,4,a^2+1,inf"
SETS = {F2: (2, 4), F4: (4, 6), F4Q: (4, 7), F6: (6, 8), F6Q: (6, 9), F6QQ: (6, 10), F8Q: (8, 11), F10Q: (10, 13)}

# VGG-16's thirteen 3x3 convolutions: H = W, C, K, max-pool after the layer
VGG = ((224, 3, 64, False), (224, 64, 64, True), (112, 64, 128, False), (112, 128, 128, True),
       (56, 128, 256, False), (56, 256, 256, False), (56, 256, 256, True),
       (28, 256, 512, False), (28, 512, 512, False), (28, 512, 512, True),
       (14, 512, 512, False), (14, 512, 512, False), (14, 512, 512, True))


def _conv(name, moduli, dtype, N, H, W, C, K):
    return {"name": name, "kind": "conv2d", "moduli": moduli, "dtype": dtype, "N": N, "H": H, "W": W, "C": C, "K": K}


def listed():
    return [
        # the smallest layer the test suite and the bench configurations run: launches and host work
        _conv("tiny_f32", F2, "f32", 1, 16, 16, 8, 8),
        # one image through a deep, narrow layer: serving without a batch
        _conv("one_image_bf16", F4Q, "bf16", 1, 14, 14, 512, 512),
        # the fp32 mid-size layer of the bench configurations
        _conv("mid_f32", F4, "f32", 8, 56, 56, 128, 128),
        # the bf16 layer of the bench configurations with two degree-2 moduli and 6x6 output tiles
        _conv("f6_two_quad_bf16", F6QQ, "bf16", 16, 28, 28, 256, 256),
        # three layers of the VGG-16 stack at its batch: RGB input, widest mid layer, deep layer
        _conv("vgg_rgb_bf16", F4Q, "bf16", 32, 224, 224, 3, 64),
        _conv("vgg_56_bf16", F4Q, "bf16", 32, 56, 56, 256, 256),
        _conv("vgg_28_bf16", F4Q, "bf16", 32, 28, 28, 512, 512),
        # sizes that fill no tile, block or vector: a detection-style feature map in fp16
        _conv("ragged_f16", F4Q, "f16", 6, 75, 91, 72, 120),
        # 8x8 output tiles with one degree-2 modulus (the ratio 1.89 of the paper's Table 3), run-time coefficients
        _conv("wide_m8_bf16", F8Q, "bf16", 16, 56, 56, 256, 256),
        # the 1D form on sequences
        {"name": "conv1d_f16", "kind": "conv1d", "moduli": F4Q, "dtype": "f16", "N": 16, "L": 4096, "C": 128, "K": 128},
        # the reference of an error study or a plan search: a few images of a layer's input
        {"name": "reference_f64", "kind": "direct_f64", "dtype": "bf16", "N": 2, "H": 56, "W": 56, "C": 128, "K": 128},
        # the whole stack with ReLU and pooling; its result is the last pooled activations, as a classifier's head reads them
        {"name": "vgg_stack_bf16", "kind": "stack", "moduli": F4Q, "dtype": "bf16", "N": 32},
    ]


def _direct_flops(case):
    k = case["kind"]
    if k == "stack":
        return sum(18.0 * case["N"] * hw * hw * C * K for hw, C, K, _ in VGG)
    if k == "conv1d":
        return 6.0 * case["N"] * case["L"] * case["C"] * case["K"]
    return 18.0 * case["N"] * case["H"] * case["W"] * case["C"] * case["K"]


def draw(rng):
    def log(lo, hi):
        return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))

    while True:
        kind = rng.choices(("conv2d", "conv1d", "direct_f64", "stack"), (14, 3, 2, 1))[0]
        if kind == "stack":
            return {"kind": kind, "moduli": rng.choice((F4, F4Q)), "dtype": rng.choice(("f16", "bf16")),
                    "N": log(1, 32)}
        # channels: powers of two as networks have them, or any number
        ch = [2 ** rng.randint(3, 9) if rng.random() < 0.5 else log(1, 512) for _ in range(2)]
        dtype = rng.choice(("f32", "f16", "bf16"))
        if kind == "conv1d":
            case = {"kind": kind, "moduli": rng.choice((F2, F4, F4Q, F6QQ)), "dtype": dtype,
                    "N": log(1, 64), "L": log(16, 16384), "C": ch[0], "K": ch[1]}
            limit = 4e10
        elif kind == "direct_f64":
            case = {"kind": kind, "dtype": dtype, "N": log(1, 4), "H": log(4, 112), "W": log(4, 112),
                    "C": ch[0], "K": ch[1]}
            limit = 4e9
        else:
            sets = tuple(_TOL[dtype])
            case = {"kind": kind, "moduli": rng.choice(sets), "dtype": dtype, "N": log(1, 32),
                    "H": log(7, 224), "W": log(7, 224), "C": ch[0], "K": ch[1]}
            limit = 1.5e11
        if 1e5 <= _direct_flops(case) <= limit:
            return case


def _inputs(case, seed):
    """The layer input (post-ReLU activations: half-normal) and He-scaled weights, rounded to the dtype, on the GPU."""
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * seed + 17)
    C, K = case["C"], case["K"]
    if case["kind"] == "conv1d":
        xs, ws, fan = (case["N"], case["L"], C), (K, 3, C), 3.0 * C
    else:
        xs, ws, fan = (case["N"], case["H"], case["W"], C), (K, 3, 3, C), 9.0 * C
    x = torch.randn(xs, generator=g, device="cuda").abs_()
    w = torch.randn(ws, generator=g, device="cuda").mul_(math.sqrt(2.0 / fan))
    return x.to(TORCH[case["dtype"]]), w.to(TORCH[case["dtype"]])


def _stack_input(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * seed + 29)
    return torch.randn((case["N"], 224, 224, 3), generator=g, device="cuda").abs_().to(TORCH[case["dtype"]])


def prepare(case, seed):
    if case["kind"] == "stack":
        from paper_1905_05233_amd.vgg import VggStack
        from paper_1905_05233_amd.workloads import PlanSpec
        spec = PlanSpec(case["moduli"], SETS[case["moduli"]][0])
        return {"case": case, "stack": VggStack(dtype=case["dtype"], plans=[spec] * len(VGG)),
                "x": _stack_input(case, seed)}
    x, w = _inputs(case, seed)
    state = {"case": case, "x": x, "w": w}
    if case["kind"] != "direct_f64":
        from paper_1905_05233_amd.winograd import Plan
        state["plan"] = Plan(case["moduli"], m=SETS[case["moduli"]][0], dtype=case["dtype"])
    return state


def run(state):
    kind = state["case"]["kind"]
    if kind == "stack":
        return state["stack"].forward(state["x"])
    if kind == "conv1d":
        return state["plan"].conv1d(state["x"], state["w"])
    if kind == "direct_f64":
        from paper_1905_05233_amd.layer_ops import direct_conv_f64
        return direct_conv_f64(state["x"], state["w"])
    return state["plan"].conv2d(state["x"], state["w"])


def _layer_work(N, H, W, C, K, m, alpha, es):
    tiles = N * math.ceil(H / m) * math.ceil(W / m)
    return es * (N * H * W * (C + K) + 9 * C * K), 2.0 * alpha * alpha * tiles * C * K


def work(case):
    """Input, weights and output once; the multiply-adds of the channel contraction (the transforms are additions to it)."""
    es = 4 if case["dtype"] == "f32" else 2
    kind = case["kind"]
    if kind == "direct_f64":
        px = case["N"] * case["H"] * case["W"]
        return {"bytes": es * (px * case["C"] + 9 * case["C"] * case["K"]) + 8 * px * case["K"],
                "flops": _direct_flops(case)}
    m, alpha = SETS[case["moduli"]]
    if kind == "conv1d":
        N, L, C, K = case["N"], case["L"], case["C"], case["K"]
        return {"bytes": es * (N * L * (C + K) + 3 * C * K), "flops": 2.0 * alpha * N * math.ceil(L / m) * C * K}
    if kind == "stack":
        # each layer's input and output cross memory once; ReLU and pooling ride along
        rows = [_layer_work(case["N"], hw, hw, C, K, m, alpha, es) for hw, C, K, _ in VGG]
        return {"bytes": sum(r[0] for r in rows), "flops": sum(r[1] for r in rows)}
    b, f = _layer_work(case["N"], case["H"], case["W"], case["C"], case["K"], m, alpha, es)
    return {"bytes": b, "flops": f}


# Largest relative error that another correct implementation at the same
# precision shows: four times the error against float64 measured at C = 96
# (fp32: with room for longer sums).  In 16 bits U, V and y are rounded to the
# dtype, and the transforms multiply those roundings by an amount that belongs
# to the modulus set.  The 10x10 tiles leave fp16 and bf16 no correct digits, so
# they are run in fp32 alone.
_TOL = {"f32": {F2: 2e-6, F4: 8e-6, F4Q: 2e-6, F6: 1.5e-5, F6Q: 4e-6, F6QQ: 6e-6, F8Q: 6e-6, F10Q: 8e-5},
        "f16": {F2: 1.7e-3, F4: 7.5e-3, F4Q: 1.8e-3, F6: 1.4e-2, F6Q: 3e-3, F6QQ: 6e-3, F8Q: 6.6e-3},
        "bf16": {F2: 1.4e-2, F4: 6e-2, F4Q: 1.5e-2, F6: 1.1e-1, F6Q: 2.5e-2, F6QQ: 4.8e-2, F8Q: 5e-2}}


def tolerance(case):
    if case["kind"] == "direct_f64":
        return {"rel": 1e-14}
    # through thirteen layers the error against float64 grows by 2.5 (measured)
    return {"rel": _TOL[case["dtype"]][case["moduli"]] * (2.5 if case["kind"] == "stack" else 1.0)}


def _direct(x, w):
    """float64 convolution, NHWC, pad 1, by one matrix product a tap."""
    N, H, W, C = x.shape
    K = w.shape[0]
    xp = torch.zeros((N, H + 2, W + 2, C), dtype=torch.float64, device=x.device)
    xp[:, 1:-1, 1:-1] = x
    y = torch.zeros((N * H * W, K), dtype=torch.float64, device=x.device)
    for i in range(3):
        for j in range(3):
            y += xp[:, i:i + H, j:j + W].reshape(-1, C) @ w[:, i, j].double().t().contiguous()
    return y.view(N, H, W, K)


def exact(case, seed):
    if case["kind"] == "stack":
        x = _stack_input(case, seed).double()
        for i, (_, C, K, pool) in enumerate(VGG):
            rng = np.random.Generator(np.random.PCG64(1 + i))   # the weights a VggStack holds
            w = torch.from_numpy((rng.standard_normal(size=(K, 3, 3, C)) * np.sqrt(2.0 / (9.0 * C))).astype(np.float32))
            w = w.cuda().to(TORCH[case["dtype"]])
            # a few images at a time: float64 activations are large
            x = torch.cat([_direct(c, w).clamp_(min=0.0) for c in x.split(8)])
            if pool:
                N, H, W, _ = x.shape
                x = x.view(N, H // 2, 2, W // 2, 2, K).amax(dim=(2, 4))
        return x
    x, w = _inputs(case, seed)
    if case["kind"] == "conv1d":
        N, L, C = x.shape
        xp = torch.zeros((N, L + 2, C), dtype=torch.float64, device=x.device)
        xp[:, 1:-1] = x
        y = sum(xp[:, j:j + L].reshape(-1, C) @ w[:, j].double().t().contiguous() for j in range(3))
        return y.view(N, L, -1)
    return _direct(x, w)
