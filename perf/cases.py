"""Workloads whose time is watched, each one a pass through the package's public calls.

A case is one quantised 3x3 layer (or the VGG-16-shaped stack of them) with its sizes, layout and arithmetic mode.
Filters are transformed once in ``prepare`` (Section 4.3 of the paper: off the inference path) and reused by every
pass, as a serving program does; layer calls return fresh outputs, the stack writes into buffers it keeps.

``op`` names the call:
  conv        winograd_conv2d_int8: int8 in, int32 out, complex F(4x4,3x3)
  requant     winograd_conv2d_int8_requant: int8 out (shift, ReLU, optional 2x2 max-pool), what a network runs per layer
  u8          winograd_conv2d_u8: uint8 with zero points (the affine tensors of Section 4.1)
  act_scaled  winograd_conv2d_int8_act_scaled: filters and activations scaled
  f2x2        f2x2_conv2d_int8: rational F(2x2,3x3), the variant the paper's own evaluation used
  f2x2_requant  f2x2_conv2d_int8_requant
  direct      direct_conv2d_int8 followed by requant_relu_pool_int8: the same layer without Winograd
  stack       13 requant layers of the VGG-16-shaped network, each feeding the next
"""
import math

import torch

import paper_1901_01965_amd as wg
from paper_1901_01965_amd import workloads as wl

# A drawn layer has at most this many direct operations (2*9*N*K*C*H*W): those of the largest listed single layers.
LARGEST_LAYER_OPS = 59.5e9


def _layer(name, op, N, C, K, H, W, mode="lossless", layout="nhwc", pool=False, zero_point=128):
    case = {"op": op, "N": N, "C": C, "K": K, "H": H, "W": W, "mode": mode, "layout": layout}
    if name:
        case["name"] = name
    if op in ("requant", "f2x2_requant", "direct"):
        case.update(pool=pool, shift=_shift(C))
    if op == "u8":
        case["zero_point"] = zero_point
    return case


def _shift(C):
    """Power-of-two requantisation that brings outputs of the synthetic distributions to about 7 bits."""
    return max(4, round(math.log2(math.sqrt(9 * C) * 26)))


def listed():
    return [
        # the smallest layer of the test configurations, with the default layout: a call's fixed cost
        _layer("small", "conv", 1, 16, 16, 16, 16, layout="nchw"),
        # the ResNet-style layer that the benchmark quotes
        _layer("resnet56", "conv", 8, 64, 64, 56, 56),
        # the same layer at a throughput batch
        _layer("resnet56_batch", "conv", 256, 64, 64, 56, 56),
        # mid-network layer, filters scaled into int8
        _layer("mid28_scaled", "conv", 32, 128, 128, 28, 28, mode="scaled"),
        # deepest layer: few pixels, 7x7 leaves partial tiles, filters dominate the bytes
        _layer("deep7_scaled", "conv", 64, 512, 512, 7, 7, mode="scaled"),
        # PyTorch's default layout with nothing divisible: odd image, odd channels on both sides
        _layer("ragged_nchw", "conv", 4, 100, 75, 37, 53, layout="nchw"),
        # a whole network at the benchmark's batch, int8 from layer to layer
        {"name": "vgg16_scaled", "op": "stack", "N": wl.VGG16_BATCH, "mode": "scaled"},
        # one image through the same network: thirteen dependent launches, exact mode
        {"name": "vgg16_one_image", "op": "stack", "N": 1, "mode": "lossless"},
        # affine-quantised uint8 tensors, as frameworks export them
        _layer("affine_u8", "u8", 32, 128, 128, 28, 28, mode="scaled"),
        # both operands scaled
        _layer("both_scaled", "act_scaled", 64, 256, 256, 14, 14, mode="scaled"),
        # the paper's evaluated variant
        _layer("f2x2_scaled", "f2x2", 32, 128, 128, 28, 28, mode="scaled"),
        # direct convolution and requantisation of a VGG layer: what the Winograd layers are compared against
        _layer("direct_pool", "direct", 16, 256, 256, 56, 56, pool=True),
    ]


def draw(rng):
    op = rng.choice(("conv", "conv", "conv", "requant", "requant", "u8", "act_scaled", "f2x2", "f2x2_requant", "direct", "stack"))
    mode = "scaled" if op == "act_scaled" else rng.choice(("lossless", "scaled"))
    if op == "stack":
        return {"op": op, "N": _log_int(rng, 1, wl.VGG16_BATCH), "mode": mode}
    while True:
        # most networks keep channels divisible by 16; a quarter of the draws has any number
        C, K = (_channels(rng, 229 if op == "u8" else 512) for _ in range(2))
        H = _log_int(rng, 7, 112)
        W = H if rng.random() < 0.5 else _log_int(rng, 7, 112)
        N = _log_int(rng, 1, 256)
        ops = 2 * 9 * N * C * K * H * W
        if 16 * 16 * 16 * 16 * 18 <= ops <= LARGEST_LAYER_OPS:
            break
    pool = op in ("requant", "f2x2_requant", "direct") and H % 2 == 0 and W % 2 == 0 and rng.random() < 0.5
    return _layer(None, op, N, C, K, H, W, mode, rng.choice(("nhwc", "nhwc", "nchw")), pool, rng.randrange(256))


def _log_int(rng, low, high):
    return min(high, int(math.exp(rng.uniform(math.log(low), math.log(high + 1)))))


def _channels(rng, most):
    c = _log_int(rng, 16, most)
    return c if rng.random() < 0.25 else c // 16 * 16


# ---- inputs: the distributions of workloads.py, made on the GPU -------------------------------------------------

def _relu_like(shape, gen):
    """int8, half zeros, else uniform in [0, 127]."""
    x = torch.randint(0, 256, shape, dtype=torch.int16, device="cuda", generator=gen)
    return torch.where(x < 128, x, torch.zeros_like(x)).to(torch.int8)


def _filters(shape, gen):
    """int8, round(N(0, 32)) within +-127."""
    return (torch.randn(shape, device="cuda", generator=gen) * 32).round_().clamp_(-127, 127).to(torch.int8)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    mode = wg.LOSSLESS if case["mode"] == "lossless" else wg.SCALED
    op, N = case["op"], case["N"]
    if op == "stack":
        x = _relu_like((N, 224, 224, 3), gen)
        packed = [wg.winograd_filter_transform(_filters((k, 3, 3, c), gen), wg.NHWC, mode) for c, k, _, _ in wl.VGG16_LAYERS]
        acts = [torch.empty((N, hw // (1 + pool), hw // (1 + pool), k), dtype=torch.int8, device="cuda")
                for _, k, hw, pool in wl.VGG16_LAYERS]
        return {"op": op, "x": x, "packed": packed, "acts": acts}
    nhwc = case["layout"] == "nhwc"
    C, K, H, W = case["C"], case["K"], case["H"], case["W"]
    layout = wg.NHWC if nhwc else wg.NCHW
    x = _relu_like((N, H, W, C) if nhwc else (N, C, H, W), gen)
    w = _filters((K, 3, 3, C) if nhwc else (K, C, 3, 3), gen)
    state = {"op": op, "layout": layout, "case": dict(case)}
    if op == "u8":
        # affine activations: bytes spread over the range, half of them at the zero point (exact zeros)
        zx = case["zero_point"]
        b = torch.randint(0, 256, x.shape, dtype=torch.int16, device="cuda", generator=gen)
        x = torch.where(x == 0, torch.full_like(b, zx), b).to(torch.uint8)
        state.update(x=x, packed=wg.winograd_filter_transform_u8((w.to(torch.int16) + 128).to(torch.uint8), 128, layout, mode))
    elif op == "direct":
        state.update(x=x, w=w)
    elif op in ("f2x2", "f2x2_requant"):
        state.update(x=x, packed=wg.f2x2_filter_transform(w, layout, mode))
    else:
        state.update(x=x, packed=wg.winograd_filter_transform(w, layout, mode))
    return state


def run(state):
    op = state["op"]
    if op == "stack":
        x = state["x"]
        for packed, shift, (_, _, _, pool), out in zip(state["packed"], wl.VGG16_SHIFTS, wl.VGG16_LAYERS, state["acts"]):
            x = wg.winograd_conv2d_int8_requant(x, packed, shift, True, pool, wg.NHWC, out=out)
        return state["acts"]
    case, x, layout = state["case"], state["x"], state["layout"]
    if op == "conv":
        return wg.winograd_conv2d_int8(x, state["packed"], layout)
    if op == "requant":
        return wg.winograd_conv2d_int8_requant(x, state["packed"], case["shift"], True, case["pool"], layout)
    if op == "u8":
        return wg.winograd_conv2d_u8(x, case["zero_point"], state["packed"], layout)
    if op == "act_scaled":
        return wg.winograd_conv2d_int8_act_scaled(x, state["packed"], layout)
    if op == "f2x2":
        return wg.f2x2_conv2d_int8(x, state["packed"], layout)
    if op == "f2x2_requant":
        return wg.f2x2_conv2d_int8_requant(x, state["packed"], case["shift"], True, case["pool"], layout)
    y = wg.direct_conv2d_int8(x, state["w"], layout)
    return wg.requant_relu_pool_int8(y, case["shift"], True, case["pool"], layout)


# int8 multiply-adds per tile and channel pair: 46 twelve-bit products as int8 limbs (138 exact, 112 with int8 filters,
# 56 with both sides int8); F(2x2,3x3): 16 products
_PRODUCTS = {"lossless": 138, "scaled": 112}
_F2_PRODUCTS = {"lossless": 64, "scaled": 32}
# Winograd-domain filter bytes per channel pair: 36 numbers of 12 bits or of 8; F(2x2,3x3): 16
_FILTER_BYTES = {"lossless": 72, "scaled": 36}
_F2_FILTER_BYTES = {"lossless": 32, "scaled": 16}


def _layer_work(op, N, C, K, H, W, mode, pool):
    pixels = N * H * W
    if op == "direct":
        filter_bytes, ops = 9 * K * C, 2 * 9 * pixels * K * C
    elif op in ("f2x2", "f2x2_requant"):
        tiles = N * ((H + 1) // 2) * ((W + 1) // 2)
        filter_bytes, ops = _F2_FILTER_BYTES[mode] * K * C, 2 * _F2_PRODUCTS[mode] * tiles * K * C
    else:
        tiles = N * ((H + 3) // 4) * ((W + 3) // 4)
        per_pair = 56 if op == "act_scaled" else _PRODUCTS[mode]
        filter_bytes, ops = _FILTER_BYTES[mode] * K * C, 2 * per_pair * tiles * K * C
    if op in ("requant", "f2x2_requant", "direct"):
        out = pixels * K // (4 if pool else 1)
        if op == "direct":
            out += 2 * 4 * pixels * K     # the int32 outputs, written by one call and read by the other
    else:
        out = 4 * pixels * K
    return {"bytes": pixels * C + filter_bytes + out, "flops": ops}


def work(case):
    if case["op"] != "stack":
        return _layer_work(case["op"], case["N"], case["C"], case["K"], case["H"], case["W"], case["mode"], case.get("pool", False))
    layers = [_layer_work("requant", case["N"], c, k, hw, hw, case["mode"], pool) for c, k, hw, pool in wl.VGG16_LAYERS]
    return {key: sum(l[key] for l in layers) for key in ("bytes", "flops")}


def tolerance(case):
    """Integer arithmetic throughout: every mode is an exact function of its inputs."""
    return "exact"
