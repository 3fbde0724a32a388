"""The calls whose time matters to users of this library, as a list and as a way to draw more of them.

A case is one call of `cacnn_conv_forward` or `cacnn_pool_forward`: the layers of a convolutional network from its
first (three channels, large filter, stride) to its last (many channels, few positions), for a single image up to a
large batch, in both data types, with sizes that are powers of two and sizes that are nothing of the kind.
`listed()` names twelve, `draw()` gives further ones of the same ranges.
"""
import math

import torch

import paper_1802_06905_amd as cc

_DIMS = ("B", "C", "K", "W", "H", "R", "S", "sw", "sh")

# a drawn case costs at most what the largest listed one does
_MAX_FLOPS = {"f32": 7.6e9, "bf16": 59.2e9}
_MAX_BYTES = 250e6


def _case(op, dtype, dims, name=None):
    case = {"op": op, "dtype": dtype}
    case.update(zip(_DIMS, dims))
    if name is not None:
        case["name"] = name
    return case


def listed():
    return [
        # a single small image through a first layer: a call is latency and nothing else
        _case("conv", "f32", (1, 3, 8, 16, 16, 3, 3, 1, 1), "f32_b1_first_layer"),
        # full-precision inference, early layer, small batch
        _case("conv", "f32", (8, 64, 64, 56, 56, 3, 3, 1, 1), "f32_b8_3x3"),
        # the 7 x 7 stride-2 stem of an image classifier
        _case("conv", "f32", (32, 3, 64, 112, 112, 7, 7, 2, 2), "f32_b32_stem"),
        # nothing divides anything: odd batch, channels, extents and filter
        _case("conv", "f32", (5, 30, 50, 27, 19, 5, 5, 1, 1), "f32_b5_5x5_ragged"),
        # middle and late layers of a training batch
        _case("conv", "bf16", (64, 256, 256, 14, 14, 3, 3, 1, 1), "bf16_b64_3x3"),
        _case("conv", "bf16", (256, 512, 512, 7, 7, 3, 3, 1, 1), "bf16_b256_3x3"),
        # serving one image at a time
        _case("conv", "bf16", (1, 128, 128, 28, 28, 3, 3, 1, 1), "bf16_b1_3x3"),
        # the expanding 1 x 1 layer of a bottleneck block: many outputs for little arithmetic
        _case("conv", "bf16", (64, 64, 256, 56, 56, 1, 1, 1, 1), "bf16_b64_1x1"),
        # a downsampling layer
        _case("conv", "bf16", (32, 128, 256, 28, 28, 3, 3, 2, 2), "bf16_b32_3x3_s2"),
        # the stem in bf16
        _case("conv", "bf16", (16, 3, 64, 112, 112, 7, 7, 2, 2), "bf16_b16_stem"),
        # the pooling behind the stem, and an average over windows at a batch that 16-byte loads do not divide
        _case("pool_max", "f32", (32, 64, 64, 56, 56, 3, 3, 2, 2), "pool_max_f32"),
        _case("pool_avg", "bf16", (20, 192, 192, 27, 27, 3, 3, 2, 2), "pool_avg_bf16_b20"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))))


def _channels(rng, lo, hi):
    """Half of the layers have a multiple of 16 channels, the others any number."""
    n = _log_int(rng, lo, hi)
    return max(16, (n + 8) // 16 * 16) if rng.random() < 0.5 else n


def draw(rng):
    while True:
        dtype = rng.choice(("f32", "bf16", "bf16"))
        op = rng.choice(("conv", "conv", "conv", "conv", rng.choice(("pool_max", "pool_avg"))))
        B = 2 ** rng.randint(0, 8) if rng.random() < 0.5 else _log_int(rng, 1, 256)
        W = _log_int(rng, 1, 112)
        H = W if rng.random() < 0.5 else _log_int(rng, 1, 112)
        if op == "conv":
            if rng.random() < 0.15:     # a stem: three channels, or the one of a grey image
                C, K = rng.choice((3, 3, 1)), _channels(rng, 16, 96)
                W = _log_int(rng, 14, 112)
                H = W if rng.random() < 0.5 else _log_int(rng, 14, 112)
                R, s = rng.choice(((7, 2), (11, 4), (3, 1), (3, 2)))
                S, sw, sh = R, s, s
            else:
                C, K = _channels(rng, 8, 1024), _channels(rng, 8, 1024)
                R, S = rng.choice(((1, 1),) * 4 + ((3, 3),) * 6 + ((5, 5), (1, 7), (7, 1)))
                sw = sh = rng.choice((1, 1, 1, 2))
        else:
            C = K = _channels(rng, 16, 1024)
            R, s = rng.choice(((2, 2), (3, 2), (3, 1), (7, 7)))
            S, sw, sh = R, s, s
            # pooling calls are refused beyond this (their kernel's index arithmetic is 32 bits wide)
            if H * (W + 8) * C * B * max(B, C, H, 64) >= 2 ** 32:
                continue
        case = _case(op, dtype, (B, C, K, W, H, R, S, sw, sh))
        w = work(case)
        if w["bytes"] <= _MAX_BYTES and w["flops"] <= _MAX_FLOPS[dtype] and w["bytes"] >= 1e4:
            return case


def _dims(case):
    return tuple(int(case[n]) for n in _DIMS)


def _inputs(case, seed):
    B, C, K, W, H, R, S, sw, sh = _dims(case)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    typ = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    image = torch.randn((sw * (W - 1) + R, sh * (H - 1) + S, C, B), generator=gen, device="cuda", dtype=torch.float32)
    if case["op"] != "conv":
        return image.to(typ), None
    filt = torch.randn((K, R, S, C), generator=gen, device="cuda", dtype=torch.float32) / math.sqrt(C * R * S)
    return image.to(typ), filt.to(typ)


def prepare(case, seed):
    B, C, K, W, H, R, S, sw, sh = _dims(case)
    image, filt = _inputs(case, seed)
    return {
        "op": case["op"],
        "problem": cc.Problem(B, C, K, W, H, R, S, sw, sh),
        "dtype": cc.CACNN_F32 if case["dtype"] == "f32" else cc.CACNN_BF16_F32ACC,
        "image": image,
        "filter": filt,
        "out": torch.empty((K, H, W, B), device="cuda", dtype=torch.float32),
    }


def run(state):
    if state["op"] == "conv":
        cc.cacnn_conv_forward(state["problem"], state["dtype"], state["image"], state["filter"], state["out"])
    else:
        mode = cc.CACNN_POOL_MAX if state["op"] == "pool_max" else cc.CACNN_POOL_AVG
        cc.cacnn_pool_forward(state["problem"], state["dtype"], mode, state["image"], state["out"])
    return state["out"]


def work(case):
    """Image elements that some output reads, Filter and Out once each."""
    B, C, K, W, H, R, S, sw, sh = _dims(case)
    esz = 4 if case["dtype"] == "f32" else 2
    cols = min(sw * (W - 1) + R, W * R)
    rows = min(sh * (H - 1) + S, H * S)
    bytes_ = esz * cols * rows * C * B + 4 * K * H * W * B
    if case["op"] != "conv":
        return {"bytes": bytes_, "flops": B * C * W * H * R * S}
    return {"bytes": bytes_ + esz * K * R * S * C, "flops": 2 * B * C * K * W * H * R * S}


def tolerance(case):
    if case["op"] == "pool_max":
        return "exact"
    if case["op"] == "pool_avg":
        return {"rel": 1e-6, "max": 1e-5}
    # sums of up to 25600 products in 32 bits: two orders of summation differ by up to 2e-6 of the result's norm
    return {"rel": 1e-5, "max": 1e-4}


def exact(case, seed):
    """The loop nest in 64 bits: per filter tap a matrix product (or a running sum, or maximum) over all positions."""
    B, C, K, W, H, R, S, sw, sh = _dims(case)
    image, filt = _inputs(case, seed)
    out = None
    for r in range(R):
        for s in range(S):
            # [W, H, C, B] -> [C, H, W, B]
            tap = image[r:r + sw * (W - 1) + 1:sw, s:s + sh * (H - 1) + 1:sh].double().permute(2, 1, 0, 3).contiguous()
            if case["op"] == "conv":
                term = torch.mm(filt[:, r, s, :].double().contiguous(), tap.view(C, H * W * B)).view(K, H, W, B)
            else:
                term = tap
            if out is None:
                out = term
            elif case["op"] == "pool_max":
                out = torch.maximum(out, term)
            else:
                out += term
    return out / (R * S) if case["op"] == "pool_avg" else out
