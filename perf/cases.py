"""Performance cases of the integer attention library: what a program that serves quantised vision
transformers calls, through ``paper_2604_25306_amd.Context``, over the sizes it calls it with.

A case is one attention layer: a shape [B,H,N,d], the KV tile of the algorithm, the distribution its
activations are drawn from, and the entry point ("path"):

    tensor         Context.attention, one set of constants            (static per-tensor quantisation)
    head           Context.attention, one set of constants per head   (static per-head quantisation)
    static         Context.attention_static                           (callers that must not allocate)
    bias           Context.attention with a bias as it is             (windowed attention)
    packed         Context.attention_packed_bias                      (the layer's bias packed once)
    dynamic        Context.attention_dynamic from float32             (scales found on the fly)
    dynamic_bias   the same with a bias in real units and a mask

For the windowed paths B = images x windows and the bias holds one slice per window and head.
"""
import ctypes
import math

import numpy as np
import torch

import paper_2604_25306_amd as qf
from workloads import EXCLUDED, head_gains

DEV = "cuda:0"


def _case(name, path, B, H, N, d, kv_tile=64, values="normal", sigma=1.0, windows=0):
    c = {"path": path, "B": B, "H": H, "N": N, "d": d, "kv_tile": kv_tile, "values": values, "sigma": sigma,
         "windows": windows}
    return dict(c, name=name) if name else c


def listed():
    return [
        # one image through the smallest model: interactive use, all latency
        _case("vit_tiny_b1", "tensor", 1, 3, 197, 64),
        # a small server batch through the entry point for callers that must not allocate
        _case("vit_small_b8_static", "static", 8, 6, 197, 64, sigma=1.5),
        # the benchmark's headline layer: a full batch of the base model at 224 pixels
        _case("vit_base_b64", "tensor", 64, 12, 197, 64),
        # the same layer quantised per head
        _case("vit_base_b64_per_head", "head", 64, 12, 197, 64),
        # the same layer from float32 activations, scales found on the fly
        _case("vit_base_b64_dynamic", "dynamic", 64, 12, 197, 64),
        # 384 pixels, wide KV tile: the largest layer of the benchmark
        _case("deit_base384_b32_kv128", "tensor", 32, 12, 577, 64, kv_tile=128, sigma=1.5),
        # 384 pixels, large model, heavy-tailed activations (coarse scales)
        _case("vit_large384_b16_heavy", "tensor", 16, 16, 577, 64, values="student_t3"),
        # a long sequence of small heads
        _case("long_d32_n2100", "tensor", 8, 8, 2100, 32),
        # windowed attention, third stage, small batch, bias packed once
        _case("swin_s3_b8_packed", "packed", 32, 12, 49, 32, windows=4),
        # windowed attention, second stage, small batch, the bias handed over as the model holds it
        _case("swin_s2_b8_bias", "bias", 128, 6, 49, 32, windows=16),
        # windowed attention, first stage, full batch
        _case("swin_s1_b64_packed", "packed", 4096, 3, 49, 32, windows=64),
        # the same from float32 activations and a float32 bias with the shifted-window mask
        _case("swin_s1_b64_dynamic", "dynamic_bias", 4096, 3, 49, 32, windows=64),
    ]


MAX_OPS = 32.0e9       # of a drawn case: below the largest listed one
MAX_ELEMENTS = 19.0e6  # B*H*N*d of a drawn case, likewise


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One layer of the ranges the listed cases stand for: models of 3 to 16 heads at 112 to 512 pixels
    (whole sequences, 50 to 1025 tokens), long sequences of small heads, windowed models (windows of
    7, 8 or 12 tokens a side), from one image to a full batch."""
    family = rng.choice(("vit", "vit", "vit", "long", "window", "window"))
    if family == "vit":
        path = rng.choice(("tensor", "tensor", "head", "static", "dynamic"))
        H, d, N = rng.choice((3, 6, 12, 16)), 64, _log_int(rng, 50, 1025)
    elif family == "long":
        path = rng.choice(("tensor", "dynamic"))
        H, d, N = rng.choice((4, 8, 12)), 32, _log_int(rng, 300, 2100)
    if family != "window":
        most = min(64, int(MAX_OPS / (4.0 * N * N * d * H)), int(MAX_ELEMENTS / (H * N * d)))
        # (per-head ranges spread by a factor of 16: tails on top of that leave the library's window of
        # scales; attention_static refuses scales so fine that their table exceeds its memory)
        values = "normal" if path == "head" else rng.choice(("normal", "normal", "student_t3"))
        sigma = round(rng.uniform({"static": 1.4, "head": 1.0}.get(path, 0.8), 1.6), 2)
        return _case(None, path, _log_int(rng, 1, max(1, most)), H, N, d, kv_tile=rng.choice((64, 64, 128)),
                     values=values, sigma=sigma)
    path = rng.choice(("packed", "packed", "bias", "dynamic_bias"))
    side = rng.choice((7, 7, 8, 12))
    stage = rng.randrange(4)
    N, H, windows = side * side, 3 << stage, 64 >> (2 * stage)
    windows = max(windows, 1)
    images = _log_int(rng, 1, min(64, int(MAX_ELEMENTS / (H * N * 32 * windows))))
    return _case(None, path, images * windows, H, N, 32, sigma=round(rng.uniform(0.8, 1.6), 2), windows=windows)


def _floats(case, gen):
    """Activations [B,H,N,d] in float32: normal, or Student-t with 3 degrees of freedom (cut at 50) and
    1 % of the channels eight times as large."""
    shape = (case["B"], case["H"], case["N"], case["d"])
    x = torch.randn(shape, generator=gen, device=DEV)
    if case["values"] == "student_t3":
        chi = sum(torch.randn(shape, generator=gen, device=DEV).square_() for _ in range(3))
        x = (x / (chi / 3.0).sqrt_()).clamp_(-50.0, 50.0)
        channels = case["H"] * case["d"]
        loud = torch.randperm(channels, generator=gen, device=DEV)[: -(-channels // 100)]
        gain = torch.ones(channels, device=DEV)
        gain[loud] = 8.0
        x *= gain.view(1, case["H"], 1, case["d"])
    return x.mul_(case["sigma"])


def _quantise(x):
    """Per-tensor symmetric int8: (int8 tensor, scale)."""
    s = float(x.abs().max()) / 127.0
    return torch.clamp(torch.round(x / s), -127, 127).to(torch.int8), s


def _window_bias(case, gen):
    """Relative-position bias in real units (table ~ N(0, 0.5^2)) and the shifted-window mask, which
    every second window carries: ([windows,H,N,N] float32, the same as uint8)."""
    n, H, w = case["N"], case["H"], case["windows"]
    side = int(round(math.sqrt(n)))
    ys, xs = np.divmod(np.arange(n), side)
    index = (ys[:, None] - ys[None, :] + side - 1) * (2 * side - 1) + (xs[:, None] - xs[None, :] + side - 1)
    table = 0.5 * torch.randn((H, (2 * side - 1) ** 2), generator=gen, device=DEV)
    real = table[:, torch.from_numpy(index).to(DEV)].expand(w, H, n, n).contiguous()
    split = side - side // 2
    label = (ys >= split) * 2 + (xs >= split)
    mask = torch.zeros((w, H, n, n), dtype=torch.uint8, device=DEV)
    mask[1::2] = torch.from_numpy((label[:, None] != label[None, :]).astype(np.uint8)).to(DEV)
    return real, mask


_context = None


def _ctx():
    """A program keeps one context for all its layers."""
    global _context
    if _context is None:
        _context = qf.Context(0)
    return _context


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    path, d, ctx = case["path"], case["d"], _ctx()
    B, H, N = case["B"], case["H"], case["N"]
    s = {"ctx": ctx, "path": path, "tile": case["kv_tile"],
         "O": torch.empty((B, H, N, d), dtype=torch.int8, device=DEV)}
    x = [_floats(case, gen) for _ in range(3)]
    if path in ("dynamic", "dynamic_bias"):
        s["x"] = x
        s["info"] = torch.zeros(ctypes.sizeof(qf.DynamicInfo), dtype=torch.uint8, device=DEV)
        s["bias"] = s["mask"] = None
        if path == "dynamic_bias":
            s["bias"], s["mask"] = _window_bias(case, gen)
            n = qf.qflash_dynamic_bias_workspace_bytes(B, H, N, d, case["windows"], H)
        else:
            n = qf.qflash_dynamic_workspace_bytes(B, H, N, d)
        s["workspace"] = torch.empty(n, dtype=torch.uint8, device=DEV)
        return s
    if path == "head":
        gains = torch.from_numpy(head_gains(H)).to(DEV, torch.float32).view(1, H, 1, 1)
        heads = [[_quantise(t[:, h]) for h in range(H)] for t in (y * gains for y in x)]
        s["x"] = [torch.stack([q for q, _ in t], dim=1).contiguous() for t in heads]
        (sq, sk, sv) = ([scale for _, scale in t] for t in heads)
        s["params"] = qf.params_array([qf.qflash_params_from_scales(sq[h], sk[h], sv[h], d) for h in range(H)])
        return s
    (Q, sq), (K, sk), (V, sv) = (_quantise(y) for y in x)
    s["x"] = [Q, K, V]
    s["params"] = qf.qflash_params_from_scales(sq, sk, sv, d)
    if path in ("bias", "packed"):
        real, mask = _window_bias(case, gen)
        unit = (sq * sk) / math.sqrt(float(d))
        bias = torch.floor(real.double() / unit + 0.5).to(torch.int32)
        bias[mask != 0] = int(EXCLUDED)
        s["bias_shape"] = (case["windows"], H)
        s["bias"] = ctx.pack_bias(bias) if path == "packed" else bias
    return s


def run(s):
    path, ctx, O, tile = s["path"], s["ctx"], s["O"], s["tile"]
    q, k, v = s["x"]
    if path == "tensor" or path == "head":
        ctx.attention(q, k, v, O, s["params"], tile)
    elif path == "static":
        ctx.attention_static(q, k, v, O, s["params"], tile)
    elif path == "bias":
        ctx.attention(q, k, v, O, s["params"], tile, bias=s["bias"])
    elif path == "packed":
        ctx.attention_packed_bias(q, k, v, O, s["params"], tile, s["bias"], *s["bias_shape"])
    else:
        ctx.attention_dynamic(q, k, v, O, tile, s["workspace"], info=s["info"], bias_real=s["bias"], excluded=s["mask"])
        return {"O": O, "info": s["info"]}
    return {"O": O}


def work(case):
    """Every input read once and every output written once; multiply-adds of the two products count two."""
    n = float(case["B"]) * case["H"] * case["N"] * case["d"]
    slices = float(case["windows"]) * case["H"] * case["N"] * case["N"]
    per_element = 13 if case["path"] in ("dynamic", "dynamic_bias") else 4
    per_bias = {"bias": 4, "packed": 4, "dynamic_bias": 5}.get(case["path"], 0)
    return {"bytes": per_element * n + per_bias * slices, "flops": 4.0 * case["N"] * n}


def tolerance(case):
    return "exact"            # integers throughout; the quantiser's float32 operations are pinned one by one
