"""Performance cases: the calls that a program serving weight-only-quantized decoder layers makes.

Sizes are those of the decoder blocks in workloads.py (LLaMA / OPT linear layers) and, for drawn cases, anything
the entry points take in the same range: ragged row counts, odd token counts, every weight format and epilogue.
Weights are N(0, 0.02) and activations N(0, 1), as in the benchmark.
"""
from __future__ import annotations

import math

import torch

import paper_2401_14112_amd as fp6

# largest listed call: M * K weights and M * K * N multiply-adds
_MAX_WEIGHTS = 57344 * 8192
_MAX_MACS = 57344 * 8192 * 4096


def _linear(name, fmt, M, K, N, bias=False, residual=False, gated=False, buffers="kept"):
    return {"name": name, "op": "linear", "fmt": fmt, "M": M, "K": K, "N": N, "bias": bias, "residual": residual,
            "gated": gated, "buffers": buffers}


def listed():
    return [
        # one token through the smallest attention projection: launches and host work count
        _linear("decode 1 token, 4096x4096", "fp6", 4096, 4096, 1),
        # the headline feed-forward layer at a decode batch
        _linear("decode 16, 8192x22016", "fp6", 8192, 22016, 16),
        # gate and up projection of a 13b block with silu(gate) * up in the same call, odd batch
        _linear("decode 7 gated, 27648x5120", "fp6", 27648, 5120, 7, gated=True),
        # 4-bit weights, down projection with its residual, a full decode batch
        _linear("decode 32 fp4, 8192x28672", "fp4", 8192, 28672, 32, residual=True),
        # stacked q, k, v projection with bias at the largest decode batch
        _linear("decode 64 bias, 10240x8192", "fp6", 10240, 8192, 64, bias=True),
        # 5-bit weights, attention output of the widest model, batch that fills no token tile
        _linear("decode 45 fp5, 12288x12288", "fp5", 12288, 12288, 45, bias=True, residual=True),
        # a short prompt through 3-bit weights, the call as the short tour writes it (nothing kept by the caller)
        _linear("prompt 100 fp3, 6656x17920", "fp3", 6656, 17920, 100, buffers="fresh"),
        # group-wise scales, prompt of an odd length
        _linear("prompt 201 fp6g, 28672x8192", "fp6g", 28672, 8192, 201),
        # a layer that the program leaves in fp16 (the library's own fp16 kernel)
        _linear("prompt 256 fp16, 9216x9216", "fp16", 9216, 9216, 256),
        # the headline layer at the longest prompt of the benchmark
        _linear("prompt 512, 8192x22016", "fp6", 8192, 22016, 512),
        # a long prompt (or several packed together) through the stacked gate and up projection of a 70b block
        _linear("prompt 4096 gated, 57344x8192", "fp6", 57344, 8192, 4096, gated=True, buffers="fresh"),
        # loading a model: fp16 weights to the packed form
        {"name": "quantize_pack, 8192x22016", "op": "pack", "fmt": "fp6", "M": 8192, "K": 22016},
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    op = rng.choice(["decode", "decode", "decode", "decode", "prompt", "prompt", "prompt", "prompt", "pack", "unpack"])
    fmt = rng.choice(["fp6", "fp6", "fp6", "fp5", "fp4", "fp3", "fp6g", "fp16"])
    while True:
        M = max(1, round(_log_uniform(rng, 1024, 57344) / 16)) * 16
        K = max(1, round(_log_uniform(rng, 1024, 28672) / 256)) * 256
        N = round(_log_uniform(rng, 1, 64)) if op == "decode" else round(_log_uniform(rng, 65, 4096))
        if M * K <= _MAX_WEIGHTS and M * K * N <= _MAX_MACS:
            break
    if op in ("pack", "unpack"):
        return {"op": op, "fmt": "fp6" if fmt == "fp16" else fmt, "M": M, "K": K}
    plain = fmt == "fp16"
    return {"op": "linear", "fmt": fmt, "M": M, "K": K, "N": N,
            "bias": not plain and rng.random() < 0.3, "residual": not plain and rng.random() < 0.3,
            "gated": not plain and rng.random() < 0.3, "buffers": rng.choice(["kept", "kept", "fresh"])}


def _normal(shape, std, generator):
    t = torch.empty(shape, dtype=torch.float32, device="cuda")
    t.normal_(0.0, std, generator=generator)
    return t.to(torch.float16)


def _inputs(case, seed):
    """Weights, activations, bias and residual of a case (None where it has none), from the seed alone."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    M, K = case["M"], case["K"]
    W = _normal((M, K), 0.02, g)
    if case["op"] != "linear":
        return W, None, None, None
    N, rows = case["N"], M // 2 if case["gated"] else M
    X = _normal((N, K), 1.0, g)
    bias = _normal((M,), 0.5, g) if case["bias"] else None
    residual = _normal((N, rows), 1.0, g) if case["residual"] else None
    return W, X, bias, residual


def prepare(case, seed):
    W, X, bias, residual = _inputs(case, seed)
    fmt, M, K = case["fmt"], case["M"], case["K"]
    if case["op"] == "pack":
        # a loader reuses its destination buffers from call to call
        packed, scales = getattr(fp6, fmt + "_quantize_pack")(W)
        return {"call": getattr(fp6, fmt + "_quantize_pack"), "args": (W,), "kwargs": {"packed": packed, "scales": scales}}
    kwargs = {}
    if case["op"] == "unpack":
        packed, scales = getattr(fp6, fmt + "_quantize_pack")(W)
        kwargs["out"] = torch.empty((M, K), dtype=torch.float16, device="cuda")
        return {"call": getattr(fp6, fmt + "_unpack"), "args": (packed, scales, M, K), "kwargs": kwargs}
    N, rows = case["N"], M // 2 if case["gated"] else M
    if case["buffers"] == "kept":
        # a serving loop keeps its output and its zero-filled workspace
        sizes = {"fp16": fp6.fp16_linear_workspace_bytes, "fp6g": fp6.fp6_linear_workspace_bytes}
        nbytes = sizes.get(fmt, getattr(fp6, fmt + "_linear_workspace_bytes", None))(M, N, K)
        kwargs["out"] = torch.empty((N, rows), dtype=torch.float16, device="cuda")
        if nbytes:
            kwargs["workspace"] = torch.zeros(nbytes, dtype=torch.uint8, device="cuda")
    if fmt == "fp16":
        return {"call": fp6.fp16_linear, "args": (W, X), "kwargs": kwargs}
    packed, scales = getattr(fp6, fmt + "_quantize_pack")(W)
    args = (packed, scales, X, M, K)
    if case["bias"] or case["residual"] or case["gated"]:
        kwargs.update(bias=bias, residual=residual, gated=case["gated"])
        return {"call": getattr(fp6, fmt + "_linear_fused"), "args": args, "kwargs": kwargs}
    return {"call": getattr(fp6, fmt + "_linear"), "args": args, "kwargs": kwargs}


def run(state):
    return state["call"](*state["args"], **state["kwargs"])


_BITS = {"fp6": 6, "fp6g": 6, "fp5": 5, "fp4": 4, "fp3": 3, "fp16": 16}


def _weight_bytes(case):
    M, K, fmt = case["M"], case["K"], case["fmt"]
    scales = 0 if fmt == "fp16" else (2 * M * (K // 128) if fmt == "fp6g" else 2 * M)
    return M * K * _BITS[fmt] // 8 + scales


def work(case):
    M, K = case["M"], case["K"]
    if case["op"] != "linear":
        return {"bytes": 2 * M * K + _weight_bytes(case), "flops": 0}
    N, rows = case["N"], M // 2 if case["gated"] else M
    extra = (2 * M if case["bias"] else 0) + (2 * N * rows if case["residual"] else 0)
    return {"bytes": _weight_bytes(case) + 2 * N * K + 2 * N * rows + extra, "flops": 2 * M * K * N}


def tolerance(case):
    # codes, scales and de-quantized weights have one right value, bit for bit
    if case["op"] != "linear":
        return "exact"
    # fp32 sums, one rounding to fp16 (2^-11 of a value at most, 2.1e-4 in the 2-norm); fp6g also rounds each
    # de-quantized weight to fp16 once (2.9e-4 together).  About four times what exact() shows.
    return {"rel": 1.2e-3 if case["fmt"] == "fp6g" else 9e-4, "max": 4e-3}


# (mantissa bits, exponent of the lowest normal binade, largest magnitude)
_GRID = {"fp6": (2, -2, 28.0), "fp6g": (2, -2, 28.0), "fp5": (2, 0, 7.0), "fp4": (1, 0, 6.0), "fp3": (0, 0, 4.0)}


def _grid_values(ratio, fmt):
    """Nearest magnitude of the format, ties to the even code, saturating; ratio >= 0 in 64 bits."""
    m, e_min, largest = _GRID[fmt]
    if m == 0:
        one, two, four = (torch.tensor(v, dtype=ratio.dtype, device=ratio.device) for v in (1.0, 2.0, 4.0))
        q = torch.where(ratio < 1.5, one, torch.where(ratio <= 3.0, two, four))
        return torch.where(ratio <= 0.5, torch.zeros_like(q), q)
    exponent = torch.floor(torch.log2(ratio.clamp(min=2.0 ** e_min)))
    step = torch.exp2(exponent - m)
    return (torch.round(ratio / step) * step).clamp(max=largest)


def _quantized(W, fmt):
    """(64-bit scale before its rounding, 64-bit value of every de-quantized weight)."""
    M, K = W.shape
    w = W.double().view(M, -1, 128 if fmt == "fp6g" else K)
    raw = w.abs().amax(dim=2, keepdim=True) / _GRID[fmt][2]
    scale = raw.half().double()
    ratio = torch.where(scale > 0, w.abs() / torch.where(scale > 0, scale, torch.ones_like(scale)), torch.zeros_like(w))
    return raw.view(M, -1), (torch.copysign(_grid_values(ratio, fmt), w) * scale).view(M, K)


def exact(case, seed):
    W, X, bias, residual = _inputs(case, seed)
    fmt, M = case["fmt"], case["M"]
    chunk = 2048  # rows at a time: the 64-bit copies of a whole layer would be large
    if case["op"] == "pack":
        raw = torch.cat([_quantized(W[i:i + chunk], fmt)[0] for i in range(0, M, chunk)])
        return None, raw if fmt == "fp6g" else raw.view(-1)
    if case["op"] == "unpack":
        return torch.cat([_quantized(W[i:i + chunk], fmt)[1] for i in range(0, M, chunk)])
    X = X.double()
    z = torch.cat([X @ (W[i:i + chunk].double() if fmt == "fp16" else _quantized(W[i:i + chunk], fmt)[1]).t().contiguous()
                   for i in range(0, M, chunk)], dim=1)
    if bias is not None:
        z += bias.double()
    if case["gated"]:
        gate, up = z[:, 0::2], z[:, 1::2]
        z = gate * torch.sigmoid(gate) * up
    if residual is not None:
        z = z + residual.double()
    return z
