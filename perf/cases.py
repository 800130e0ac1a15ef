"""The calls this library is used for, as measurable cases.

A case is one call on packed low-bit weights through the public Python entry points:
``LutGemm.fused`` and ``LutGemm.__call__`` (one-call and precompute + mpGEMM forms),
``LutGemm.dequant`` (the matrix-core comparison path) or ``pack_weights`` (the offline
mapping).  Layer shapes are those of ``workloads/`` (LLaMA-2 7B / 13B / 70B and BitNet
layers) plus a ragged one; ``draw`` spreads the same options over the whole range of sizes.
"""
from __future__ import annotations

import math

import torch

import paper_2408_06003_amd as L

KBLK = 128             # K granularity of the packed weights
MNK_MAX = 2048 * 5120 * 27648
WEIGHTS_MAX = 8192 * 28672

_WFMT = {"uint": L.WFMT_UINT, "binary": L.WFMT_BINARY, "ternary": L.WFMT_TERNARY, "ternary3in5": L.WFMT_TERNARY_3IN5}
_ACT = {"fp16": L.ACT_FP16, "int8": L.ACT_INT8, "lut8": L.ACT_FP16_LUT8}
_OUT = {"fp16": torch.float16, "fp32": torch.float32, "int32": torch.int32}


def _case(name, entry, fmt, bits, group, act, out, m, k, n, residual=False):
    """group: quantization group along K, 0 = one scale per tensor, -1 = per channel."""
    c = {"entry": entry, "fmt": fmt, "bits": bits, "group": group, "act": act, "out": out,
         "m": m, "k": k, "n": n, "residual": residual}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: a 1k GEMV, all latency (precompute + mpGEMM, two launches)
        _case("gemv_int2_1k", "call", "uint", 2, 128, "fp16", "fp16", 1, 1024, 1024),
        # BitNet-style decode: ternary weights, per-token INT8 activations, one launch
        _case("gemv_ternary_int8_4k", "fused", "ternary", 2, 0, "int8", "fp32", 1, 4096, 4096),
        # LLaMA-7B decode, the gate/up projection with INT4 groups of 128
        _case("decode_int4_7b_up", "fused", "uint", 4, 128, "fp16", "fp16", 1, 4096, 22016),
        # LLaMA-70B decode, the down projection with binary weights, precompute + mpGEMM
        _case("decode_binary_70b_down", "call", "binary", 1, -1, "fp16", "fp16", 1, 28672, 8192),
        # a small serving batch on the 7B QKV projection
        _case("batch8_int4_7b_qkv", "fused", "uint", 4, 128, "fp16", "fp16", 8, 4096, 12288),
        # a serving batch on the 70B up projection, precompute + mpGEMM
        _case("batch16_binary_70b_up", "call", "binary", 1, -1, "fp16", "fp16", 16, 8192, 28672),
        # a BitNet serving batch: exact INT8 path with several tokens
        _case("batch64_ternary_int8_4k", "fused", "ternary", 2, 0, "int8", "fp32", 64, 4096, 4096),
        # odd sizes: ragged tokens and columns, per-channel scale and zero, added onto a residual
        _case("ragged37_int2_residual", "fused", "uint", 2, -1, "fp16", "fp32", 37, 2944, 3001, residual=True),
        # prompt processing, INT2 groups of 128, precompute + mpGEMM
        _case("prefill_int2_4k", "call", "uint", 2, 128, "fp16", "fp16", 4096, 4096, 4096),
        # prompt processing on the LLaMA-2-13B MLP shape, binary weights: the largest call
        _case("prefill_binary_13b_mlp", "fused", "binary", 1, -1, "fp16", "fp16", 2048, 5120, 27648),
        # the dequantization path on a prompt chunk of a 7B layer
        _case("dequant256_int4_7b_qkv", "dequant", "uint", 4, 128, "fp16", "fp16", 256, 4096, 12288),
        # loading a model: packing one 7B layer's INT4 codes
        _case("pack_int4_7b_qkv", "pack", "uint", 4, 128, "fp16", "fp16", 1, 4096, 12288),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    fmt, bits, act = rng.choice([
        ("uint", 4, "fp16"), ("uint", 4, "fp16"), ("uint", 2, "fp16"), ("uint", 2, "fp16"), ("uint", 1, "fp16"),
        ("binary", 1, "fp16"), ("binary", 1, "fp16"), ("ternary", 2, "fp16"), ("ternary", 2, "int8"),
        ("ternary", 2, "int8"), ("binary", 1, "int8"), ("ternary3in5", 2, "int8"), ("uint", 4, "lut8")])
    entry = rng.choice(["fused", "fused", "fused", "call", "call", "call", "dequant", "pack"])
    if entry == "dequant" and (act != "fp16" or fmt == "ternary3in5"):
        entry = "call"
    # the niche formats stay at decode and small-batch sizes
    niche = fmt == "ternary3in5" or act == "lut8"
    k = KBLK * _log_int(rng, 4, 224)
    n = _log_int(rng, 64, 28672)
    if rng.random() < 0.5:
        n |= 1                                  # odd column counts
    while n * k > WEIGHTS_MAX:
        n = max(64, n // 2)
    m = 1 if entry == "pack" else _log_int(rng, 1, 16 if niche else 4096)
    while m * n * k > MNK_MAX:
        m = max(1, m // 2)
    if fmt == "uint":
        group = rng.choice([128, 128, 128, -1, 0])
    elif fmt == "ternary" and act == "fp16":
        group = rng.choice([0, -1])
    elif fmt in ("ternary", "ternary3in5"):
        group = 0
    else:
        group = -1
    out = rng.choice(["fp32", "int32"]) if act == "int8" else rng.choice(["fp16", "fp16", "fp32"])
    residual = entry in ("fused", "call") and out != "int32" and rng.random() < 0.2
    return _case(None, entry, fmt, bits, group, act, out, m, k, n, residual)


def _n_groups(case):
    return 1 if case["group"] <= 0 else case["k"] // case["group"]


def _problem(case):
    k, group = case["k"], case["group"]
    return L.problem(k, case["n"], case["bits"], _WFMT[case["fmt"]], k if group < 0 else group,
                     act=_ACT[case["act"]], scale_fp32=(group == 0 and case["fmt"] != "uint"))


def _inputs(case, seed):
    """Codes, scales, zeros, activations (and residual) as tensors on the GPU."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed) % (1 << 62))
    m, k, n = case["m"], case["k"], case["n"]
    shape = (1,) if case["group"] == 0 else (n, _n_groups(case))

    def uniform(lo, hi, size):
        return torch.rand(size, generator=gen, device="cuda") * (hi - lo) + lo

    if case["fmt"].startswith("ternary"):
        codes = torch.randint(-1, 2, (n, k), generator=gen, device="cuda", dtype=torch.int8)
    else:
        codes = torch.randint(0, 1 << case["bits"], (n, k), generator=gen, device="cuda", dtype=torch.uint8)
    scales = uniform(0.01, 0.1, shape)
    fp32_scale = case["group"] == 0 and case["fmt"] != "uint"
    scales = scales if fp32_scale else scales.half()
    zeros = uniform(0.0, float((1 << case["bits"]) - 1), shape).half() if case["fmt"] == "uint" else None
    # hidden states: normal, a different magnitude per token, a few outlier channels
    a = torch.randn((m, k), generator=gen, device="cuda")
    a *= torch.exp(0.5 * torch.randn((m, 1), generator=gen, device="cuda"))
    a[:, torch.randint(0, k, (max(1, k // 1024),), generator=gen, device="cuda")] *= 6.0
    residual = None
    if case["residual"]:
        residual = torch.randn((m, n), generator=gen, device="cuda").to(_OUT[case["out"]])
    return codes, scales, zeros, a.half(), residual


def prepare(case, seed):
    p = _problem(case)
    codes, scales, zeros, act, residual = _inputs(case, seed)
    if case["entry"] == "pack":
        packed = torch.zeros(L.packed_weight_size(p), dtype=torch.uint8, device="cuda")
        return {"case": case, "p": p, "codes": codes, "scales": scales, "zeros": zeros, "packed": packed}
    return {"case": case, "layer": L.LutGemm(p, codes, scales, zeros), "act": act, "residual": residual}


def run(state):
    case = state["case"]
    if case["entry"] == "pack":
        L.pack_weights(state["p"], state["codes"], state["scales"], state["zeros"], state["packed"])
        return state["packed"]
    layer, act = state["layer"], state["act"]
    call = {"fused": layer.fused, "call": layer, "dequant": layer.dequant}[case["entry"]]
    if state["residual"] is not None:
        return call(act, out=state["residual"].clone(), accumulate=True)
    return call(act, out_dtype=_OUT[case["out"]])


def work(case):
    m, k, n, bits = case["m"], case["k"], case["n"], case["bits"]
    groups = _n_groups(case)
    meta = 8 if case["group"] == 0 else n * groups * (4 if case["fmt"] == "uint" else 2)
    weights = n * k * bits // 8
    if case["fmt"] == "ternary3in5":
        weights = n * ((k + 2) // 3) * 5 // 8
    if case["entry"] == "pack":
        return {"bytes": n * k + weights + 2 * meta, "flops": 0}
    out = m * n * (2 if case["out"] == "fp16" else 4)
    return {"bytes": weights + meta + 2 * m * k + out * (2 if case["residual"] else 1), "flops": 2 * m * k * n}


def tolerance(case):
    if case["entry"] == "pack" or (case["act"] == "int8" and not case["residual"]):
        return "exact"                       # bytes; integer sums and two fixed FP32 products
    if case["act"] == "int8":
        return {"rel": 1e-6, "max": 1e-5}    # one more FP32 addition (the residual)
    if case["act"] == "lut8":
        return {"rel": 1.5e-2, "max": 1e-1}  # tables rounded to 8 bits
    # FP16 table entries (or FP16 weights) and FP16 sums of a few of them, FP16 or FP32 out:
    # measured 2e-4 .. 5e-4 and up to 3e-3 against float64
    return {"rel": 2e-3, "max": 1e-2}


def exact(case, seed):
    if case["entry"] == "pack":
        return None
    codes, scales, zeros, act, residual = _inputs(case, seed)
    m, k, n = case["m"], case["k"], case["n"]
    if case["act"] == "int8":                # the quantizer is defined in FP32
        a32 = act.float()
        amax = a32.abs().amax(dim=1, keepdim=True)
        inv = torch.where(amax == 0, torch.zeros_like(amax), 127.0 / amax)
        a = torch.clamp(torch.round(a32 * inv), -127, 127).double()
        token = amax.double() / 127.0
    else:
        a = act.double()
    groups = _n_groups(case)
    y = torch.empty((m, n), dtype=torch.float64, device=act.device)
    for lo in range(0, n, 4096):
        hi = min(n, lo + 4096)
        w = codes[lo:hi].double()
        if case["fmt"] == "binary":
            w = 2.0 * w - 1.0
        if zeros is not None:
            z = zeros.double() if case["group"] == 0 else zeros[lo:hi].double()
            w = (w.view(hi - lo, groups, -1) - z.view(-1, groups, 1)).view(hi - lo, k)
        if case["out"] != "int32":
            s = scales.double() if case["group"] == 0 else scales[lo:hi].double()
            w = (w.view(hi - lo, groups, -1) * s.view(-1, groups, 1)).view(hi - lo, k)
        y[:, lo:hi] = a @ w.t()
    if case["act"] == "int8" and case["out"] != "int32":
        y = y * token
    if residual is not None:
        y = y + residual.double()
    return y
