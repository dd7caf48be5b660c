"""The calls whose speed matters to a user of the quantized linear layer.

A serving program packs its layers once, keeps the packed buffers, a workspace and the output buffers, and then calls
the linear entry points for every token (decode), for a few sequences at a time (batched or speculative decoding) and
for every prompt (prefill).  The sizes are the layer shapes of `paper_2506_10443_amd.synth.MODELS` (Qwen2-1.5B,
Qwen2-7B, Llama-3-8B), with q|k|v and gate|up concatenated along N as `bench.py` does; `draw` fills the ranges between
them, ragged sizes included.

A case is one of
  kind "layer": one projection, rows = N, cols = K;
  kind "block": the four projections of a transformer block, hidden / kv / ffn its widths;
  kind "load":  packing one fp32 matrix, rows = N, cols = K (what a program does once per layer when it starts);
with tokens = M, weights = the packed form, act = "a8" (fp32 in, quantized to int8 inside the call) or "a16" (fp16 in),
out = the type of the result.
"""
from __future__ import annotations

import math

import torch

from paper_2506_10443_amd import binding as B

MODES = {
    "w4": B.MODE_W4_ZP_INT,                              # int4, integer zero point: smallest packed form
    "w4+plane": B.MODE_W4_ZP_INT | B.WITH_MATRIX_PLANE,  # the same and the copy for the matrix instructions
    "w4min": B.MODE_W4_MIN_FLOAT,                        # Eq. 1 as printed: float group minimum
    "w8": B.MODE_W8_MIN_FLOAT | B.NATIVE_8BIT,           # int8 weights stored as bytes
    "w8planes": B.MODE_W8_MIN_FLOAT,                     # int8 weights as nibble planes (what fp16 activations take)
}
BYTES_PER_WEIGHT = {  # codes and the group parameters, read once
    "w4": 0.5 + 5 / 64, "w4+plane": 0.5 + 5 / 64, "w4min": 0.5 + 8 / 64, "w8": 1 + 8 / 64, "w8planes": 1 + 8 / 64,
}
LARGEST = 2048 * (6144 * 4096 + 4096 * 4096 + 28672 * 4096 + 4096 * 14336)  # multiply-adds of the largest listed case


def _layer(name, tokens, rows, cols, weights, act="a8", out="f32"):
    return {"name": name, "kind": "layer", "tokens": tokens, "rows": rows, "cols": cols,
            "weights": weights, "act": act, "out": out}


def _block(name, tokens, hidden, kv, ffn, weights, act="a8", out="f32"):
    return {"name": name, "kind": "block", "tokens": tokens, "hidden": hidden, "kv": kv, "ffn": ffn,
            "weights": weights, "act": act, "out": out}


def listed():
    return [
        # the smallest call: one token through one square projection of the smallest model
        _layer("decode 1.5b o", 1, 1536, 1536, "w4"),
        # one token through a block: what every generated token costs, 28 times
        _block("decode 7b block", 1, 3584, 512, 18944, "w4"),
        # the same with fp16 activations and results
        _block("decode 8b block a16", 1, 4096, 1024, 14336, "w4", "a16", "f16"),
        # the vocabulary projection of one token, int4 and (what the method recommends for this layer) int8
        _layer("decode 7b lm_head", 1, 152064, 3584, "w4"),
        _layer("decode 7b lm_head w8", 1, 152064, 3584, "w8"),
        # five tokens: speculative decoding, or a few sequences at once
        _block("5 tokens 8b block", 5, 4096, 1024, 14336, "w4"),
        # batched decoding of 48 sequences on the buffers that prefill uses too
        _block("48 tokens 7b block", 48, 3584, 512, 18944, "w4+plane"),
        # prompts: the smallest model, the middle one, and a ragged prompt on int8 weights
        _block("512 tokens 1.5b block", 512, 1536, 256, 8960, "w4+plane"),
        _block("1024 tokens 7b block", 1024, 3584, 512, 18944, "w4+plane"),
        _block("333 tokens 8b block w8", 333, 4096, 1024, 14336, "w8"),
        # the largest: a long prompt with fp16 activations and results
        _block("2048 tokens 8b block a16", 2048, 4096, 1024, 14336, "w4", "a16", "f16"),
        # loading a model: quantize and rearrange the largest matrix of a block
        {"name": "load 7b gate|up", "kind": "load", "rows": 37888, "cols": 3584, "weights": "w4+plane"},
    ]


def _log_uniform(rng, lo, hi, step=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / step)) * step))


def _form(rng, tokens):
    """Packed form, activations and result type of a drawn case."""
    act = "a16" if rng.random() < 0.25 else "a8"
    if act == "a16":
        weights = rng.choices(["w4", "w4min", "w8planes"], [6, 1, 1])[0]
    elif tokens <= 16:
        weights = rng.choices(["w4", "w4+plane", "w4min", "w8"], [5, 2, 1, 2])[0]
    else:
        weights = rng.choices(["w4", "w4+plane", "w4min", "w8"], [2, 5, 1, 2])[0]
    return weights, act, rng.choice(["f32", "f16"])


def draw(rng):
    kind = rng.choices(["layer", "block", "load"], [3, 8, 1])[0]
    if kind == "load":
        return {"kind": "load", "rows": _log_uniform(rng, 1024, 37888, 16), "cols": _log_uniform(rng, 1024, 18944, 128),
                "weights": rng.choice(["w4", "w4+plane", "w4min", "w8"])} if rng.random() < 0.5 else \
               {"kind": "load", "rows": _log_uniform(rng, 1024, 37888, 16), "cols": _log_uniform(rng, 1024, 4096, 64),
                "weights": rng.choice(["w4", "w4+plane"])}
    phase = rng.choices(["decode", "few", "batch", "prompt"], [4, 2, 2, 4])[0]
    tokens = {"decode": 1, "few": rng.randint(2, 16), "batch": rng.randint(17, 128),
              "prompt": _log_uniform(rng, 129, 2048)}[phase]
    weights, act, out = _form(rng, tokens)
    step = 128 if weights in ("w8", "w8planes") else 64  # int8 weights: K a multiple of 128
    case = {"kind": kind, "tokens": tokens}
    if kind == "layer":
        cols = _log_uniform(rng, 1024, 4096, step)
        # the vocabulary projection is called with one token, or with one per sequence
        rows = _log_uniform(rng, 512, 152064 if tokens <= 16 else 37888, 16)
        if rng.random() < 0.25:  # a down projection: the long axis is the reduction
            rows, cols = _log_uniform(rng, 1024, 4096, 16), _log_uniform(rng, 4096, 18944, step)
        case.update(rows=rows, cols=cols)
        weight = rows * cols
    else:
        hidden = _log_uniform(rng, 1024, 4096, step)
        kv = max(128, hidden // rng.choice([1, 2, 4, 7, 8]) // 16 * 16)
        ffn = min(18944, int(hidden * rng.uniform(2.5, 5.8)) // step * step)
        case.update(hidden=hidden, kv=kv, ffn=ffn)
        weight = sum(n * k for n, k in _shapes(case))
    case.update(weights=weights, act=act, out=out)
    case["tokens"] = max(1, min(tokens, int(0.6 * LARGEST) // weight))
    return case


def _shapes(case):
    """(N, K) of the case's projections."""
    if case["kind"] != "block":
        return [(case["rows"], case["cols"])]
    h, kv, f = case["hidden"], case["kv"], case["ffn"]
    return [(h + 2 * kv, h), (h, h), (2 * f, h), (h, f)]


def _inputs(gen, tokens, cols, act):
    """N(0, 1) activations, 0.1 % of the channels of every token twenty times larger."""
    x = torch.randn((tokens, cols), generator=gen, device="cuda")
    channels = torch.randperm(cols, generator=gen, device="cuda")[:max(1, round(0.001 * cols))]
    x[:, channels] *= 20.0
    return x.half() if act == "a16" else x


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    mode = MODES[case["weights"]]
    state = {"kind": case["kind"], "mode": mode}
    if case["kind"] == "load":
        n, k = case["rows"], case["cols"]
        state["W"] = torch.randn((n, k), generator=gen, device="cuda").mul_(0.02)
        state["packed"] = torch.zeros(B.mnnq_packed_size(n, k, B.GROUP, mode), dtype=torch.uint8, device="cuda")
        return state
    tokens, work, calls = case["tokens"], 16, []
    for n, k in _shapes(case):
        w = torch.randn((n, k), generator=gen, device="cuda").mul_(0.02)
        packed = B.mnnq_pack_weights(w, mode=mode)
        del w
        x = _inputs(gen, tokens, k, case["act"])
        y = torch.empty((tokens, n), dtype=torch.float16 if case["out"] == "f16" else torch.float32, device="cuda")
        calls.append((packed, n, k, x, y[0] if tokens == 1 else y))
        work = max(work, B.mnnq_workspace_size(tokens, n, k, B.GROUP, mode))
    state["calls"] = calls
    state["workspace"] = torch.empty(work, dtype=torch.uint8, device="cuda")
    state["entry"] = {
        (True, "a8", "f32"): B.mnnq_linear_decode_fused, (True, "a8", "f16"): B.mnnq_linear_decode_fused_o16,
        (True, "a16", "f32"): B.mnnq_linear_decode_f16, (True, "a16", "f16"): B.mnnq_linear_decode_f16_o16,
        (False, "a8", "f32"): B.mnnq_linear_prefill_fused, (False, "a8", "f16"): B.mnnq_linear_prefill_fused_o16,
        (False, "a16", "f32"): B.mnnq_linear_prefill_f16, (False, "a16", "f16"): B.mnnq_linear_prefill_f16_o16,
    }[tokens == 1, case["act"], case["out"]]
    state["act"] = case["act"]
    return state


def run(state):
    mode = state["mode"]
    if state["kind"] == "load":
        return B.mnnq_pack_weights(state["W"], out=state["packed"], mode=mode)
    entry = state["entry"]
    if state["act"] == "a16":
        return [entry(packed, n, k, x, out=y, mode=mode) for packed, n, k, x, y in state["calls"]]
    workspace = state["workspace"]
    return [entry(packed, n, k, x, out=y, workspace=workspace, mode=mode) for packed, n, k, x, y in state["calls"]]


def work(case):
    if case["kind"] == "load":
        n, k = case["rows"], case["cols"]
        plane = n * k * (0.75 + 4 / 64) if case["weights"] == "w4+plane" else 0
        return {"bytes": 4 * n * k + n * k * BYTES_PER_WEIGHT[case["weights"]] + plane, "flops": 0}
    m, total, flops = case["tokens"], 0.0, 0
    for n, k in _shapes(case):
        total += n * k * BYTES_PER_WEIGHT[case["weights"]]
        total += m * k * (2 if case["act"] == "a16" else 4) + m * n * (2 if case["out"] == "f16" else 4)
        flops += 2 * m * n * k
    return {"bytes": total, "flops": flops}


def tolerance(case):
    if case["kind"] == "load":
        return "exact"  # the quantizer is a fixed sequence of IEEE operations
    # fp32 sums over up to 296 groups in any order; a binary16 result is such a sum rounded once (half a unit: 2^-11
    # of the value at most, where two sums fall on either side of a tie)
    return {"rel": 1e-5} if case["out"] == "f32" else {"rel": 3e-4, "max": 2e-3}
