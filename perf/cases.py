"""Timed cases of the packed attention library: what its users call, over the range of sizes they call it with.

A case names a length recipe and a shape; `prepare` makes the packed batch, `run` is one call (or one training
step: forward, then backward) through the Python binding.  Values are N(0, 1) rounded to bf16, as in the
repository's workloads.

Keys of an attention case
    recipe, n, lo, hi, lens_seed   how the sample lengths come about (see `lengths`)
    hq, hkv, d, causal             heads, head dimension, mask
    step                           True: forward + backward, False: forward only
    hint                           pass the longest sample as max_seqlen, as callers of a varlen interface do
    kept                           outputs and workspaces are the caller's, kept from call to call; otherwise the
                                   binding allocates them, as in its shortest call
Keys of a merge case: parts, tokens, hq, d.
"""
import math

import numpy as np
import torch

from paper_2605_08962_amd import binding
from paper_2605_08962_amd import workloads as W

DIMS = (64, 80, 96, 128)


def _attn(name, recipe, n, lo, hi, hq, hkv, d, causal, step, hint=True, kept=True, lens_seed=0):
    case = {"kind": "attn", "recipe": recipe, "n": n, "lo": lo, "hi": hi, "lens_seed": lens_seed, "hq": hq, "hkv": hkv,
            "d": d, "causal": causal, "step": step, "hint": hint, "kept": kept}
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # The smallest calls: a handful of short samples, where launches and host time are everything.  The four
        # samples of the repository's first workload, forward; and a small causal batch, one training step.
        _attn("tiny-fwd-d64", "tiny", 4, 16, 129, 2, 2, 64, False, False, hint=False, kept=False),
        _attn("tiny-causal-step-d128", "log", 6, 30, 200, 4, 1, 128, True, True, hint=False, kept=False, lens_seed=3),
        # One rank's share in the sequence-parallel state: every token of one long sample, a few of the heads.  Too
        # small to fill the GPU by rows alone: forward of a ViT-like sample, training steps of causal ones.
        _attn("slice-8k-fwd-d80", "one", 1, 8192, 8192, 2, 2, 80, False, False),
        _attn("slice-4k-causal-step-d128", "one", 1, 4096, 4096, 2, 2, 128, True, True),
        _attn("slice-8k-gqa-causal-step-d128", "one", 1, 8191, 8191, 4, 1, 128, True, True),
        # Batches of short samples (speech clips, small images): bound by memory and latency, not by arithmetic.
        _attn("short-fwd-d64", "log", 512, 64, 384, 16, 16, 64, False, False, lens_seed=5),
        _attn("short-step-d80", "log", 256, 64, 1024, 16, 16, 80, False, True, lens_seed=1003),
        # The ViT encoder on dynamic-resolution images: a frozen encoder's forward and a training step.
        _attn("vit-fwd-d64", "vit", 64, 0, 0, 16, 16, 64, False, False, lens_seed=1002),
        _attn("vit-step-d64", "vit", 64, 0, 0, 16, 16, 64, False, True, lens_seed=1002),
        # A 65536-token sample packed with 256 short ones (one rank of the sequence-parallel state).
        _attn("long-short-step-d80", "long", 256, 65536, 0, 16, 16, 80, False, True, lens_seed=1003),
        # The LLM backbone's packed microbatch: causal, grouped heads, training step.
        _attn("llm-step-d128", "pack", 32768, 0, 0, 32, 8, 128, True, True, lens_seed=1004),
        # Context parallelism over key shards: partial results of four shards merged.
        {"kind": "merge", "name": "merge-4-d64", "parts": 4, "tokens": 178572, "hq": 16, "d": 64},
    ]


def lengths(case):
    """Sample lengths, from the case alone."""
    rng = np.random.Generator(np.random.PCG64(case["lens_seed"]))
    n, lo, hi = case["n"], case["lo"], case["hi"]
    if case["recipe"] == "tiny":
        return np.array([16, 37, 64, 129], dtype=np.int64)
    if case["recipe"] == "one":
        return np.full(n, lo, dtype=np.int64)
    if case["recipe"] == "log":  # log-uniform
        return np.floor(np.exp(rng.uniform(math.log(lo), math.log(hi), size=n))).astype(np.int64)
    if case["recipe"] == "vit":
        return W.lengths_vit(rng, n)
    if case["recipe"] == "long":
        return W.lengths_long_short(rng, long_len=lo, n_short=n)
    return W.lengths_llm_pack(rng, budget=n)


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ones' ranges."""
    most = work(next(c for c in listed() if c["name"] == "long-short-step-d80"))["flops"]
    while True:
        case = _draw(rng)
        if work(case)["flops"] <= most:
            return case


def _draw(rng):
    kind = rng.choice(("tiny", "slice", "slice", "short", "short", "vit", "long", "llm", "llm", "merge"))
    d, seed = rng.choice(DIMS), rng.randrange(1 << 20)
    step, kept = rng.random() < 0.6, rng.random() < 0.5
    if kind == "merge":
        return {"kind": "merge", "parts": rng.choice((2, 3, 4, 6, 8)), "tokens": _log_int(rng, 3000, 150000),
                "hq": rng.choice((2, 4, 8, 16)), "d": d}
    if kind == "tiny":
        g, hkv = rng.choice((1, 1, 2, 4)), rng.choice((1, 2, 4))
        return _attn(None, "log", rng.randint(1, 8), rng.randint(8, 40), rng.randint(60, 300), g * hkv, hkv, d,
                     rng.random() < 0.5, step, rng.random() < 0.5, kept, seed)
    if kind == "slice":
        g, hkv = rng.choice((1, 1, 2, 4)), rng.choice((1, 2, 3))
        size = _log_int(rng, 1000, 20000)
        return _attn(None, "one", 1, size, size, g * hkv, hkv, d, rng.random() < 0.6, step, True, kept, seed)
    if kind == "short":
        lo = _log_int(rng, 20, 200)
        hi = min(1024, lo + _log_int(rng, 50, 900))
        hkv, g = rng.choice((8, 12, 16)), rng.choice((1, 1, 1, 2))
        return _attn(None, "log", _log_int(rng, 40, 120000 // hi), lo, hi, g * hkv, hkv, d, rng.random() < 0.25, step, True,
                     kept, seed)
    if kind == "vit":
        hkv = rng.choice((8, 12, 16))
        return _attn(None, "vit", _log_int(rng, 4, 64), 0, 0, hkv, hkv, d, False, step, True, kept, seed)
    if kind == "long":
        hkv = rng.choice((8, 16))
        return _attn(None, "long", _log_int(rng, 16, 256), _log_int(rng, 6000, 60000), 0, hkv, hkv, d, False, step, True,
                     kept, seed)
    hkv, g = rng.choice((4, 8)), rng.choice((2, 4, 5))
    return _attn(None, "pack", _log_int(rng, 8192, 49152), 0, 0, g * hkv, hkv, rng.choice((96, 128, 128)), True, step, True,
                 kept, seed)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def normal(*shape):
        return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).to(torch.bfloat16)

    hq, d = case["hq"], case["d"]
    if case["kind"] == "merge":
        o = torch.empty((case["parts"], case["tokens"], hq, d), dtype=torch.bfloat16, device="cuda")
        for p in range(case["parts"]):
            o[p] = normal(case["tokens"], hq, d)
        # LSE of a shard of n keys with N(0, 1) scores: ln n + 1/2, give or take
        lse = 6.0 + 0.5 * torch.randn((case["parts"], hq, case["tokens"]), generator=gen, device="cuda")
        return {"case": case, "o_parts": o, "lse_parts": lse}
    lens = lengths(case)
    total, hkv = int(lens.sum()), case["hkv"]
    cu = np.zeros(len(lens) + 1, dtype=np.int32)
    np.cumsum(lens, out=cu[1:])
    s = {"case": case, "scale": 1.0 / math.sqrt(d), "hint": int(lens.max()) if case["hint"] else 0,
         "cu": torch.from_numpy(cu).cuda(), "q": normal(total, hq, d), "k": normal(total, hkv, d), "v": normal(total, hkv, d)}
    fwd, bwd = {}, {}
    if case["kept"]:
        p = binding.make_params(total, len(lens), hq, hkv, d, case["causal"], s["scale"], 0, s["hint"])
        fwd = {"out": torch.empty_like(s["q"]), "lse": torch.empty((hq, total), dtype=torch.float32, device="cuda"),
               "workspace": torch.empty(binding.fwd_workspace_bytes(p), dtype=torch.uint8, device="cuda")}
        if case["step"]:
            bwd = {"dq": torch.empty_like(s["q"]), "dk": torch.empty_like(s["k"]), "dv": torch.empty_like(s["v"]),
                   "workspace": torch.empty(binding.bwd_workspace_bytes(p), dtype=torch.uint8, device="cuda")}
    if case["step"]:
        s["dout"] = normal(total, hq, d)
    s["fwd"], s["bwd"] = fwd, bwd
    return s


def run(s):
    case = s["case"]
    if case["kind"] == "merge":
        return binding.varlen_attn_merge(s["o_parts"], s["lse_parts"])
    o, lse = binding.varlen_attn_fwd(s["q"], s["k"], s["v"], s["cu"], case["causal"], s["scale"], max_seqlen=s["hint"],
                                     **s["fwd"])
    if not case["step"]:
        return o, lse
    dq, dk, dv = binding.varlen_attn_bwd(s["dout"], s["q"], s["k"], s["v"], o, lse, s["cu"], case["causal"], s["scale"],
                                         max_seqlen=s["hint"], **s["bwd"])
    return o, lse, dq, dk, dv


def work(case):
    """Each input read once, each output written once; the matrix products of the definition (forward 2, backward 5)."""
    hq, d = case["hq"], case["d"]
    if case["kind"] == "merge":
        rows = case["tokens"] * hq
        return {"bytes": (case["parts"] + 1) * rows * (2 * d + 4), "flops": (2 * d + 4) * case["parts"] * rows}
    lens = lengths(case).astype(np.float64)
    total, hkv = float(lens.sum()), case["hkv"]
    pairs = float(np.sum(lens * (lens + 1) / 2 if case["causal"] else lens * lens))
    flops = 4.0 * d * hq * pairs
    tensors = 2 * hq + 2 * hkv                                                          # q, o; k, v
    if case["step"]:
        flops *= 3.5
        tensors += 2 * hq + 2 * hkv                                                     # dout, dq; dk, dv
    return {"bytes": 2 * d * total * tensors + 4 * total * hq + 4 * (len(lens) + 1), "flops": flops}


def tolerance(case):
    """bf16 results of bf16 inputs: P and dS are rounded to bf16 before their products and every output once more.
    Measured against the same arithmetic in 64 bits (2-norm of the difference over 2-norm): O 1.6e-3 to 2.3e-3, the
    gradients 1.7e-3 to 2.4e-3, LSE 6e-8; the merge, which only rounds its output, 1.7e-3.  Four times these."""
    return {"rel": 7e-3 if case["kind"] == "merge" else 1e-2}
