"""Workloads of the attention library for timing: what a program that uses it calls, over the range it is used on.

`listed()` holds the fixed cases, `draw()` gives more of the same ranges; `prepare()` makes what the caller has in
hand before the call (tensors on the GPU, and for decoding the workspace that a serving loop keeps), `run()` is one
call through the public Python entry points.  Shapes are the repository's own workloads (the five prefill
configurations, their FP8 and D = 256 forms and the two decode workloads of bench.py) and generic ones beside them.
"""
import math

import torch

from paper_2604_14825_amd import binding as nb
from paper_2604_14825_amd import synth

DTYPES = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}
FP8_DESCALE = (1.0 / 64, 1.0 / 8, 1.0 / 64)  # per-tensor scales of q, k, v, as in bench.py
OUTLIER_SCALE = 8.0                          # 1 % of the K rows are scaled by this where `outliers` is set
MOST_FLOPS = 4.0 * 32 * 256 * 16384 * 16385 / 2  # of the largest listed case
MOST_BYTES = 1 << 30                             # of a drawn decode case: twice the listed cache


def _prefill(name, B, Hq, Hkv, S, D, causal, dtype="bf16", out="bf16", seq_major=False, outliers=False):
    return {"name": name, "path": "prefill", "B": B, "Hq": Hq, "Hkv": Hkv, "S": S, "D": D, "causal": causal,
            "dtype": dtype, "out": out, "seq_major": seq_major, "outliers": outliers}


def _decode(name, B, Hq, Hkv, Sq, Sk, D, dtype="bf16", out="bf16", seq_major=False, outliers=False):
    return {"name": name, "path": "decode", "B": B, "Hq": Hq, "Hkv": Hkv, "Sq": Sq, "Sk": Sk, "D": D, "causal": True,
            "dtype": dtype, "out": out, "seq_major": seq_major, "outliers": outliers}


def _of(name):
    w = synth.WORKLOADS[name]
    kind = {synth.BF16: "bf16", synth.F16: "f16", synth.F32: "f32"}
    return _prefill(name, w.B, w.Hq, w.Hkv, w.S, w.D, w.causal, kind[w.in_dtype], kind[w.out_dtype],
                    outliers=w.outlier_frac > 0)


def listed():
    return [
        _of("tiny"),       # the smallest call: one short sequence, two heads, fp32 output; latency and launch
        # one request's prompt in a serving engine: grouped-query heads, an odd length, sequence-major tensors
        _prefill("prompt", 1, 32, 8, 1003, 128, True, seq_major=True),
        _of("encoder"),    # a batch through a vision or text encoder: short sequences, D = 64, no mask
        # an encoder with a head size that no kernel is compiled for and a ragged length, sequence-major
        _prefill("ragged_d80", 4, 16, 16, 1777, 80, False, "f16", "f16", seq_major=True),
        _of("prefill"),    # a batch of prompts
        _of("gqa"),        # long prompts, grouped-query heads
        _of("long"),       # one very long prompt, some keys much larger than the rest
        _of("long_d256"),  # the same at the widest head
        dict(_of("long"), name="long_fp8", dtype="fp8"),  # and with FP8 tensors
        # generation: a lone request, the latency of one step
        _decode("decode_one", 1, 32, 8, 1, 4099, 128),
        # a full batch against 16k caches, in bf16 and FP8
        _decode("decode", 8, 32, 8, 1, 16384, 128, outliers=True),
        _decode("decode_fp8", 8, 32, 8, 1, 16384, 128, dtype="fp8", outliers=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    fp8 = rng.random() < 0.25
    dtype = "fp8" if fp8 else rng.choice(["bf16", "bf16", "bf16", "f16"])
    out = "bf16" if fp8 else rng.choice([dtype, dtype, dtype, "f32"])
    group = rng.choice([1, 1, 4, 8])
    Hkv = rng.choice([1, 2, 4, 8]) if group > 1 else rng.choice([4, 8, 12, 16, 32])
    Hq = Hkv * group
    D = rng.choice([64, 128, 128, 80, 96] if fp8 else [64, 64, 128, 128, 128, 72, 80, 96, 192, 256])
    seq_major = rng.random() < 0.5
    outliers = rng.random() < 0.25
    if rng.random() < 0.6:
        causal = rng.random() < 0.6
        B, S = _log(rng, 1, 8), _log(rng, 128, 16384)
        if rng.random() < 0.5:  # padded to a round length as often as not
            S = max(128, S // 128 * 128)
        case = _prefill("", B, Hq, Hkv, S, D, causal, dtype, out, seq_major, outliers)
        while work(case)["flops"] > MOST_FLOPS:
            S //= 2
            case["S"] = S
    else:
        # one new position for generation, a few for speculative decoding
        Sq, B, Sk = rng.choice([1, 1, 1, 2, 4, 8]), _log(rng, 1, 64), _log(rng, 256, 131072)
        case = _decode("", B, Hq, Hkv, Sq, Sk, D, dtype, out, seq_major, outliers)
        while work(case)["bytes"] > MOST_BYTES:
            Sk //= 2
            case["Sk"] = Sk
    del case["name"]
    return case


def _values(gen, B, H, S, c, descale, outliers=False):
    """N(0,1) values in the storage type, [B,H,S,D], the memory in that order or sequence-major."""
    D = c["D"]
    x = torch.randn((B, S, H, D) if c["seq_major"] else (B, H, S, D), generator=gen, device="cuda", dtype=torch.float32)
    n = S // 100
    if outliers and n:
        rows = torch.randperm(S, generator=gen, device="cuda")[:n]
        factor = torch.ones(S, device="cuda")
        factor[rows] = OUTLIER_SCALE
        x *= factor.view(1, S, 1, 1) if c["seq_major"] else factor.view(1, 1, S, 1)
    if c["dtype"] == "fp8":
        x = (x / descale).clamp_(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8)
    else:
        x = x.to(DTYPES[c["dtype"]])
    return x.transpose(1, 2) if c["seq_major"] else x


def prepare(case, seed):
    c = dict(case)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed) + 2604)
    decode = c["path"] == "decode"
    Sq, Sk = (c["Sq"], c["Sk"]) if decode else (c["S"], c["S"])
    B, Hq, Hkv, D = c["B"], c["Hq"], c["Hkv"], c["D"]
    c["q"] = _values(gen, B, Hq, Sq, c, FP8_DESCALE[0])
    c["k"] = _values(gen, B, Hkv, Sk, c, FP8_DESCALE[1], c["outliers"])
    c["v"] = _values(gen, B, Hkv, Sk, c, FP8_DESCALE[2])
    o = torch.empty((B, Sq, Hq, D) if c["seq_major"] else (B, Hq, Sq, D), device="cuda", dtype=DTYPES[c["out"]])
    c["o"] = o.transpose(1, 2) if c["seq_major"] else o
    c["lse"] = torch.empty((B, Hq, Sq), device="cuda", dtype=torch.float32)
    c["scale"] = 1.0 / math.sqrt(D)
    if decode:
        c["ws"] = torch.empty(nb.decode_workspace_bytes(B, Hq, Hkv, Sq, Sk, D), device="cuda", dtype=torch.uint8)
    # The plain entry points take contiguous tensors of the compiled head sizes, the strided ones the rest.
    compiled = (64, 128) if decode or c["dtype"] == "fp8" else (64, 128, 256)
    c["strided"] = c["seq_major"] or D not in compiled
    return c


def run(state):
    c = state
    q, k, v, o, lse, causal, scale = c["q"], c["k"], c["v"], c["o"], c["lse"], c["causal"], c["scale"]
    if c["path"] == "decode":
        if c["dtype"] == "fp8":
            f = nb.naut_attn_decode_fp8_strided if c["strided"] else nb.naut_attn_decode_fp8
            f(q, k, v, o, lse, causal, scale, *FP8_DESCALE, c["ws"])
        else:
            f = nb.naut_attn_decode_strided if c["strided"] else nb.naut_attn_decode
            f(q, k, v, o, lse, causal, scale, c["ws"])
    elif c["dtype"] == "fp8":
        f = nb.naut_attn_fwd_fp8_strided if c["strided"] else nb.naut_attn_fwd_fp8
        f(q, k, v, o, lse, causal, scale, *FP8_DESCALE)
    else:
        f = nb.naut_attn_fwd_strided if c["strided"] else nb.naut_attn_fwd
        f(q, k, v, o, lse, causal, scale)
    return {"o": o, "lse": lse}


def work(case):
    c = case
    Sq, Sk = (c["Sq"], c["Sk"]) if c["path"] == "decode" else (c["S"], c["S"])
    size = {"fp8": 1, "bf16": 2, "f16": 2, "f32": 4}
    n_q, n_kv = c["B"] * c["Hq"] * Sq * c["D"], c["B"] * c["Hkv"] * Sk * c["D"]
    pairs = Sq * Sk - (Sq * (Sq - 1) // 2 if c["causal"] else 0)  # (query, key) pairs that the mask leaves
    return {"bytes": (n_q + 2 * n_kv) * size[c["dtype"]] + n_q * size[c["out"]] + c["B"] * c["Hq"] * Sq * 4,
            "flops": 4.0 * c["B"] * c["Hq"] * c["D"] * pairs}


def tolerance(case):
    """About four times the error measured against 64-bit attention on these cases (2-norm of O, and the largest
    error over max(rms, |value|)): bf16 2.3e-3 and 4.0e-2, f16 3.0e-4 and 1.4e-3, FP8 2.7e-2 and 0.22 (P rounded to
    E4M3, half a unit in the last place being 2^-4; kept to 3e-2).  The fp32 lse is far inside (7e-8 to 6e-6)."""
    if case["dtype"] == "fp8":
        return {"rel": 3e-2, "max": 0.9}
    if case["dtype"] == "f16":
        return {"rel": 1.2e-3, "max": 6e-3}
    return {"rel": 1e-2, "max": 0.16}
