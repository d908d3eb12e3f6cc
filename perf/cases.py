"""Timed cases of the library: what a program that uses it calls, over the range of sizes it serves.

Three paths, each through its Python binding and the C ABI behind it:

* ``attention``  fused fault-tolerant attention, ``FtAttn.forward`` on a context the program keeps
                 (or ``forward_static``, the entry point without a context), optionally followed by
                 ``report``;
* ``linear``     the fault-tolerant linear layer, ``FtGemm.forward`` on a context whose weights have
                 been encoded once (or, with ``fold_tokens``, checksums over the token rows, encoded
                 inside every call);
* ``decoupled``  the three-kernel scheme with S and P in device memory, ``FtDecoupled.forward``.

All of them are forward passes: the library has no backward direction.  Values follow the
recipes of ``synth.py``: standard-normal operands (weights N(0, 1/k)), 1 % of the key rows eight
times larger where ``outliers`` is set.
"""
import math

import torch

from paper_2504_02211_amd import ftattn, ftdecoupled, ftgemm

DTYPES = {"fp16": (0, torch.float16), "bf16": (1, torch.bfloat16), "fp32": (2, torch.float32)}
MODES = {"off": ftattn.FT_OFF, "correct": ftattn.FT_CORRECT, "detect": ftattn.FT_DETECT}


def _attention(batch, heads, seq, head_dim, dtype, causal, out="fp32", mode="correct", rowsum_fold=False,
               outliers=False, static=False, report=False):
    return {"path": "attention", "batch": batch, "heads": heads, "seq": seq, "head_dim": head_dim, "dtype": dtype,
            "causal": causal, "out": out, "mode": mode, "rowsum_fold": rowsum_fold, "outliers": outliers,
            "static": static, "report": report}


def _linear(m, n, k, dtype, out, mode="correct", fold_tokens=False, report=False):
    return {"path": "linear", "m": m, "n": n, "k": k, "dtype": dtype, "out": out, "mode": mode,
            "fold_tokens": fold_tokens, "report": report}


def _decoupled(batch, heads, seq, head_dim, dtype, causal, mode="correct"):
    return {"path": "decoupled", "batch": batch, "heads": heads, "seq": seq, "head_dim": head_dim, "dtype": dtype,
            "causal": causal, "mode": mode}


def listed():
    named = {
        # the smallest attention of the benchmark (one head of 128 tokens), through the entry point made for tight serving loops
        "attn_tiny_static": _attention(1, 1, 128, 64, "fp16", False, static=True),
        # a short ragged prompt whose report the program reads after every pass
        "attn_ragged_report": _attention(2, 3, 333, 128, "fp16", True, out="fp16", report=True),
        # encoder layer over a batch of short sequences
        "attn_encoder": _attention(16, 12, 512, 64, "fp16", False),
        # decoder layer, head size 64
        "attn_decoder_causal": _attention(8, 16, 2048, 64, "bf16", True),
        # large heads with outlier keys
        "attn_large_head_causal": _attention(4, 32, 4096, 128, "bf16", True, outliers=True),
        # one long sequence: the headline workload
        "attn_long_causal": _attention(1, 32, 16384, 128, "bf16", True),
        # a few sequences of odd length attending in both directions, result in the input type, exact row-sum check
        "attn_odd_length_fold": _attention(3, 16, 1531, 128, "fp16", False, out="fp16", rowsum_fold=True),
        # the same kernel with its checks off: what a program runs where it does not need them
        "attn_unprotected": _attention(4, 16, 3000, 64, "bf16", True, out="bf16", mode="off"),
        # feed-forward up-projection of a 16K-token batch
        "linear_ffn": _linear(16384, 16384, 4096, "fp16", "fp16"),
        # projection of a handful of tokens (a decoding step)
        "linear_few_tokens": _linear(37, 1000, 1024, "bf16", "fp32"),
        # projection of a medium batch with checksums over the tokens
        "linear_fold_tokens": _linear(2048, 2048, 1024, "bf16", "bf16", fold_tokens=True),
        # the scheme with S and P in memory, at a size whose scores still fit comfortably
        "decoupled_causal": _decoupled(2, 16, 2048, 128, "bf16", True),
    }
    return [dict(case, name=name) for name, case in named.items()]


def _log(rng, lo, hi):
    """A whole number between lo and hi, spread over its logarithm: any value, odd ones among them."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


FLOPS_MAX = 2.1e12          # just below the longest listed pass


def draw(rng):
    """One more case of the same ranges."""
    while True:
        path = rng.choice(["attention"] * 5 + ["linear"] * 3 + ["decoupled"] * 2)
        dtype = rng.choice(["fp16", "bf16"])
        if path == "attention":
            c = _attention(_log(rng, 1, 16), _log(rng, 1, 32), _log(rng, 16, 16384), rng.choice([64, 128]), dtype,
                           rng.random() < 0.6, out=rng.choice(["fp32", dtype]),
                           mode=rng.choice(["correct"] * 4 + ["detect", "off"]))
            rows = c["batch"] * c["heads"] * c["seq"]
            c["rowsum_fold"] = c["mode"] != "off" and rng.random() < 0.2
            c["outliers"] = rng.random() < 0.2
            c["report"] = rng.random() < 0.2
            # the static entry point holds the encoded tiles in 64 MiB
            c["static"] = not c["report"] and rows * c["head_dim"] < 4e6 and rng.random() < 0.3
            if rows <= 32 * 16384:
                if work(c)["flops"] <= FLOPS_MAX * (1.0 if c["head_dim"] == 128 else 0.4):
                    return c
        elif path == "linear":
            c = _linear(_log(rng, 1, 16384), _log(rng, 64, 16384), 8 * _log(rng, 8, 1024), dtype, rng.choice(["fp32", dtype]),
                        mode=rng.choice(["correct"] * 4 + ["detect", "off"]), fold_tokens=rng.random() < 0.25)
            c["report"] = rng.random() < 0.2
            if work(c)["flops"] <= FLOPS_MAX:
                return c
        else:
            c = _decoupled(_log(rng, 1, 4), _log(rng, 1, 16), _log(rng, 64, 4096), rng.choice([64, 128]), dtype, rng.random() < 0.6,
                           mode=rng.choice(["correct"] * 4 + ["off"]))
            if c["batch"] * c["heads"] * c["seq"] ** 2 <= 2 * 16 * 2048 ** 2:
                return c


def _normal(seed, which, shape, dtype, scale=1.0):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 16 + which)
    x = torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)
    return x.mul_(scale).to(DTYPES[dtype][1])


def prepare(case, seed):
    path, code = case["path"], DTYPES[case["dtype"]][0]
    if path == "linear":
        m, n, k = case["m"], case["n"], case["k"]
        out_code, out_type = DTYPES[case["out"]]
        s = {"case": case, "x": _normal(seed, 0, (m, k), case["dtype"]),
             "w": _normal(seed, 1, (n, k), case["dtype"], 1.0 / math.sqrt(k)),
             "y": torch.empty((m, n), dtype=out_type, device="cuda"),
             "ctx": ftgemm.FtGemm(m, n, k, out_dtype=out_code, ft_mode=MODES[case["mode"]], in_dtype=code,
                                  fold_tokens=case["fold_tokens"])}
        s["ctx"].encode_weights(s["w"], torch.cuda.current_stream().cuda_stream)
        return s
    shape = (case["batch"], case["heads"], case["seq"], case["head_dim"])
    s = {"case": case}
    for i, name in enumerate("qkv"):
        s[name] = _normal(seed, i, shape, case["dtype"])
    if case.get("outliers"):
        g = torch.Generator(device="cuda")
        g.manual_seed(seed * 16 + 3)
        big = torch.rand(shape[:3], generator=g, device="cuda") < 0.01
        s["k"] *= torch.where(big, 8.0, 1.0).unsqueeze(-1).to(s["k"].dtype)
    out_code, out_type = DTYPES[case.get("out", "fp32")]
    s["o"] = torch.empty(shape, dtype=out_type, device="cuda")
    if path == "decoupled":
        s["ctx"] = ftdecoupled.FtDecoupled(*shape, code, case["causal"], ft_mode=MODES[case["mode"]])
    elif case["static"]:
        s["n_events"] = torch.zeros(1, dtype=torch.int32, device="cuda")
    else:
        s["ctx"] = ftattn.FtAttn(*shape, code, case["causal"], out_dtype=out_code, ft_mode=MODES[case["mode"]],
                                 rowsum_fold=case["rowsum_fold"])
    return s


def run(s):
    case = s["case"]
    stream = torch.cuda.current_stream().cuda_stream
    if case["path"] == "linear":
        s["ctx"].forward(s["x"], s["w"], s["y"], None, stream)
        if not case["report"]:
            return s["y"]
        rep = s["ctx"].report()
        return {"y": s["y"], "events": rep.n_events, "dropped": rep.n_events_dropped}
    if case["path"] == "decoupled":
        s["ctx"].forward(s["q"], s["k"], s["v"], s["o"], None, stream)
        return s["o"]
    if case["static"]:
        code, out_code = DTYPES[case["dtype"]][0], DTYPES[case["out"]][0]
        ftattn.forward_static(s["q"], s["k"], s["v"], s["o"], case["batch"], case["heads"], case["seq"], case["head_dim"],
                              code, case["causal"], out_dtype=out_code, ft_mode=MODES[case["mode"]],
                              n_events=s["n_events"], stream=stream, rowsum_fold=case["rowsum_fold"])
        return {"o": s["o"], "events": s["n_events"]}
    s["ctx"].forward(s["q"], s["k"], s["v"], s["o"], None, stream)
    if not case["report"]:
        return s["o"]
    rep = s["ctx"].report()
    return {"o": s["o"], "events": rep.n_events, "dropped": rep.n_events_dropped, "range_flags": rep.range_flags,
            "tile_flags": rep.tile_flags, "rowtile_flags": rep.rowtile_flags}


def work(case):
    """Operands once, result once; the products' multiplications and additions without checksums."""
    size = {"fp16": 2, "bf16": 2, "fp32": 4}
    if case["path"] == "linear":
        m, n, k = case["m"], case["n"], case["k"]
        return {"bytes": (m * k + n * k) * 2 + m * n * size[case["out"]], "flops": 2.0 * m * n * k}
    heads, n, d = case["batch"] * case["heads"], case["seq"], case["head_dim"]
    scores = n * (n + 1) // 2 if case["causal"] else n * n
    return {"bytes": heads * n * d * (3 * 2 + size[case.get("out", "fp32")]), "flops": 4.0 * heads * scores * d}


def tolerance(case):
    """About four times the distance from the same pass in 64 bits: what rounding the result to its type
    gives (2-norm 2.1e-4 in fp16, 1.7e-3 in bf16), on top of the fp16 weights P of an attention (up to 2.1e-4)
    or the fp32 accumulation of a linear layer (up to 5e-7 at 5464 terms, growing with their root).
    Counts and flags of a report are whole numbers and stay as they are."""
    out = case.get("out", "fp32")
    if case["path"] == "linear":
        return {"rel": {"fp32": 4e-6, "fp16": 8.5e-4, "bf16": 7e-3}[out]}
    return {"rel": {"fp32": 8.5e-4, "fp16": 1.2e-3, "bf16": 7e-3}[out]}
