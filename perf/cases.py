"""The work a user of this library has it do, as a list of measurable cases.

Four entry points carry everything the library does: ``attn_fwd`` (fp16 / bf16, head dimension 64 or 128,
causal or not), ``attn_fwd_fp8`` (E4M3 inputs, 16-bit output), ``gemm_nt`` (fp16 / bf16) and ``gemm_nt_fp8``
(E4M3 operands, 16-bit result).  ``listed()`` holds the shapes of the benchmark configurations, of the
sweeps over sequence length and over K, and of the ragged shapes the tests use; ``draw`` takes more cases from the
ranges they stand for:

    attention   B 1 ... 16, H 1 ... 32, N 64 ... 16384, d in {64, 128}, causal or not, every element type
    products    M, N 16 ... 8192, K 64 ... 16384 in steps of 32 (16-bit) or 64 (E4M3), every element type

A user's program holds the operands and the output buffers on the device and calls the binding; the library
has no plan or handle object, so ``prepare`` makes tensors only and ``run`` is one call.
"""
from __future__ import annotations

import math

import torch

from paper_2510_14719_amd import binding

TORCH_TYPE = {"fp16": torch.float16, "bf16": torch.bfloat16, "e4m3": torch.float8_e4m3fn}
BYTES = {"fp16": 2, "bf16": 2, "e4m3": 1}


def _attn(name, B, H, N, d, dtype, causal, out="fp16", peaky=False):
    return {"name": name, "op": "attn", "B": B, "H": H, "N": N, "d": d, "dtype": dtype, "causal": causal,
            "out": out if dtype == "e4m3" else dtype, "peaky": peaky}


def _gemm(name, M, N, K, dtype, out="fp16"):
    return {"name": name, "op": "gemm", "M": M, "N": N, "K": K, "dtype": dtype, "out": out if dtype == "e4m3" else dtype}


def listed():
    return [
        # The smallest benchmark configuration: two heads of 128 tokens.  Launch and latency, as in the first
        # steps of a prompt or a unit test of a model.
        _attn("attn_smallest", 1, 2, 128, 64, "fp16", False),
        # Head dimension 64 at sequence length 1024: an encoder's batch, and the same batch in a decoder's prefill.
        _attn("attn_d64_full", 16, 16, 1024, 64, "fp16", False),
        _attn("attn_d64_causal", 16, 16, 1024, 64, "fp16", True),
        # A single prompt of a length that is a multiple of nothing, few heads: the chip is not full.
        _attn("attn_ragged_causal", 1, 8, 2309, 128, "bf16", True),
        # Long-context prefill with the mask, keys with a few dominant rows (softmax rows close to one-hot).
        _attn("attn_long_causal", 2, 32, 8192, 128, "bf16", True, peaky=True),
        # The headline configuration: the longest sequence of the sweep, no mask.
        _attn("attn_longest", 1, 16, 16384, 128, "fp16", False),
        # 8-bit attention: the short causal end of the sweep (batch 4) and its middle without the mask.
        _attn("attn_fp8_short_causal", 4, 16, 1024, 128, "e4m3", True, out="bf16"),
        _attn("attn_fp8_full", 4, 16, 4096, 128, "e4m3", False),
        # Matrix products: a small ragged one (a layer on a few hundred tokens), the short-K end of the paper's
        # sweep (the result dominates the traffic), and a large square one.
        _gemm("gemm_small_ragged", 1000, 777, 512, "fp16"),
        _gemm("gemm_short_k", 8192, 8192, 256, "bf16"),
        _gemm("gemm_large", 8192, 8192, 8192, "fp16"),
        # The long-K end of the sweep on 8-bit operands.
        _gemm("gemm_fp8_long_k", 8192, 8192, 16384, "e4m3"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


MAX_FLOPS = 1.1e12      # half of the largest listed case: a drawn shape may sit in a less efficient corner


def draw(rng):
    """One more case of the ranges above; sizes are spread over their logarithm, most of them odd."""
    kind = rng.choice(("attn16", "attn16", "attn8", "gemm16", "gemm8"))
    if kind.startswith("attn"):
        dtype = rng.choice(("fp16", "bf16")) if kind == "attn16" else "e4m3"
        N, H, d = _log_int(rng, 64, 16384), _log_int(rng, 1, 32), rng.choice((64, 128))
        if rng.random() < 0.3:
            N = max(64, N // 64 * 64)           # lengths are often padded to a multiple of 64
        cap = max(1, int(MAX_FLOPS / (4.0 * H * N * N * d)))
        B = min(_log_int(rng, 1, 16), cap)
        while 4.0 * B * H * float(N) * N * d > MAX_FLOPS and H > 1:
            H //= 2
        return _attn("", B, H, N, d, dtype, rng.random() < 0.5, out=rng.choice(("fp16", "bf16")), peaky=rng.random() < 0.2)
    dtype = rng.choice(("fp16", "bf16")) if kind == "gemm16" else "e4m3"
    step = 64 if dtype == "e4m3" else 32
    M, N, K = _log_int(rng, 16, 8192), _log_int(rng, 16, 8192), max(64, _log_int(rng, 64, 16384) // step * step)
    if rng.random() < 0.3:
        M, N = max(16, M // 16 * 16), max(16, N // 16 * 16)
    while 2.0 * M * N * K > MAX_FLOPS:
        K = max(64, K // 2 // step * step)
    return _gemm("", M, N, K, dtype, out=rng.choice(("fp16", "bf16")))


def _normal(shape, dtype, gen, rows_scaled=None):
    x = torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32)
    if rows_scaled is not None:
        x.mul_(rows_scaled)
    return x.to(TORCH_TYPE[dtype])


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    if case["op"] == "attn":
        B, H, N, d, dtype = case["B"], case["H"], case["N"], case["d"], case["dtype"]
        scaled = None
        if case["peaky"]:                       # about 5 % of the key rows are eight times as long
            scaled = torch.where(torch.rand((B, H, N, 1), generator=gen, device="cuda") < 0.05, 8.0, 1.0)
        q = _normal((B, H, N, d), dtype, gen)
        k = _normal((B, H, N, d), dtype, gen, scaled)
        v = _normal((B, H, N, d), dtype, gen)
        o = torch.empty((B, H, N, d), dtype=TORCH_TYPE[case["out"]], device="cuda")
        lse = torch.empty((B, H, N), dtype=torch.float32, device="cuda")
        call = binding.attn_fwd_fp8 if dtype == "e4m3" else binding.attn_fwd
        return {"op": "attn", "call": call, "args": (q, k, v, o, lse, B, H, N, d, 1.0 / math.sqrt(d), case["causal"])}
    M, N, K = case["M"], case["N"], case["K"]
    a, b = _normal((M, K), case["dtype"], gen), _normal((N, K), case["dtype"], gen)
    c = torch.empty((M, N), dtype=TORCH_TYPE[case["out"]], device="cuda")
    if case["dtype"] == "e4m3":
        out_dtype = binding.BF16 if case["out"] == "bf16" else binding.FP16
        return {"op": "gemm", "call": binding.gemm_nt_fp8, "args": (a, b, c, M, N, K), "kwargs": {"out_dtype": out_dtype}}
    return {"op": "gemm", "call": binding.gemm_nt, "args": (a, b, c, M, N, K)}


def run(state):
    state["call"](*state["args"], **state.get("kwargs", {}))
    return state["args"][3:5] if state["op"] == "attn" else state["args"][2]


def work(case):
    if case["op"] == "attn":
        rows, d = case["B"] * case["H"] * case["N"], case["d"]
        pairs = case["B"] * case["H"] * case["N"] * ((case["N"] + 1) / 2 if case["causal"] else case["N"])
        return {"bytes": rows * d * (3 * BYTES[case["dtype"]] + 2) + 4 * rows, "flops": 4.0 * pairs * d}
    M, N, K = case["M"], case["N"], case["K"]
    return {"bytes": (M + N) * K * BYTES[case["dtype"]] + 2 * M * N, "flops": 2.0 * M * N * K}


# Relative 2-norm error of an output against the same computation in 64 bits, times about four.  Measured on the MI355X
# over the listed cases and thirty drawn ones, worst of each kind: attention fp16 2.9e-4, bf16 2.1e-3 (the rounding of
# the result and of the probabilities), attention on E4M3 2.7e-2 (its probabilities are rounded to 3 fraction bits and
# V has zero mean, so the result shows that in full), products fp16 2.1e-4, bf16 1.7e-3 (the rounding of the result).
TOLERANCE = {("attn", "fp16"): 1.2e-3, ("attn", "bf16"): 8.5e-3, ("attn", "e4m3"): 1.1e-1,
             ("gemm", "fp16"): 8.5e-4, ("gemm", "bf16"): 6.8e-3}


def tolerance(case):
    key = case["dtype"] if case["op"] == "attn" else case["out"]
    return {"rel": TOLERANCE[(case["op"], key)]}
