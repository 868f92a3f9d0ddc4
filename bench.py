#!/usr/bin/env python3
"""Benchmark of the attention forward hot path on one MI355X.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload c4] [--no-cpu-baseline]

One "step" is one pass of the whole hot path (tile walk, K/V staging, QK^T,
masking, streaming softmax, PV, epilogue: a single kernel launch) over one batch
of the synthetic workload.  The default workload is the headline configuration
the metric is quoted on: B=1, H=16, N=16384, d=128, fp16, non-causal.  Inputs are
resident in HBM before the timed region.

Prints ONE JSON line: attention-forward TFLOP/s (4*B*H*N^2*d flops, halved when
causal), the MFMA roofline of the kernel from per-launch HIP-event durations, and
the CPU oracle timed on a bounded sample of the same workload on the host cores.
"""
from __future__ import annotations

import argparse
import json
import math
import os
import statistics
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

PEAK_TFLOPS = {0: 2500.0, 1: 2500.0, 2: 5000.0}   # MI355X dense MFMA peak: fp16, bf16, fp8
GEMM_SHAPES = ((256, 256), (64, 64), (128, 128), (128, 128))   # rows and columns of C per workgroup of gemm_nt_shape's kernels
DTYPE_NAME = {0: "fp16", 1: "bf16", 2: "fp8-e4m3"}

# HBM bytes per launch measured with rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE (two runs, each scaled by what the
# counter reads for a 1 GiB copy): a profile's figure, not measured by this script.  Every summary under
# profiles/ that holds such a measurement carries one line "TRAFFIC_BYTES_PER_LAUNCH = <bytes>".
PROFILE_OF = {"c4": "profiles/attn_fwd_c4_fp16_noncausal.md", "c3": "profiles/attn_fwd_c3_bf16_noncausal.md", "c5": "profiles/attn_fwd_c5_bf16_causal.md",
              "c2": "profiles/attn_fwd_c2_fp16_d64_noncausal.md", "c2_causal": "profiles/attn_fwd_c2_fp16_d64_causal.md",
              "f4": "profiles/attn_fwd_fp8_f4_e4m3_noncausal.md",
              ("gemm", 256): "profiles/gemm_nt_m8192_n8192_k256_fp16.md",
              ("gemm", 16384): "profiles/gemm_nt_m8192_n8192_k16384_fp16.md",
              ("gemm_fp8", 16384): "profiles/gemm_nt_fp8_m8192_n8192_k16384_e4m3.md"}


def measured_traffic(key):
    """(bytes per launch, profile path) from the committed profile summary of this workload, or (None, None)."""
    import re
    rel = PROFILE_OF.get(key)
    if rel is None or not os.path.exists(os.path.join(ROOT, rel)):
        return None, None
    m = re.search(r"TRAFFIC_BYTES_PER_LAUNCH\s*=\s*([0-9.eE+]+)", open(os.path.join(ROOT, rel)).read())
    return (float(m.group(1)), rel) if m else (None, None)


def describe(w) -> str:
    return "%s: B=%d H=%d N=%d d=%d %s %s%s" % (
        w.name, w.B, w.H, w.N, w.d, DTYPE_NAME[w.dtype],
        "causal" if w.causal else "non-causal", " peaky-K" if w.peaky else "")


# The tolerances for N(0,1) inputs (O max-abs, O mean-abs, LSE max-abs); the 8-bit-float workloads
# of these shapes stay inside them as well, but for the mean of the short ones (see tolerances()).
TOL = {"o_max_abs": 2e-2, "o_mean_abs": 2e-3, "lse_max_abs": 1e-2}


def tolerances(w, fp8):
    """TOL, with E4M3 probabilities also the mean error that their rounding gives: relative to its weight p_j each has an
    error of at most 2^-4, an rms below 2^-4 / sqrt(3), independent of the others; O is off by sum_j p_j e_j (v_j - O), and with
    N(0,1) scores and values sum_j p_j^2 is e / N on the average: rms 2^-4 sqrt(e / 3 N), mean magnitude sqrt(2 / pi) of that."""
    if not fp8:
        return TOL
    return dict(TOL, o_mean_abs=max(TOL["o_mean_abs"], (2.0 / math.pi) ** 0.5 * 2.0 ** -4 * (math.e / (3.0 * w.N)) ** 0.5))


def cpu_baseline(w, qn, kn, vn, budget_heads: int = 2):
    """The oracle as it stands, timed on whole heads of the workload's own tensors (a bounded sample: the first
    heads and the last one).  Returns (record, head list, O reference, LSE reference)."""
    import numpy as np
    from oracle import attn_ref
    attn_ref.build()
    total = w.B * w.H
    heads = min(budget_heads, total)
    # c2-sized heads are cheap: take enough of them for a stable number, capped near 10-30 s of work
    per_head = 4.0 * w.N * w.N * w.d / (2 if w.causal else 1)
    while heads < total and heads * per_head < 1.0e12:
        heads += 1
    sel = list(range(heads - 1)) + [total - 1] if heads > 1 else [0]
    sel = sorted(set(sel))
    qs, ks, vs = (np.ascontiguousarray(x.reshape(total, w.N, w.d)[sel][None]) for x in (qn, kn, vn))
    t0 = time.perf_counter()
    o_ref, l_ref = attn_ref.attn_ref(qs, ks, vs, w.dtype, w.scale, w.causal)
    dt = time.perf_counter() - t0
    rec = {"value": len(sel) * per_head / dt * 1e-12, "unit": "TFLOP/s", "cores": attn_ref.max_threads(),
           "kind": "oracle", "seconds": dt,
           "sample": "%d of %d heads of %s (all N=%d query rows of each; the first ones and the last), fp64" % (len(sel), total, w.name, w.N)}
    return rec, sel, o_ref[0], l_ref[0]


def all_configs(binding, torch, I, stream) -> dict:
    """ms / TFLOP/s / fraction of the dense MFMA peak of every benchmark configuration (c1 ... c5, c2 also with
    the causal mask), a few launches each; the same entry point and launch configuration as the headline line."""
    res = {}
    for name in ("c1", "c2", "c2_causal", "c3", "c4", "c5"):
        w = I.WORKLOADS[name]
        q, k, v = (torch.from_numpy(x.view("int16")).cuda() for x in I.make_workload(w))
        o = torch.empty_like(q)
        lse = torch.empty((w.B, w.H, w.N), dtype=torch.float32, device="cuda")
        warm, steps = (30, 100) if w.flops < 1e11 else (15, 30)
        for _ in range(warm):
            binding.attn_fwd(q, k, v, o, lse, w.B, w.H, w.N, w.d, w.scale, w.causal, stream=stream, dtype=w.dtype)
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record(stream)
        for _ in range(steps):
            binding.attn_fwd(q, k, v, o, lse, w.B, w.H, w.N, w.d, w.scale, w.causal, stream=stream, dtype=w.dtype)
        e1.record(stream)
        torch.cuda.synchronize()
        ms = e0.elapsed_time(e1) / steps
        tf = w.flops / (ms * 1e-3) * 1e-12
        res[name] = {"workload": describe(w), "steps": steps, "ms_per_step": ms, "tflops": tf, "frac_of_mfma_peak": tf / PEAK_TFLOPS[w.dtype]}
        del q, k, v, o, lse
    return res


def mfma_sustained(binding, torch, dtype: int, stream, launches: int = 150, warm: int = 60) -> dict:
    """Register-only MFMA stream of the library's probe: what the matrix cores sustain on this GPU
    with zero operands (nothing toggles) and with pseudo-random operands (toggling of real data)."""
    wgs = torch.cuda.get_device_properties(0).multi_processor_count
    sink = torch.empty(binding.load_library().attn_fwd_mfma_probe_sink_floats(wgs), dtype=torch.float32, device="cuda")
    iters = 4000    # about as long as one attention launch of the headline workload
    out = {"workgroups": wgs, "mfmas_per_wave": iters * 8, "launches": launches}
    for name, rnd in (("zero_operands", False), ("random_operands", True)):
        for _ in range(warm):
            binding.mfma_probe(sink, wgs, iters, rnd, dtype, stream)
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record(stream)
        for _ in range(launches):
            flops = binding.mfma_probe(sink, wgs, iters, rnd, dtype, stream)
        e1.record(stream)
        torch.cuda.synchronize()
        out[name] = flops * launches / (e0.elapsed_time(e1) * 1e-3) * 1e-12
    return out


def gemm_cpu_baseline(M, N, K, dtype, seed, rows: int = 24) -> dict:
    """The matrix-product oracle as it stands, timed on a few whole rows of C of the same workload."""
    from oracle import gemm_ref
    from paper_2510_14719_amd import inputs as I
    gemm_ref.build()
    rows = min(rows, M)
    a, b = I.make_ab(rows, N, K, dtype, seed)
    t0 = time.perf_counter()
    gemm_ref.gemm_nt(a, b, dtype)
    dt = time.perf_counter() - t0
    return {"value": 2.0 * rows * N * K / dt * 1e-12, "unit": "TFLOP/s", "cores": gemm_ref.max_threads(), "kind": "oracle",
            "seconds": dt, "sample": "%d of %d rows of C (all N=%d columns, K=%d), fp64" % (rows, M, N, K)}


def main_gemm(args) -> int:
    """`--op gemm` / `--op gemm_fp8`: the paper's matrix-multiplication workload, M = N = 8192, one K of
    its sweep, on fp16 operands or on 8-bit-float (E4M3) operands with an fp16 result."""
    import numpy as np
    import torch
    from paper_2510_14719_amd import binding, inputs as I
    if not torch.cuda.is_available():
        print("bench.py: no GPU visible; the HIP path has no CPU fallback", file=sys.stderr)
        return 3
    binding.load_library()
    M = N = 8192
    fp8 = args.op == "gemm_fp8"
    K, dtype, seed = args.K, (I.E4M3 if fp8 else I.FP16), 7000 + args.K
    a_bits, b_bits = I.make_ab(M, N, K, dtype, seed)
    a = torch.from_numpy(a_bits if fp8 else a_bits.view("int16")).cuda()
    b = torch.from_numpy(b_bits if fp8 else b_bits.view("int16")).cuda()
    c = torch.empty((M, N), dtype=torch.int16, device="cuda")
    stream = torch.cuda.current_stream()
    flops = 2.0 * M * N * K
    lib = binding.load_library()
    shape = lib.gemm_nt_fp8_shape(M, N, K) if fp8 else lib.gemm_nt_shape(M, N, K)

    def step():
        if fp8:
            binding.gemm_nt_fp8(a, b, c, M, N, K, stream=stream, out_dtype=I.FP16)
        else:
            binding.gemm_nt(a, b, c, M, N, K, stream=stream, dtype=dtype)

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(args.steps + 1)]
    t0 = time.perf_counter()
    ev[0].record(stream)
    for i in range(args.steps):
        step()
        ev[i + 1].record(stream)
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    per_launch = [ev[i].elapsed_time(ev[i + 1]) for i in range(args.steps)]
    ms_per_step = ev[0].elapsed_time(ev[-1]) / args.steps
    kern_ms = statistics.fmean(per_launch)
    achieved = flops / (kern_ms * 1e-3) * 1e-12
    out = {
        "metric": "matrix product C = A B^T TFLOP/s (2*M*N*K), 1 GPU", "value": flops / (ms_per_step * 1e-3) * 1e-12,
        "unit": "TFLOP/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": ms_per_step,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f8e4m3" if fp8 else "f16", "data": "synthetic",
        "config": {"workload": "gemm_nt: M=8192 N=8192 K=%d %s" % (K, "E4M3 operands, fp16 result" if fp8 else "fp16"),
                   "tile": dict(zip(("BM", "BN"), GEMM_SHAPES[shape]), shape=shape),
                   "flops_per_step": flops, "wall_s_timed_region": wall},
        "roofline": {"bound": "mfma", "achieved": achieved, "peak": PEAK_TFLOPS[dtype], "unit": "TFLOP/s",
                     "frac": achieved / PEAK_TFLOPS[dtype],
                     "traffic": measured_traffic((args.op, K))[0],
                     "traffic_unit": "bytes of HBM traffic per launch (rocprofv3 counters, see %s)"
                                     % measured_traffic((args.op, K))[1] if measured_traffic((args.op, K))[0] else None,
                     "kernel_ms": {"mean": kern_ms, "median": statistics.median(per_launch), "min": min(per_launch)}},
        "context": {"paper_h100_fp16_gemm_tflops_k16384": 718.0,
                    "paper_workload": "H100 SXM5, M=N=8192, K=16384, fp16 (Section 5.6); other hardware, not a target"},
    }
    if not args.no_mfma_probe:
        sus = mfma_sustained(binding, torch, dtype, stream)
        sus["unit"] = "TFLOP/s"
        sus["frac_of_random_operands"] = achieved / sus["random_operands"]
        sus["frac_of_zero_operands"] = achieved / sus["zero_operands"]
        out["roofline"]["mfma_only_measured"] = sus
    if not args.no_cpu_baseline:
        from oracle import gemm_ref
        idx = I.sample_entries(M, N, 32, seed=seed + 5, always=[(0, 0), (M - 1, N - 1)])
        ref = gemm_ref.gemm_nt_samples(a_bits, b_bits, dtype, idx)
        ii = np.asarray(idx)
        got = c.view(torch.float16)[ii[:, 0], ii[:, 1]].double().cpu().numpy()
        slack = 2e-6 * K
        if fp8:   # the tests' tolerance: half an ulp of the result plus 2^-14 of sum_k |a_k b_k|
            af, bf = (torch.from_numpy(np.ascontiguousarray(x[ii[:, j]])).view(torch.float8_e4m3fn).double().abs().numpy()
                      for x, j in ((a_bits, 0), (b_bits, 1)))
            slack = 2.0 ** -14 * (af * bf).sum(axis=1)
        out["parity"] = {"entries": len(idx), "max_abs": float(np.abs(got - ref).max()),
                         "max_rel_to_tolerance": float((np.abs(got - ref) / (1.01 * 2.0 ** -11 * np.abs(ref) + slack)).max())}
        out["parity"]["ok"] = bool(out["parity"]["max_rel_to_tolerance"] <= 1.0)
        out["cpu_baseline"] = gemm_cpu_baseline(M, N, K, dtype, seed)
    print(json.dumps(out), flush=True)
    if "parity" in out and not out["parity"]["ok"]:
        print("bench.py: the timed kernel's output is outside the tolerance: %s" % json.dumps(out["parity"]), file=sys.stderr)
        return 4
    return 0


def main() -> int:
    ap = argparse.ArgumentParser()
    ap.add_argument("--op", default="attn", choices=["attn", "gemm", "gemm_fp8"],
                    help="attn: the headline attention workloads (default); gemm: the paper's M=N=8192 matrix product "
                         "in fp16; gemm_fp8: the same on E4M3 operands")
    ap.add_argument("--K", type=int, default=16384, help="inner dimension of --op gemm (the paper sweeps 256 ... 16384)")
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=200)
    ap.add_argument("--warmup", type=int, default=25)
    ap.add_argument("--workload", default="c4",
                    help="c1 ... c5: the 16-bit configurations (c4 = headline, the default); "
                         "f1, f3, f4, f5: the same shapes with Q, K, V in 8-bit float (E4M3), O in fp16")
    ap.add_argument("--no-cpu-baseline", action="store_true",
                    help="skip the CPU oracle (its timing AND the parity check of the timed kernel's output against it)")
    ap.add_argument("--no-all-configs", action="store_true",
                    help="skip the short timing of the other benchmark configurations (key all_configs)")
    ap.add_argument("--no-mfma-probe", action="store_true",
                    help="skip the register-only MFMA stream that measures the sustained matrix-core rate")
    ap.add_argument("--calibrate-copy", action="store_true",
                    help="also run one plain 1 GiB device copy before the timed region (reference point for "
                         "the FETCH_SIZE / WRITE_SIZE counters of a rocprofv3 --pmc run)")
    args = ap.parse_args()

    if args.gpus != 1:
        print("bench.py: this build runs on ONE GPU; the path shards over (batch, head) with no "
              "communication and no multi-GPU figure is produced (asked for --gpus %d)" % args.gpus, file=sys.stderr)
        return 2

    if args.op in ("gemm", "gemm_fp8"):
        return main_gemm(args)

    import torch
    from paper_2510_14719_amd import binding, inputs as I

    if not torch.cuda.is_available():
        print("bench.py: no GPU visible; the HIP path has no CPU fallback", file=sys.stderr)
        return 3
    binding.load_library()
    fp8 = args.workload in I.FP8_WORKLOADS
    w = I.FP8_WORKLOADS[args.workload] if fp8 else I.WORKLOADS[args.workload]
    out_dtype = I.FP16 if fp8 else w.dtype      # element type of O

    # ---- inputs: seeded synthetic tensors, resident in HBM before anything is timed
    if fp8:
        q, k, v = (torch.from_numpy(x).cuda() for x in I.make_workload(w))
        o = torch.full((w.B, w.H, w.N, w.d), 0x7FFF, dtype=torch.int16, device="cuda")
    else:
        q, k, v = (torch.from_numpy(x.view("int16")).cuda() for x in I.make_workload(w))
        o = torch.full_like(q, 0x7FFF)
    # (the outputs start out as NaN patterns: finite outputs afterwards prove that every element was written)
    lse = torch.full((w.B, w.H, w.N), float("nan"), dtype=torch.float32, device="cuda")
    stream = torch.cuda.current_stream()

    def step():
        if fp8:
            binding.attn_fwd_fp8(q, k, v, o, lse, w.B, w.H, w.N, w.d, w.scale, w.causal, stream=stream, out_dtype=out_dtype)
        else:
            binding.attn_fwd(q, k, v, o, lse, w.B, w.H, w.N, w.d, w.scale, w.causal, stream=stream, dtype=w.dtype)

    if args.calibrate_copy:
        src = torch.empty(1 << 28, dtype=torch.float32, device="cuda").fill_(1.0)   # 1 GiB read + 1 GiB written
        dst = torch.empty_like(src)
        dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()

    # ---- timed region: exactly K steps; one HIP event pair per launch on the launch stream
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(args.steps + 1)]
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    ev[0].record(stream)
    for i in range(args.steps):
        step()
        ev[i + 1].record(stream)
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    total_ms = ev[0].elapsed_time(ev[-1])
    per_launch = [ev[i].elapsed_time(ev[i + 1]) for i in range(args.steps)]

    ms_per_step = total_ms / args.steps
    tflops = w.flops / (ms_per_step * 1e-3) * 1e-12
    kern_ms = statistics.fmean(per_launch)
    achieved = w.flops / (kern_ms * 1e-3) * 1e-12
    peak = PEAK_TFLOPS[w.dtype]

    # ---- the timed variant's output against the oracle: the whole heads that the CPU baseline computes anyway,
    # element by element, within the tolerances above.  A violation fails the run (exit code 4).
    parity, base = None, None
    if not args.no_cpu_baseline:
        import numpy as np
        qn, kn, vn = (x.cpu().numpy().view("uint8" if fp8 else "uint16") for x in (q, k, v))
        base, sel, o_ref, l_ref = cpu_baseline(w, qn, kn, vn)
        of = o.view(torch.float16 if out_dtype == 0 else torch.bfloat16).reshape(w.B * w.H, w.N, w.d)[sel].double().cpu().numpy()
        lf = lse.reshape(w.B * w.H, w.N)[sel].double().cpu().numpy()
        whole_o = o.view(torch.float16 if out_dtype == 0 else torch.bfloat16)
        tol = tolerances(w, fp8)
        parity = {"heads": len(sel), "elements": int(of.size), "o_max_abs": float(np.abs(of - o_ref).max()),
                  "o_mean_abs": float(np.abs(of - o_ref).mean()), "lse_max_abs": float(np.abs(lf - l_ref).max()),
                  "all_outputs_finite": bool(torch.isfinite(whole_o).all()) and bool(torch.isfinite(lse).all()),
                  "tolerance": tol}
        parity["ok"] = bool(parity["all_outputs_finite"] and all(parity[k_] <= tol[k_] for k_ in tol))

    lib = binding.load_library()
    tile = binding.fp8_tile_params(w.d) if fp8 else binding.tile_params(w.d, w.causal)
    tile["BM"] = (lib.attn_fwd_fp8_call_rows if fp8 else lib.attn_fwd_call_rows)(w.B, w.H, w.N, w.d, int(w.causal))

    out = {
        "metric": "attention fwd TFLOP/s (4*B*H*N^2*d, halved causal), 1 GPU",
        "value": tflops,
        "unit": "TFLOP/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_per_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": {0: "f16", 1: "bf16", 2: "f8e4m3"}[w.dtype],
        "data": "synthetic",
        "config": {"workload": describe(w), "scale": w.scale,
                   "tile": tile,
                   "flops_per_step": w.flops, "wall_s_timed_region": wall},
        "frac_of_mfma_peak": tflops / peak,
        "roofline": {"bound": "mfma", "achieved": achieved, "peak": peak, "unit": "TFLOP/s", "frac": achieved / peak,
                     "traffic": measured_traffic(w.name)[0],
                     "traffic_unit": "bytes of HBM traffic per launch (rocprofv3 counters, see %s)"
                                     % measured_traffic(w.name)[1] if measured_traffic(w.name)[0] else None,
                     "kernel_ms": {"mean": kern_ms, "median": statistics.median(per_launch), "min": min(per_launch)}},
        "context": {"paper_h100_fp16_mha_tflops": 654.0,
                    "paper_workload": "H100 SXM5, L=16384, batch 4, d=128 (Section 5.6); other hardware, not a target"},
    }
    if fp8:
        out["context"] = {"paper": "the paper plots FP8 attention (Section 5.4) without printing a number for it",
                          "p_precision": "probabilities rounded to E4M3 before P V; O in fp16"}
    if not args.no_mfma_probe:
        # outside the timed region: the measured MFMA-only rates next to the datasheet peak
        sus = mfma_sustained(binding, torch, w.dtype, stream)
        sus["unit"] = "TFLOP/s"
        sus["frac_of_random_operands"] = achieved / sus["random_operands"]
        sus["frac_of_zero_operands"] = achieved / sus["zero_operands"]
        out["roofline"]["mfma_only_measured"] = sus
    if parity is not None:
        out["parity"] = parity
        out["cpu_baseline"] = base
    if not args.no_all_configs and not fp8:
        out["all_configs"] = all_configs(binding, torch, I, stream)
    print(json.dumps(out), flush=True)
    if parity is not None and not parity["ok"]:
        print("bench.py: the timed kernel's output is outside the tolerances: %s" % json.dumps(parity), file=sys.stderr)
        return 4
    return 0


if __name__ == "__main__":
    sys.exit(main())
