#!/usr/bin/env python3
"""Benchmark of the deterministic decode hot path on one MI355X.

    python bench.py [--gpus 1] [--steps K] [--warmup W]

A step is one pass over the Llama-3-8B-shaped projection GEMM workload: the four weight shapes
(K=4096 -> N=4096 / 6144 / 28672, K=14336 -> N=4096) at every M in {1,2,4,8,16,32,64,128,256},
36 det_gemm_bf16 launches on synthetic data that is already resident in HBM.  Weights rotate
through three distinct sets (1.3 GB) so that every launch streams its weights from HBM, not from
the 256 MB last-level cache.  `value` is the step's total FLOP over its wall time.

The JSON line also carries: the roofline record of the dominant kernel; the CPU oracle timed on this host as a
reported baseline; greedy-decode tokens/s; and a bit-identical rate over repeated and re-batched runs.
It is kept short (LINE_BYTES), since what reads it may keep only so much of the output.  The tables (every (shape, M) measured
with HIP events, cache-cold and cache-warm, attention, decoder layers, quantized and library products, token selection) go
to stderr as one JSON object, and to a file with --tables.
"""
from __future__ import annotations

import argparse
import json
import math
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

SHAPES = [(4096, 4096), (4096, 6144), (4096, 28672), (14336, 4096)]  # (K, N)
MS = [1, 2, 4, 8, 16, 32, 64, 128, 256]
N_SETS = 3
PEAK_MFMA_TFLOPS = 2500.0   # MI355X dense bf16
PEAK_HBM_GBS = 8000.0       # MI355X HBM3E
DOMINANT = (4096, 28672)    # the launch that moves most of the step's bytes (gemm_kernel<8,144,0,8,4,8,false,0>)
LINE_BYTES = 4000
LINE_KEYS = ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline",
             "dtype", "data", "config", "roofline", "fingerprint", "cpu_baseline", "bit_identical")


def split_record(result):
    """(the JSON line's object, the tables' object) of everything a run measured."""
    line = {k: dict(result[k]) if isinstance(result[k], dict) else result[k] for k in LINE_KEYS if k in result}
    tables = {k: v for k, v in result.items() if k not in line}
    if "other_legs" in line.get("cpu_baseline", {}):
        tables["cpu_baseline_other_legs"] = line["cpu_baseline"].pop("other_legs")
    peaks = result.get("measured_peaks", {})
    line["measured_peaks"] = {k: peaks[k] for k in ("copy_1GiB_gbs", "read_1GiB_gbs") if k in peaks}
    line["decode_tokens_per_s"] = {
        k: v["generated_tokens_per_s"] if isinstance(v, dict) else {f"B{r['B']}": r["tokens_per_s"] for r in v}
        for k, v in result.get("decode", {}).items() if isinstance(v, dict) or "tokens_per_s" in v[0]}
    return line, tables


def dominant_traffic_bytes():
    """HBM bytes per launch of the dominant kernel as measured with rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE
    (scaled by a plain copy kernel of known size): read from the committed summary of those runs,
    profiles/gemm_kernel_llama_sweep.md.  None if the summary is missing (the bench never guesses it)."""
    import re
    try:
        text = open(os.path.join(ROOT, "profiles", "gemm_kernel_llama_sweep.md")).read()
    except OSError:
        return None
    m = re.search(r"measured HBM traffic ([0-9.]+) MB per launch", text)
    return float(m.group(1)) * 1e6 if m else None


def gemm_flops(M, N, K):
    return 2.0 * M * N * K


def gemm_bytes(M, N, K):
    """Algorithmic bytes: weights once, activations once, bf16 output once."""
    return 2.0 * (K * N + M * K + M * N)


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--tables", default=None, metavar="FILE", help="also write the tables to this file")
    ap.add_argument("--skip-extras", action="store_true", help="only the timed GEMM workload")
    ap.add_argument("--calibrate-copy", action="store_true",
                    help="run a plain device-to-device copy of known size (for scaling rocprofv3 --pmc "
                         "FETCH_SIZE / WRITE_SIZE readings) and exit")
    ap.add_argument("--probe", default=None, metavar="SPEC",
                    help="run a few launches of ONE operation and exit (the program that rocprofv3 counter "
                         "passes run): gemm:K:N:M, gemm_fixed:K:N:M, qgemm:K:N:M, attn:B:L, prefill:S:T, layer:B, step:B")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py: this build runs on one GPU only (no collectives, no sharding); use --gpus 1",
              file=sys.stderr)
        sys.exit(2)

    import torch

    import detsynth as ds
    import paper_2602_00182_amd as det

    if not torch.cuda.is_available():
        print("bench.py: no GPU visible", file=sys.stderr)
        sys.exit(2)
    dev = "cuda:0"
    torch.cuda.set_device(0)

    if args.calibrate_copy:
        nbytes = 256 << 20
        a = torch.full((nbytes,), 7, dtype=torch.uint8, device=dev)
        b = torch.empty_like(a)
        for _ in range(5):
            b.copy_(a)
        torch.cuda.synchronize()
        print(json.dumps({"calibrate_copy_bytes_read": nbytes, "calibrate_copy_bytes_written": nbytes,
                          "launches": 5}))
        return

    if args.probe:
        probe(torch, det, ds, dev, args.probe)
        return

    # ------------------------------------------------------------------ resident inputs
    weights = {}   # (K, N, set) -> packed weight
    for si in range(N_SETS):
        for j, (K, N) in enumerate(SHAPES):
            w = ds.normal_bf16_torch(ds.tensor_seed(2, 10 * si + j), (K, N), 0.02, 0.0, dev)
            weights[(K, N, si)] = det.pack_weight(w)
            del w
    X = {K: ds.normal_bf16_torch(ds.tensor_seed(2, 7) + K, (256, K), 1.0, 0.0, dev) for K in (4096, 14336)}
    C = {(K, N): torch.empty((256, N), dtype=torch.bfloat16, device=dev) for (K, N) in SHAPES}
    torch.cuda.synchronize()

    # Launch arguments are marshalled once: inside the timed region a launch is one call into the C ABI
    # (the thin binding's shape checks cost several microseconds a call, as much as the small kernels).
    from paper_2602_00182_amd._lib import lib as _det_lib
    L = _det_lib()
    stream = torch.cuda.current_stream().cuda_stream
    launch_args = {(K, N, M, si): (X[K].data_ptr(), K, weights[(K, N, si)].data_ptr(), C[(K, N)].data_ptr(), N, M, N, K,
                                   0, stream)
                   for (K, N) in SHAPES for M in MS for si in range(N_SETS)}

    # HIP events without the system-scope fence (device-scope timestamps on this stream): the fence of a
    # default event costs the GPU a few microseconds per record, which would be charged to 48 us launches.
    import ctypes
    hip = ctypes.CDLL("libamdhip64.so")
    hip.hipEventCreateWithFlags.argtypes = [ctypes.POINTER(ctypes.c_void_p), ctypes.c_uint]
    hip.hipEventRecord.argtypes = [ctypes.c_void_p, ctypes.c_void_p]
    hip.hipEventSynchronize.argtypes = [ctypes.c_void_p]
    hip.hipEventElapsedTime.argtypes = [ctypes.POINTER(ctypes.c_float), ctypes.c_void_p, ctypes.c_void_p]

    class Ev:
        def __init__(self):
            self.h = ctypes.c_void_p()
            if hip.hipEventCreateWithFlags(ctypes.byref(self.h), 0x20000000) != 0:   # hipEventDisableSystemFence
                raise RuntimeError("hipEventCreateWithFlags failed")

        def record(self):
            if hip.hipEventRecord(self.h, stream) != 0:
                raise RuntimeError("hipEventRecord failed")

        def elapsed_time(self, other):
            ms = ctypes.c_float()
            hip.hipEventSynchronize(other.h)
            if hip.hipEventElapsedTime(ctypes.byref(ms), self.h, other.h) != 0:
                raise RuntimeError("hipEventElapsedTime failed")
            return ms.value

    def run_step(step_idx, events=None, which=None, entry=None):
        """One step: the 36 launches.  events: list to collect (key, e0, e1) HIP-event pairs for the
        shapes in `which` (None: every shape).  entry: the C entry point (default det_gemm_bf16)."""
        entry = entry or L.det_gemm_bf16
        for mi, M in enumerate(MS):
            si = (step_idx * len(MS) + mi) % N_SETS
            for (K, N) in SHAPES:
                timed = events is not None and (which is None or (K, N) in which)
                if timed:
                    e0, e1 = Ev(), Ev()
                    e0.record()
                rc = entry(*launch_args[(K, N, M, si)])
                if rc != 0:
                    raise RuntimeError(f"det_gemm_bf16 failed with status {rc}")
                if timed:
                    e1.record()
                    events.append(((K, N, M), e0, e1))

    for s in range(args.warmup):
        run_step(s)
    torch.cuda.synchronize()
    dom_events = []   # the dominant shape's launches are timed live, inside the timed region
    t0 = time.perf_counter()
    for s in range(args.steps):
        run_step(args.warmup + s, dom_events, (DOMINANT,))
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    ms_per_step = (t1 - t0) * 1e3 / args.steps
    step_flops = sum(gemm_flops(M, N, K) for (K, N) in SHAPES for M in MS)
    value = step_flops / (ms_per_step * 1e-3) / 1e12

    # per-(shape, M) table: the same steps again, outside the timed region, with events on every launch
    events = []
    for s in range(min(args.steps, 10)):
        run_step(args.warmup + args.steps + s, events)
    torch.cuda.synchronize()

    per = {}
    for key, e0, e1 in events:
        per.setdefault(key, []).append(e0.elapsed_time(e1))

    def table(per_ms):
        rows = []
        for (K, N) in SHAPES:
            for M in MS:
                ms = float(np.mean(per_ms[(K, N, M)]))
                fl, by = gemm_flops(M, N, K), gemm_bytes(M, N, K)
                tf, gbs = fl / ms / 1e9, by / ms / 1e6
                roof = min(PEAK_MFMA_TFLOPS, fl / by * PEAK_HBM_GBS / 1e3)
                rows.append({"K": K, "N": N, "M": M, "us": round(ms * 1e3, 2), "tflops": round(tf, 2),
                             "gbs": round(gbs, 1), "frac_mfma": round(tf / PEAK_MFMA_TFLOPS, 4),
                             "frac_hbm": round(gbs / PEAK_HBM_GBS, 4), "frac_roofline": round(tf / roof, 4)})
        return rows

    sweep_cold = table(per)

    # The same cold sweep through det_gemm_bf16_fixed_tile: one tiling per (N, K) whatever M.  The gap to
    # sweep_cold is what the tiling keyed on M buys (the bytes are the same, see the tests).
    events_fixed = []
    for s in range(min(args.steps, 10)):
        run_step(args.warmup + args.steps + s, events_fixed, entry=L.det_gemm_bf16_fixed_tile)
    torch.cuda.synchronize()
    per_fixed = {}
    for key, e0, e1 in events_fixed:
        per_fixed.setdefault(key, []).append(e0.elapsed_time(e1))
    sweep_cold_fixed_tile = table(per_fixed)

    # Per shape: the worst fraction of the HBM peak over M <= 8 and of the MFMA peak over M >= 128 (cold).
    per_shape = []
    for (K, N) in SHAPES:
        rows = [r for r in sweep_cold if r["K"] == K and r["N"] == N]
        rows_f = [r for r in sweep_cold_fixed_tile if r["K"] == K and r["N"] == N]
        per_shape.append({"K": K, "N": N,
                          "min_frac_hbm_M_le_8": min(r["frac_hbm"] for r in rows if r["M"] <= 8),
                          "min_frac_mfma_M_ge_128": min(r["frac_mfma"] for r in rows if r["M"] >= 128),
                          "min_frac_mfma_M_ge_128_fixed_tile": min(r["frac_mfma"] for r in rows_f if r["M"] >= 128)})

    # dominant kernel: all launches of the N=28672 shape inside the timed region
    dom_ms = [e0.elapsed_time(e1) for _, e0, e1 in dom_events]
    dom_bytes = float(np.mean([gemm_bytes(M, DOMINANT[1], DOMINANT[0]) for M in MS]))
    dom_avg_ms = float(np.mean(dom_ms))
    achieved = dom_bytes / dom_avg_ms / 1e6
    roofline = {"bound": "hbm", "kernel": "det::gemm_kernel<8,144,0,8,4,8,false,0> (K=4096, N=28672, M=1..256)",
                "achieved": round(achieved, 1), "peak": PEAK_HBM_GBS, "unit": "GB/s",
                "frac": round(achieved / PEAK_HBM_GBS, 4), "traffic": dominant_traffic_bytes(),
                "avg_launch_us": round(dom_avg_ms * 1e3, 2), "bytes_per_launch": int(dom_bytes),
                "per_shape": per_shape}

    result = {
        "metric": "det. GEMM TFLOP/s & %MFMA peak (M=1..256); decode tokens/s; bit-identical rate",
        "value": round(value, 3), "unit": "TFLOP/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": round(ms_per_step, 4), "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "bf16", "data": "synthetic",
        "config": {"workload": "Llama-3-8B-shaped projection GEMMs, K=4096 x N in {4096,6144,28672} and "
                               "K=14336 x N=4096, M in {1,2,4,8,16,32,64,128,256}, bf16 in, fp32 accumulate, "
                               "bf16 out; weights rotate over 3 sets (HBM-cold)",
                   "launches_per_step": len(SHAPES) * len(MS), "flop_per_step": step_flops},
        "roofline": roofline,
        "sweep_cold": sweep_cold,
        "sweep_cold_fixed_tile": sweep_cold_fixed_tile,
        "fingerprint": det.det_fingerprint(),
    }

    if not args.skip_extras:
        result["measured_peaks"] = measured_peaks(torch, dev, roofline)
        result["sweep_warm"] = warm_sweep(torch, det, weights, X, C, table)
        result["cpu_baseline"] = cpu_baseline(ds)
        result["bit_identical"] = bit_identical(torch, det, weights, X)
        del weights, C
        torch.cuda.empty_cache()
        result["attention"] = attention_numbers(torch, det, ds, dev)
        result["decode"] = decode_numbers(torch, det, ds, dev)
        result["qgemm_w4a8"] = qgemm_numbers(torch, det, ds, dev)
        result["library_gemm"] = library_gemm(torch, ds, dev, sweep_cold)
        result["token_selection"] = selection_numbers(torch, det, ds, dev)
    line, tables = split_record(result)
    print(json.dumps(tables), file=sys.stderr, flush=True)
    if args.tables:
        with open(args.tables, "w") as f:
            json.dump(tables, f, indent=1)
    print(json.dumps(line))


def probe(torch, det, ds, dev, spec):
    """A few launches of one operation at one size, for counter passes of rocprofv3 (every launch of the
    named kernel in the run is the same work, so per-dispatch counters can be averaged)."""
    kind, *nums = spec.split(":")
    nums = [int(x) for x in nums]
    scale = float(np.float32(1.0 / math.sqrt(128.0)))
    reps = 12
    if kind in ("gemm", "gemm_fixed", "qgemm"):
        K, N, M = nums
        X = ds.normal_bf16_torch(ds.tensor_seed(2, 7) + K, (M, K), 1.0, 0.0, dev)
        C = torch.empty((M, N), dtype=torch.bfloat16, device=dev)
        Ws = [ds.normal_bf16_torch(ds.tensor_seed(2, 10 * si), (K, N), 0.02, 0.0, dev) for si in range(3)]
        if kind == "qgemm":
            Wp = [det.quant_pack_weight(w) for w in Ws]
            codes, scales = det.quant_activations(X)
            for i in range(reps):
                det.det_qgemm_w4a8(codes, scales, Wp[i % 3], C, N)
        else:
            Wp = [det.pack_weight(w) for w in Ws]
            fn = det.det_gemm_bf16 if kind == "gemm" else det.det_gemm_bf16_fixed_tile
            for i in range(reps):
                fn(X, Wp[i % 3], C, N, K)
    elif kind in ("attn", "prefill"):
        Hq, Hkv, D = 32, 8, 128
        if kind == "attn":
            B, L = nums
            S, R = B, B
            lens = torch.full((B,), L, dtype=torch.int32, device=dev)
            slots = None
        else:
            S, T = nums
            L, R = ((T + 255) // 256) * 256, S * T
            lens = (torch.arange(R, device=dev, dtype=torch.int32) % T + 1).contiguous()
            slots = (torch.arange(R, device=dev, dtype=torch.int32) // T).contiguous()
        q = ds.normal_bf16_torch(ds.tensor_seed(3, 10), (R, Hq, D), 1.0, 0.0, dev)
        k = ds.normal_bf16_torch(ds.tensor_seed(3, 11), (S, Hkv, L, D), 1.0, 0.0, dev)
        v = ds.normal_bf16_torch(ds.tensor_seed(3, 12), (S, Hkv, L, D), 1.0, 0.0, dev)
        ws = torch.empty(det.det_attn_decode_workspace_bytes(R, Hq, D, L), dtype=torch.uint8, device=dev)
        out = torch.empty((R, Hq, D), dtype=torch.bfloat16, device=dev)
        for _ in range(reps):
            if slots is None:
                det.det_attn_decode(q, k, v, lens, out, ws, scale)
            else:
                det.det_attn_decode_rows(q, k, v, lens, slots, out, ws, scale)
    elif kind == "layer":
        (B,) = nums
        H, Hq, Hkv, D, F, Lmax = 4096, 32, 8, 128, 14336, 2048
        g = lambda i, shape, std=0.02, mean=0.0: ds.normal_bf16_torch(ds.tensor_seed(4, i), shape, std, mean, dev)
        w = det.layer_weights(g(0, (H,), 0.0, 1.0), det.pack_qkv(g(1, (H, (Hq + 2 * Hkv) * D)), Hq, Hkv, D),
                              det.pack_weight(g(2, (Hq * D, H))), g(3, (H,), 0.0, 1.0),
                              det.pack_gate_up(g(4, (H, 2 * F))), det.pack_weight(g(5, (F, H))))
        cfg = det.layer_cfg(H, Hq, Hkv, D, F, Lmax, 1e-5, scale)
        cos_t, sin_t = ds.rope_tables(Lmax, D, 5.0e5)
        cos_d, sin_d = torch.from_numpy(cos_t).to(dev), torch.from_numpy(sin_t).to(dev)
        x = g(50, (B, H), 1.0)
        kc, vc = g(70, (B, Hkv, Lmax, D), 1.0), g(80, (B, Hkv, Lmax, D), 1.0)
        pos = torch.full((B,), Lmax - 1, dtype=torch.int32, device=dev)
        ws = torch.empty(det.det_decoder_layer_workspace_bytes(cfg, B), dtype=torch.uint8, device=dev)
        for _ in range(reps):
            det.det_decoder_layer(w, cfg, x, kc, vc, pos, cos_d, sin_d, ws)
    elif kind == "step":
        # one greedy decode step of the 8-layer model of decode_numbers (context 512), B sequences
        from paper_2602_00182_amd.decode import DecodeModel, ModelCfg
        (B,) = nums
        H, Hq, Hkv, D, F, V, NL, Lm = 2048, 16, 4, 128, 5632, 32000, 8, 640
        s = ds.tensor_seed(5, 0)
        g = lambda i, shape, std=0.02, mean=0.0: ds.normal_bf16_torch(s + i, shape, std, mean, dev)
        layers = [dict(norm1=g(10 + 10 * l, (H,), 0.0, 1.0), wqkv=g(11 + 10 * l, (H, (Hq + 2 * Hkv) * D)),
                       wo=g(12 + 10 * l, (Hq * D, H)), norm2=g(13 + 10 * l, (H,), 0.0, 1.0),
                       wgu=g(14 + 10 * l, (H, 2 * F)), wdown=g(15 + 10 * l, (F, H))) for l in range(NL)]
        model = DecodeModel(ModelCfg(H, Hq, Hkv, D, F, V, NL),
                            dict(embed=g(1, (V, H), 1.0), lm_head=g(2, (H, V)), final_norm=g(3, (H,), 0.0, 1.0), layers=layers))
        cos_t, sin_t = ds.rope_tables(Lm, D, 5.0e5)
        st = model.new_state(B, Lm, torch.from_numpy(cos_t).to(dev), torch.from_numpy(sin_t).to(dev))
        st.tokens.copy_(torch.from_numpy(ds.uniform_int(s + 900, (B,), 0, V - 1)).to(dev))
        st.positions.fill_(511)
        idx = torch.empty(B, dtype=torch.int32, device=dev)
        for _ in range(reps):
            st.forward()
            det.det_argmax(st.logits, idx)
    else:
        raise SystemExit(f"bench.py: unknown probe {spec!r}")
    torch.cuda.synchronize()
    print(json.dumps({"probe": spec, "launches": reps}))


def measured_peaks(torch, dev, roofline):
    """What this GPU streams in practice, next to the datasheet peak: a 1 GiB device-to-device copy (bytes
    read plus bytes written over the time) and a read-only pass (torch's sum over 1 GiB).  Also restates the
    dominant kernel's achieved bandwidth as a fraction of the better of the two."""
    n = 1 << 30
    a = torch.empty(n, dtype=torch.uint8, device=dev)
    b = torch.empty_like(a)
    a.zero_()
    f = a.view(torch.float32)

    def timed(fn, reps=10):
        fn()
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(reps):
            fn()
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) / reps

    copy_ms = timed(lambda: b.copy_(a))
    read_ms = timed(lambda: f.sum())
    # LDS fill rate of a compute unit for L2-resident data (the library's probe kernels): 256 workgroups, one per
    # compute unit, all streaming the same 2 MB
    import paper_2602_00182_amd as det
    small = torch.ones(2 << 20, dtype=torch.uint8, device=dev)
    sink = torch.zeros(4, dtype=torch.uint8, device=dev)
    fill = {}
    for path, name in ((0, "registers_then_lds_store"), (1, "lds_dma")):
        iters = 2000
        ms = timed(lambda: det.det_probe_lds_fill(small, path, 256, iters, sink), reps=3)
        fill[name + "_bytes_per_clock_per_cu_at_2p4ghz"] = round(256 * iters * 32768 / ms / 1e6 / 256 / 2.4, 1)
    copy_gbs = 2 * n / copy_ms / 1e6
    read_gbs = n / read_ms / 1e6
    best = max(copy_gbs, read_gbs)
    # What a launch of a shape's size can reach at all: a plain device copy that moves as many bytes as the
    # shape's weights (K*N bytes read, K*N written), buffers rotating through the 1 GiB arrays so that every
    # copy is HBM-cold, launches back to back.  A launch of 33 MB is over before the chip streams at its rate.
    same_bytes = []
    for (K, N) in SHAPES:
        kn = K * N
        slots = max(2, n // kn)
        state = [0]

        def one(kn=kn, slots=slots, state=state):
            i = state[0] % slots
            state[0] += 1
            b[i * kn:(i + 1) * kn].copy_(a[i * kn:(i + 1) * kn])
        ms = timed(one, reps=3 * slots)
        same_bytes.append({"K": K, "N": N, "bytes_mb": round(2 * kn / 1e6, 1), "copy_us": round(ms * 1e3, 2),
                           "copy_frac_hbm": round(2 * kn / ms / 1e6 / PEAK_HBM_GBS, 4)})
    del a, b, f
    torch.cuda.empty_cache()
    return {"copy_1GiB_gbs": round(copy_gbs, 1), "read_1GiB_gbs": round(read_gbs, 1),
            "dominant_kernel_frac_of_measured": round(roofline["achieved"] / best, 4),
            "copy_of_a_shapes_bytes": same_bytes,
            "lds_fill_l2_resident": fill,
            "note": "device-to-device copy counts read + written bytes; the read pass is torch's sum over fp32"}


def selection_numbers(torch, det, ds, dev):
    """det_argmax and det_sample (seeded temperature / top-k / top-p) on V = 32000 fp32 logits, GPU time per
    call from marshalled calls."""
    from paper_2602_00182_amd._lib import lib as _det_lib
    L = _det_lib()
    V = 32000
    stream = torch.cuda.current_stream().cuda_stream
    rows = []
    for B in (1, 64):
        logits = ds.normal_bf16_torch(ds.tensor_seed(5, 700), (B, V), 3.0, 0.0, dev).float().contiguous()
        out = torch.empty(B, dtype=torch.int32, device=dev)
        ids = torch.arange(B, dtype=torch.int32, device=dev)
        steps = torch.zeros(B, dtype=torch.int32, device=dev)
        cases = [("argmax", lambda: L.det_argmax(logits.data_ptr(), out.data_ptr(), B, V, 1, stream))]
        for (T, k, p) in ((1.0, 50, 0.9), (0.7, 1024, 1.0)):
            cases.append((f"sample T={T} top_k={k} top_p={p}",
                          lambda T=T, k=k, p=p: L.det_sample(logits.data_ptr(), B, V, T, k, p, 1234, ids.data_ptr(),
                                                             steps.data_ptr(), out.data_ptr(), stream)))
        for name, call in cases:
            for _ in range(3):
                if call() != 0:
                    raise RuntimeError(name + " failed")
            torch.cuda.synchronize()
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(20):
                call()
            e1.record()
            torch.cuda.synchronize()
            rows.append({"B": B, "op": name, "us": round(e0.elapsed_time(e1) / 20 * 1e3, 1)})
    return rows


def library_gemm(torch, ds, dev, sweep_cold):
    """Context for the cost of determinism (the paper's section 6.5 quotes its kernels at 95-98 % of the
    vendor library): torch.matmul, i.e. the platform's default bf16 GEMM with no ordering guarantee, on the
    same shapes and M with the same rotation over three weight sets.  det_over_library = this library's
    cold time / the default GEMM's time (below 1: the deterministic kernel is faster).  Not part of `value`."""
    ours = {(r["K"], r["N"], r["M"]): r["us"] for r in sweep_cold}
    rows = []
    for (K, N) in SHAPES:
        ws = [ds.normal_bf16_torch(ds.tensor_seed(2, 50 + si) + K // 64 + N, (K, N), 0.02, 0.0, dev) for si in range(N_SETS)]
        x = ds.normal_bf16_torch(ds.tensor_seed(2, 7), (256, K), 1.0, 0.0, dev)
        c = torch.empty((256, N), dtype=torch.bfloat16, device=dev)
        for M in MS:
            n = 12

            def launches():
                for i in range(n):
                    torch.matmul(x[:M], ws[i % N_SETS], out=c[:M])

            launches()
            torch.cuda.synchronize()
            # The twelve launches are replayed from a captured graph so that the host's dispatch time (10-20 us
            # a call, more than the small kernels take) is not charged to the library; eager timing otherwise.
            timed, how = launches, "eager"
            try:
                side = torch.cuda.Stream()
                with torch.cuda.stream(side):
                    launches()
                torch.cuda.synchronize()
                graph = torch.cuda.CUDAGraph()
                with torch.cuda.graph(graph):
                    launches()
                graph.replay()
                torch.cuda.synchronize()
                timed, how = graph.replay, "graph"
            except Exception:
                torch.cuda.synchronize()
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            timed()
            e1.record()
            torch.cuda.synchronize()
            us = e0.elapsed_time(e1) / n * 1e3
            rows.append({"K": K, "N": N, "M": M, "us": round(us, 2), "timed": how,
                         "det_over_library": round(ours[(K, N, M)] / us, 3)})
        del ws, x, c
        torch.cuda.empty_cache()
    return rows


def warm_sweep(torch, det, weights, X, C, table):
    """Same weights back to back: the 33-235 MB matrix can stay in the last-level cache."""
    from paper_2602_00182_amd._lib import lib as _det_lib
    L = _det_lib()
    stream = torch.cuda.current_stream().cuda_stream
    per = {}
    for (K, N) in SHAPES:
        for M in MS:
            a = (X[K].data_ptr(), K, weights[(K, N, 0)].data_ptr(), C[(K, N)].data_ptr(), N, M, N, K, 0, stream)
            for _ in range(3):
                L.det_gemm_bf16(*a)
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(10):
                L.det_gemm_bf16(*a)
            e1.record()
            torch.cuda.synchronize()
            per[(K, N, M)] = [e0.elapsed_time(e1) / 10]
    return table(per)


def cpu_baseline(ds):
    """The oracle as it stands, timed on this host: fp64 reference GEMM of the four shapes at
    M = 256 rows (the largest M of the workload; a bounded sample of it: one M of nine), all host
    threads, repeated until about ten seconds of CPU work have been timed."""
    import oracle

    oracle.lib()
    M = 256
    flops = 0.0
    t = 0.0
    reps = 0
    mats = []
    for j, (K, N) in enumerate(SHAPES):
        mats.append((ds.normal_bf16(ds.tensor_seed(2, 7) + K, (M, K)), ds.normal_bf16(ds.tensor_seed(2, j), (K, N), 0.02), K, N))
    while t < 10.0 and reps < 4:
        for A, B, K, N in mats:
            t0 = time.perf_counter()
            oracle.gemm_f64(A, B, want_abs=False)
            t += time.perf_counter() - t0
            flops += gemm_flops(M, N, K)
        reps += 1
    return {"value": round(flops / t / 1e12, 6), "unit": "TFLOP/s", "cores": oracle.num_threads(),
            "cores_note": "threads of the oracle's parallel loops (OpenMP), as many as the host offers this process",
            "kind": "oracle", "sample": f"fp64 reference GEMM, the four shapes at M={M}, {reps} pass(es) "
                                        f"({flops / 1e9:.0f} GFLOP in {t:.1f} s)", "cpu": _cpu_model(),
            "other_legs": cpu_baseline_other_legs(ds)}


def cpu_baseline_other_legs(ds):
    """The oracle timed on the other parts of the path, each a bounded sample (a few seconds): fp32 RMSNorm /
    softmax / argmax, fp64 attention at one point of the attention grid, one Llama-shaped decoder layer at
    B = 1, and one decode step of a small model (2 layers, H = 256)."""
    import oracle
    from oracle import model as omodel

    legs = {}

    def timed(fn, min_s=1.0, max_reps=50):
        t, n = 0.0, 0
        while t < min_s and n < max_reps:
            t0 = time.perf_counter()
            fn()
            t += time.perf_counter() - t0
            n += 1
        return t / n, n

    x = ds.normal_bf16(901, (256, 4096))
    w = ds.normal_bf16(902, (4096,), 0.0, 1.0)
    dt, n = timed(lambda: oracle.rmsnorm(x, w, 1e-5))
    legs["rmsnorm_256x4096"] = {"us": round(dt * 1e6, 1), "rows_per_s": round(256 / dt, 1), "reps": n}
    sc = (ds.bf16_bits_to_f32(ds.normal_bf16(903, (64, 4096))) * np.float32(3.0)).astype(np.float32)
    lens = np.full(64, 4096, dtype=np.int32)
    dt, n = timed(lambda: oracle.softmax_f32(sc, lens))
    legs["softmax_64x4096"] = {"us": round(dt * 1e6, 1), "rows_per_s": round(64 / dt, 1), "reps": n}
    lg = ds.bf16_bits_to_f32(ds.normal_bf16(904, (64, 32000))).astype(np.float32)
    dt, n = timed(lambda: oracle.argmax_f32(lg))
    legs["argmax_64x32000"] = {"us": round(dt * 1e6, 1), "rows_per_s": round(64 / dt, 1), "reps": n}

    B, Hq, Hkv, D, L = 16, 32, 8, 128, 4096
    q = ds.normal_bf16(905, (B, Hq, D))
    k = ds.normal_bf16(906, (B, Hkv, L, D))
    v = ds.normal_bf16(907, (B, Hkv, L, D))
    scale = float(np.float32(1.0 / math.sqrt(128.0)))
    dt, n = timed(lambda: oracle.attn_decode_f64(q, k, v, np.full(B, L, dtype=np.int32), scale), max_reps=5)
    legs["attention_f64_B16_L4096"] = {"ms": round(dt * 1e3, 2), "kv_gb_per_s": round(B * Hkv * L * D * 4 / dt / 1e9, 2),
                                        "reps": n}

    H, F, Lmax = 4096, 14336, 2048
    s = ds.tensor_seed(4, 0)
    g = lambda i, shape, std=0.02, mean=0.0: ds.normal_bf16(s + i, shape, std, mean)
    lw = dict(norm1=g(0, (H,), 0.0, 1.0), wqkv=g(1, (H, (Hq + 2 * Hkv) * D)), wo=g(2, (Hq * D, H)),
              norm2=g(3, (H,), 0.0, 1.0), wgu=g(4, (H, 2 * F)), wdown=g(5, (F, H)))
    cfg = dict(H=H, Hq=Hq, Hkv=Hkv, D=D, F=F, Lmax=Lmax, eps=1e-5, scale=scale)
    cos_t, sin_t = ds.rope_tables(Lmax, D, 5.0e5)
    x1 = ds.normal_bf16(s + 51, (1, H))
    kc = ds.normal_bf16(s + 71, (1, Hkv, Lmax, D))
    vc = ds.normal_bf16(s + 81, (1, Hkv, Lmax, D))
    dt, n = timed(lambda: omodel.layer(x1, lw, kc, vc, [Lmax - 1], cos_t, sin_t, cfg), max_reps=3)
    legs["decoder_layer_B1_ctx2048"] = {"ms": round(dt * 1e3, 1), "layer_tokens_per_s": round(1 / dt, 2), "reps": n}
    del lw, kc, vc

    H, Hq, Hkv, F, V, NL, Lm = 256, 2, 1, 512, 512, 2, 64
    s = ds.tensor_seed(5, 700)
    g = lambda i, shape, std=0.05, mean=0.0: ds.normal_bf16(s + i, shape, std, mean)
    layers = [dict(norm1=g(10 * l, (H,), 0.0, 1.0), wqkv=g(10 * l + 1, (H, (Hq + 2 * Hkv) * D)), wo=g(10 * l + 2, (Hq * D, H)),
                   norm2=g(10 * l + 3, (H,), 0.0, 1.0), wgu=g(10 * l + 4, (H, 2 * F)), wdown=g(10 * l + 5, (F, H)))
              for l in range(1, NL + 1)]
    weights = dict(embed=g(1, (V, H), 1.0), lm_head=g(2, (H, V)), final_norm=g(3, (H,), 0.0, 1.0), layers=layers)
    cfg = dict(H=H, Hq=Hq, Hkv=Hkv, D=D, F=F, Lmax=Lm, eps=1e-5, scale=scale)
    cos_t, sin_t = ds.rope_tables(Lm, D, 5.0e5)
    kcs = [np.zeros((4, Hkv, Lm, D), dtype=np.uint16) for _ in range(NL)]
    vcs = [np.zeros((4, Hkv, Lm, D), dtype=np.uint16) for _ in range(NL)]
    toks = ds.uniform_int(s + 900, (4,), 0, V - 1)
    dt, n = timed(lambda: omodel.model_step(weights, cfg, toks, np.full(4, 10, dtype=np.int32), kcs, vcs, cos_t, sin_t))
    legs["small_model_step_B4_2layers_H256"] = {"ms": round(dt * 1e3, 2), "tokens_per_s": round(4 / dt, 1), "reps": n}
    return legs


def _cpu_model():
    """Model string of the host CPU; virtual machines often report only the family name, so the family /
    model / stepping numbers and the number of logical CPUs this process may use are appended."""
    name, fam, model, step = "unknown", None, None, None
    try:
        for line in open("/proc/cpuinfo"):
            key, _, val = line.partition(":")
            key, val = key.strip(), val.strip()
            if key == "model name" and name == "unknown":
                name = val
            elif key == "cpu family" and fam is None:
                fam = val
            elif key == "model" and model is None:
                model = val
            elif key == "stepping" and step is None:
                step = val
    except OSError:
        pass
    try:
        ncpu = len(os.sched_getaffinity(0))
    except AttributeError:
        ncpu = os.cpu_count()
    return f"{name} (family {fam}, model {model}, stepping {step}; {ncpu} logical CPUs available to this process)"


def bit_identical(torch, det, weights, X):
    """Byte comparison of repeated runs and of rows across batch sizes, GEMM sweep."""
    total = same = 0
    for (K, N) in SHAPES:
        w = weights[(K, N, 0)]
        ref = torch.empty((256, N), dtype=torch.bfloat16, device=X[K].device)
        det.det_gemm_bf16(X[K], w, ref, N, K)
        for rep in range(5):
            for M in MS:
                out = torch.empty((M, N), dtype=torch.bfloat16, device=X[K].device)
                det.det_gemm_bf16(X[K][:M], w, out, N, K)
                total += 1
                same += int(torch.equal(out.view(torch.int16), ref[:M].view(torch.int16)))
    return {"rate": same / total, "comparisons": total,
            "what": "each (shape, M) output vs rows 0..M-1 of the M=256 output, 5 repeats, bytes"}


def attention_numbers(torch, det, ds, dev):
    """det_attn_decode on the config-3 grid: 32 query heads, 8 KV heads, head_dim 128, full-length
    sequences.  Algorithmic bytes = B*Hkv*L*D*2*2 (K and V once)."""
    Hq, Hkv, D = 32, 8, 128
    scale = float(np.float32(1.0 / math.sqrt(128.0)))
    rows = []
    for L in (512, 4096, 32768):
        for B in (1, 16, 64):
            base = min(B, 2)   # two distinct sequences of synthetic cache, tiled to B (all addresses distinct)
            k = ds.normal_bf16_torch(ds.tensor_seed(3, 11), (base, Hkv, L, D), 1.0, 0.0, dev).repeat(B // base, 1, 1, 1)
            v = ds.normal_bf16_torch(ds.tensor_seed(3, 12), (base, Hkv, L, D), 1.0, 0.0, dev).repeat(B // base, 1, 1, 1)
            q = ds.normal_bf16_torch(ds.tensor_seed(3, 10), (B, Hq, D), 1.0, 0.0, dev)
            lens = torch.full((B,), L, dtype=torch.int32, device=dev)
            ws = torch.empty(det.det_attn_decode_workspace_bytes(B, Hq, D, L), dtype=torch.uint8, device=dev)
            out = torch.empty((B, Hq, D), dtype=torch.bfloat16, device=dev)
            # arguments marshalled once: the binding's checks cost as much as the small cases themselves
            from paper_2602_00182_amd._lib import lib as _det_lib
            args = (q.data_ptr(), k.data_ptr(), v.data_ptr(), lens.data_ptr(), out.data_ptr(), ws.data_ptr(),
                    ws.numel(), B, Hq, Hkv, D, L, scale, torch.cuda.current_stream().cuda_stream)
            call = _det_lib().det_attn_decode
            for _ in range(2):
                if call(*args) != 0:
                    raise RuntimeError("det_attn_decode failed")
            torch.cuda.synchronize()
            n = 20 if B * L <= 64 * 4096 else 5
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(n):
                call(*args)
            e1.record()
            torch.cuda.synchronize()
            us = e0.elapsed_time(e1) / n * 1e3
            by = B * Hkv * L * D * 2 * 2
            rows.append({"B": B, "L": L, "us": round(us, 1), "gbs": round(by / us / 1e3, 1),
                         "frac_hbm": round(by / us / 1e3 / PEAK_HBM_GBS, 4), "kv_mb": round(by / 1e6, 1)})
            del k, v, ws
            torch.cuda.empty_cache()
    return rows


def qgemm_numbers(torch, det, ds, dev):
    """Block-quantized GEMM (4-bit weights, 8-bit activations) on the same shapes, weights rotating over
    3 packed sets (HBM-cold).  us = det_qgemm_w4a8 alone, us_quant = det_quant_act_q8 of the M rows;
    bytes = packed weights (4.25 bits each) + activation codes and scales + bf16 output."""
    rows = []
    for (K, N) in SHAPES + [(2048, 32000)]:
        packs = [det.quant_pack_weight(ds.normal_bf16_torch(ds.tensor_seed(7, 10 * s + 1), (K, N), 0.02, 0.0, dev))
                 for s in range(3)]
        x = ds.normal_bf16_torch(ds.tensor_seed(7, 2), (256, K), 1.0, 0.0, dev)
        c = torch.empty((256, N), dtype=torch.bfloat16, device=dev)
        from paper_2602_00182_amd._lib import lib as _det_lib
        L = _det_lib()
        stream = torch.cuda.current_stream().cuda_stream
        for M in (1, 16, 64, 256):
            codes, scales = det.quant_activations(x[:M])
            ga = [(codes.data_ptr(), scales.data_ptr(), p.data_ptr(), c.data_ptr(), N, M, N, K, 0, stream) for p in packs]
            qa = (x.data_ptr(), K, codes.data_ptr(), scales.data_ptr(), M, K, stream)
            for i in range(3):
                L.det_qgemm_w4a8(*ga[i])
            torch.cuda.synchronize()
            e0, e1, e2 = (torch.cuda.Event(enable_timing=True) for _ in range(3))
            e0.record()
            for i in range(12):
                L.det_qgemm_w4a8(*ga[i % 3])
            e1.record()
            for i in range(12):
                L.det_quant_act_q8(*qa)
            e2.record()
            torch.cuda.synchronize()
            us, usq = e0.elapsed_time(e1) / 12 * 1e3, e1.elapsed_time(e2) / 12 * 1e3
            by = det.det_qgemm_packed_w_bytes(N, K) + M * K + 4 * M * (K // 64) + 2 * M * N
            rows.append({"K": K, "N": N, "M": M, "us": round(us, 1), "us_quant": round(usq, 1),
                         "gbs": round(by / us / 1e3, 1), "tflops": round(gemm_flops(M, N, K) / us / 1e6, 1),
                         "packed_mb": round(det.det_qgemm_packed_w_bytes(N, K) / 1e6, 1)})
        del packs
        torch.cuda.empty_cache()
    return rows


def decode_numbers(torch, det, ds, dev):
    """Decoder layer (Llama-3-8B shape, context 2048) and 8-layer model step, tokens/s."""
    from paper_2602_00182_amd.decode import DecodeModel, ModelCfg

    out = {}
    H, Hq, Hkv, D, F, Lmax = 4096, 32, 8, 128, 14336, 2048
    scale = float(np.float32(1.0 / math.sqrt(128.0)))
    s = ds.tensor_seed(4, 0)
    g = lambda i, shape, std=0.02, mean=0.0: ds.normal_bf16_torch(s + i, shape, std, mean, dev)
    packed = [g(0, (H,), 0.0, 1.0), det.pack_qkv(g(1, (H, (Hq + 2 * Hkv) * D)), Hq, Hkv, D), det.pack_weight(g(2, (Hq * D, H))),
              g(3, (H,), 0.0, 1.0), det.pack_gate_up(g(4, (H, 2 * F))), det.pack_weight(g(5, (F, H)))]
    struct = det.layer_weights(*packed)
    # the same layer with 4-bit weights and 8-bit activations (det_qdecoder_layer)
    qpacked = [packed[0], det.quant_pack_qkv(g(1, (H, (Hq + 2 * Hkv) * D)), Hq, Hkv, D), det.quant_pack_weight(g(2, (Hq * D, H))),
               packed[3], det.quant_pack_gate_up(g(4, (H, 2 * F))), det.quant_pack_weight(g(5, (F, H)))]
    qstruct = det.layer_weights(*qpacked)
    qwbytes = float(sum(t.numel() * t.element_size() for t in qpacked))
    cfg = det.layer_cfg(H, Hq, Hkv, D, F, Lmax, 1e-5, scale)
    cos_t, sin_t = ds.rope_tables(Lmax, D, 5.0e5)
    cos_d, sin_d = torch.from_numpy(cos_t).to(dev), torch.from_numpy(sin_t).to(dev)
    wbytes = 2.0 * (H * (Hq + 2 * Hkv) * D + Hq * D * H + H * 2 * F + F * H)
    layer_rows, qlayer_rows = [], []
    for B in (1, 32, 128):
        x = ds.normal_bf16_torch(s + 50, (B, H), 1.0, 0.0, dev)
        kc = ds.normal_bf16_torch(s + 51, (B, Hkv, Lmax, D), 1.0, 0.0, dev)
        vc = ds.normal_bf16_torch(s + 52, (B, Hkv, Lmax, D), 1.0, 0.0, dev)
        pos = torch.full((B,), Lmax - 1, dtype=torch.int32, device=dev)
        for quantized, rows_out, wb in ((False, layer_rows, wbytes), (True, qlayer_rows, qwbytes)):
            if quantized:
                ws = torch.empty(det.det_qdecoder_layer_workspace_bytes(cfg, B), dtype=torch.uint8, device=dev)
                call = lambda: det.det_qdecoder_layer(qstruct, cfg, x, kc, vc, pos, None, cos_d, sin_d, ws)
            else:
                ws = torch.empty(det.det_decoder_layer_workspace_bytes(cfg, B), dtype=torch.uint8, device=dev)
                call = lambda: det.det_decoder_layer(struct, cfg, x, kc, vc, pos, cos_d, sin_d, ws)
            for _ in range(3):
                call()
            torch.cuda.synchronize()
            n = 20
            t0 = time.perf_counter()
            for _ in range(n):
                call()
            torch.cuda.synchronize()
            dt = (time.perf_counter() - t0) / n
            by = wb + B * Hkv * Lmax * D * 2 * 2
            rows_out.append({"B": B, "context": Lmax, "us_per_layer": round(dt * 1e6, 1),
                             "layer_tokens_per_s": round(B / dt, 1), "gbs": round(by / dt / 1e9, 1),
                             "frac_hbm": round(by / dt / 1e9 / PEAK_HBM_GBS, 4)})
            del ws
        del x, kc, vc
    out["decoder_layer"] = layer_rows
    out["decoder_layer_w4a8"] = qlayer_rows
    del packed, struct, qpacked, qstruct
    torch.cuda.empty_cache()

    H, Hq, Hkv, D, F, V, NL = 2048, 16, 4, 128, 5632, 32000, 8
    s = ds.tensor_seed(5, 0)
    g = lambda i, shape, std=0.02, mean=0.0: ds.normal_bf16_torch(s + i, shape, std, mean, dev)
    layers = []
    for l in range(NL):
        o = 10 + 10 * l
        layers.append(dict(norm1=g(o, (H,), 0.0, 1.0), wqkv=g(o + 1, (H, (Hq + 2 * Hkv) * D)), wo=g(o + 2, (Hq * D, H)),
                           norm2=g(o + 3, (H,), 0.0, 1.0), wgu=g(o + 4, (H, 2 * F)), wdown=g(o + 5, (F, H))))
    weights = dict(embed=g(1, (V, H), 1.0), lm_head=g(2, (H, V)), final_norm=g(3, (H,), 0.0, 1.0), layers=layers)
    models = (("model_8_layer_step", DecodeModel(ModelCfg(H, Hq, Hkv, D, F, V, NL), weights)),
              ("model_8_layer_step_w4a8", DecodeModel(ModelCfg(H, Hq, Hkv, D, F, V, NL), weights, quantized=True)))
    Lm = 640
    cos_t, sin_t = ds.rope_tables(Lm, D, 5.0e5)
    cos_d, sin_d = torch.from_numpy(cos_t).to(dev), torch.from_numpy(sin_t).to(dev)
    for key, model in models:
        rows = []
        for B in (1, 8, 64):
            st = model.new_state(B, Lm, cos_d, sin_d)
            st.tokens.copy_(torch.from_numpy(ds.uniform_int(s + 900, (B,), 0, V - 1)).to(dev))
            idx = torch.empty(B, dtype=torch.int32, device=dev)
            for k in st.kcache + st.vcache:
                k.copy_(ds.normal_bf16_torch(s + 901, tuple(k.shape), 1.0, 0.0, dev))
            st.positions.fill_(511)
            for _ in range(3):
                st.forward()
                det.det_argmax(st.logits, idx)
            torch.cuda.synchronize()
            n = 30
            t0 = time.perf_counter()
            for _ in range(n):
                st.forward()
                det.det_argmax(st.logits, idx)
            torch.cuda.synchronize()
            dt = (time.perf_counter() - t0) / n
            rows.append({"B": B, "context": 512, "ms_per_step": round(dt * 1e3, 3), "tokens_per_s": round(B / dt, 1)})
            del st
        out[key] = rows
    # the whole config-5 job: 64 prompts of 16..512 tokens, 128 new tokens each, greedy, one batch:
    # one-pass prefill, then 127 decode steps (generated tokens per second of wall time, job total)
    from paper_2602_00182_amd.decode import prefill_decode
    lens = ds.uniform_int(ds.tensor_seed(5, 500), (64,), 16, 512)
    toks = ds.uniform_int(ds.tensor_seed(5, 501), (64, 512), 0, V - 1)
    toks_d, lens_d = torch.from_numpy(toks).to(dev), torch.from_numpy(lens).to(dev)
    for key, model in models:
        prefill_decode(model, toks_d[:4], lens_d[:4], 4, cos_d, sin_d)
        torch.cuda.synchronize()
        runs = []
        for _ in range(3):   # every run is reported: the job is short enough for host jitter to show
            t0 = time.perf_counter()
            gen, _ = prefill_decode(model, toks_d, lens_d, 128, cos_d, sin_d)
            torch.cuda.synchronize()
            runs.append(time.perf_counter() - t0)
        dt = float(np.median(runs))
        out["job_64_prompts" + key[len("model_8_layer_step"):]] = {
            "prompts": 64, "prompt_tokens": int(lens.sum()), "new_tokens": 64 * 128, "seconds": round(dt, 4),
            "seconds_each_run": [round(r, 4) for r in runs], "reported": "median of the runs",
            "generated_tokens_per_s": round(64 * 128 / dt, 1)}
    return out


if __name__ == "__main__":
    main()
