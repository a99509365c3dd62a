#!/usr/bin/env python3
"""Streaming decode benchmark of FlashDecoder-XL on one MI355X.

A step is one fd_decode_chunk call: one latent frame of the 720p stream
(16 x 90 x 160 latents -> 4 RGB frames of 720 x 1280) through the whole hot
path (embedding, 20 backbone blocks, temporal upsampling, 2 refinement blocks,
pixel head). Streams are 32 chunks long (the cache is reset every 32 steps);
inputs are seeded synthetic latents and N(0, 0.02) weights, resident in HBM
before timing starts. Prints one JSON line.

  python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload NAME]
  python bench.py --copy-calibration MIB   (plain device copy of MIB MiB, for
                                            scaling HBM byte counters)
  python bench.py --cpu-baselines          (the CPU oracle timed in full on the tiny
                                            workloads and per steady stream call)
  python bench.py --trace-gaps CSV         (idle time between a call's kernels in a
                                            rocprofv3 kernel trace of this script)
  python bench.py --reference-probes       (the GPU's LDS read bandwidth and the
                                            rate of torch.matmul on the decoder's
                                            720p GEMM shapes, as context for the
                                            GEMM kernels' roofline)

The roofline's "traffic" (HBM bytes per launch of the roofline kernel) comes
from two rocprofv3 counter passes (FETCH_SIZE, WRITE_SIZE) over this script,
scaled by what the same counters read for the plain copy; the figures are kept
in profiles/ together with the SHA-256 of the kernel source they were taken on,
and reported only while that source is unchanged.
"""
from __future__ import annotations

import argparse
import json
import os
import platform
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_F16_TFLOPS = 2500.0   # MI355X dense fp16 / bf16 MFMA
PEAK_HBM_GBS = 8000.0      # MI355X HBM3E
TRAFFIC_FILE = os.path.join(ROOT, "profiles", "attn_refine_xl720p_traffic.md")
ATTN_SOURCE = os.path.join(ROOT, "paper_2607_14898_amd", "csrc", "k_attn.hip")
METRIC = "decoded frames/sec at 720p (latent->pixel), p50 per-chunk latency, % MFMA peak"


def _cpu_model() -> str:
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return platform.processor() or platform.machine()


def _blas_threads() -> int:
    try:
        from threadpoolctl import threadpool_info
        return max([d.get("num_threads", 1) for d in threadpool_info() if d.get("user_api") == "blas"] or [1])
    except Exception:
        return os.cpu_count() or 1


def time_oracle(wl, weights, n_calls):
    """Wall time of the CPU oracle (fp32, numpy with the host's BLAS threads)
    decoding the first n_calls calls of workload wl, and the frames it emits."""
    import numpy as np
    from oracle.decoder import StreamingOracle
    m = wl.model
    z = wl.latents()
    F = wl.frames_per_call
    t0 = time.perf_counter()
    for b in range(z.shape[0]):
        dec = StreamingOracle(m, weights, np.float32)
        for c in range(n_calls):
            dec.decode(z[b, :, c * F:(c + 1) * F])
    dt = time.perf_counter() - t0
    return dt, z.shape[0] * n_calls * F * m.r_t


def time_oracle_steady_chunk(wl, weights, rf_frac=5):
    """CPU seconds of one steady call (one latent frame, the window full) of a
    one-frame-per-call stream, from the fp32 oracle timed on parts of it:
    backbone block 0 in full (all queries against the two visible frames'
    keys) counted once per backbone block; refinement block 0 for 1/rf_frac
    of the call's queries (against all visible keys) counted rf_frac times per
    refinement block; the latent projection, temporal upsampling and pixel
    head in full. Returns (seconds, measured seconds, description)."""
    import numpy as np
    import oracle.decoder as od
    m = wl.model
    L, r = m.tokens_per_frame, m.r_t
    W = {k: np.asarray(v, np.float32) for k, v in weights.items()
         if k.startswith(("embed.", "bb.0.", "rf.0.", "bb.norm_f", "rf.norm_f", "tup.", "head"))}
    z = wl.latents()[0, :, :2].astype(np.float32)
    meas = 0.0
    t = time.perf_counter()
    x = [od.pixel_unshuffle_frame(z[:, c], m.patch) @ W["embed.w"].T + W["embed.b"] for c in (0, 1)]
    t_embed = (time.perf_counter() - t) / 2
    pos_k = np.concatenate([od.token_positions(m, [c]) for c in (0, 1)])
    t = time.perf_counter()
    y_bb = od.block_forward_rows(m, W, "bb.0", np.concatenate(x), pos_k, x[1], od.token_positions(m, [1]))
    t_bb = time.perf_counter() - t
    # refinement inputs: the temporal upsampling of both frames' (block-0) states
    t = time.perf_counter()
    xr = [od.temporal_up_rows(m, W, od.stack_final(m, W, "bb", xc)).transpose(1, 0, 2).reshape(r * L, m.dim)
          for xc in (x[0], y_bb)]
    t_tup = (time.perf_counter() - t) / 2
    rows = np.arange(0, r * L, rf_frac)
    rpos_k = np.concatenate([od.token_positions(m, [r * c + j for j in range(r)]) for c in (0, 1)])
    rpos_q = od.token_positions(m, [r + j for j in range(r)])[rows]
    t = time.perf_counter()
    y_rf = od.block_forward_rows(m, W, "rf.0", np.concatenate(xr), rpos_k, xr[1][rows], rpos_q)
    t_rf = time.perf_counter() - t
    t = time.perf_counter()
    od.head_rows(m, W, od.stack_final(m, W, "rf", y_rf))
    t_head = time.perf_counter() - t
    meas = 2 * t_embed + t_bb + 2 * t_tup + t_rf + t_head
    total = (t_embed + m.n_backbone_blocks * t_bb + t_tup +
             rf_frac * (m.n_refine_blocks * t_rf + t_head))
    desc = (f"one steady call of the {wl.name} stream from the fp32 numpy oracle timed on its parts: "
            f"backbone block 0 in full ({t_bb:.2f} s) x {m.n_backbone_blocks} blocks, refinement block 0 on "
            f"1/{rf_frac} of the {r * L} queries against all {2 * r * L} keys ({t_rf:.2f} s) x {rf_frac} x "
            f"{m.n_refine_blocks} blocks, pixel head on the same rows ({t_head:.2f} s) x {rf_frac}, latent "
            f"projection and temporal upsampling in full; {meas:.1f} s measured")
    return total, meas, desc


def cpu_baseline(wl, weights):
    """The CPU oracle on a bounded sample of the same workload (one steady
    call, timed on parts of it), scaled to frames per second."""
    sec, _, desc = time_oracle_steady_chunk(wl, weights)
    frames = wl.frames_per_call * wl.model.r_t
    return {"value": round(frames / sec, 5), "unit": "frames/s", "cores": int(_blas_threads()),
            "kind": "oracle", "sample": desc, "cpu": _cpu_model()}


def cpu_baselines() -> int:
    """The oracle (fp32) timed in full on the tiny workloads, and per steady
    call of the streams from timed parts (one JSON line each)."""
    from paper_2607_14898_amd.workloads import WORKLOADS
    for name in ("tiny", "tiny-asis"):
        wl = WORKLOADS[name]
        dt, frames = time_oracle(wl, wl.weights(), wl.n_calls)
        print(json.dumps({"workload": name, "calls": wl.n_calls, "frames": frames, "seconds": round(dt, 3),
                          "frames_per_s": round(frames / dt, 3), "timed": "in full", "dtype": "f32",
                          "blas_threads": _blas_threads(), "cpu": _cpu_model()}), flush=True)
    for name in ("xl-480p-stream", "xl-720p-stream"):
        wl = WORKLOADS[name]
        sec, meas, desc = time_oracle_steady_chunk(wl, wl.weights())
        frames = wl.frames_per_call * wl.model.r_t
        print(json.dumps({"workload": name, "seconds_per_call": round(sec, 1),
                          "frames_per_s": round(frames / sec, 5), "timed": desc, "dtype": "f32",
                          "blas_threads": _blas_threads(), "cpu": _cpu_model()}), flush=True)
    return 0


def trace_gaps(path: str, warmup: int, steps: int) -> int:
    """Idle time between the kernels of each timed decode call in a rocprofv3
    kernel trace (--kernel-trace --output-format csv) of this script run with
    the same --warmup and --steps: per call, from the prologue (the latent
    unshuffle) to the pixel-store GEMM, the wall span against the union of kernel intervals.
    Host-only; prints one JSON line."""
    import csv
    import numpy as np
    ks = sorted((int(r["Start_Timestamp"]), int(r["End_Timestamp"]), r["Kernel_Name"])
                for r in csv.DictReader(open(path)))
    starts = [i for i, k in enumerate(ks) if "prologue_kernel" in k[2]]
    calls = []
    for a, b in zip(starts, starts[1:] + [len(ks)]):
        seg = ks[a:b]
        ends = [i for i, k in enumerate(seg) if "Li7EEEv" in k[2]]  # the EPI_PIXEL GEMM
        if not ends:
            continue
        seg = seg[:ends[-1] + 1]
        busy, cs, ce = 0, None, None
        for s0, e0, _ in seg:
            if ce is None or s0 > ce:
                if ce is not None:
                    busy += ce - cs
                cs, ce = s0, e0
            else:
                ce = max(ce, e0)
        busy += ce - cs
        gaps = [seg[i + 1][0] - seg[i][1] for i in range(len(seg) - 1)]
        calls.append((seg[-1][1] - seg[0][0], busy, len(seg), float(np.median(gaps)), max(gaps)))
    c = np.array(calls[warmup:warmup + steps])   # the timed calls follow the warmup ones
    span, busy = c[:, 0].mean() / 1e3, c[:, 1].mean() / 1e3
    print(json.dumps({"calls": len(c), "kernels_per_call": round(float(c[:, 2].mean()), 1),
                      "span_us": round(span, 1), "busy_us": round(busy, 1), "idle_us": round(span - busy, 1),
                      "idle_frac": round((span - busy) / span, 5), "median_gap_us": round(float(np.median(c[:, 3])) / 1e3, 2),
                      "max_gap_us": round(float(c[:, 4].max()) / 1e3, 1)}), flush=True)
    return 0


def counter_traffic():
    """HBM bytes per launch of the refinement attention from the committed
    counter summary, or None if it is missing or was taken on other source."""
    import hashlib
    try:
        fields = {}
        for line in open(TRAFFIC_FILE):
            if line.startswith("    ") and ":" in line:
                k, v = line.strip().split(":", 1)
                fields[k.strip()] = v.strip()
        src = hashlib.sha256(open(ATTN_SOURCE, "rb").read()).hexdigest()
        if fields.get("kernel_source_sha256") != src:
            return None
        return int(fields["hbm_bytes_per_launch"])
    except (OSError, KeyError, ValueError):
        return None


def copy_calibration(mib: int) -> int:
    """A plain device-to-device copy of known size: the reference for scaling
    the FETCH_SIZE / WRITE_SIZE counters."""
    import torch
    n = mib * (1 << 20) // 4
    src = torch.ones(n, dtype=torch.float32, device="cuda")
    dst = torch.empty_like(src)
    for _ in range(3):
        dst.copy_(src)
    torch.cuda.synchronize()
    print(json.dumps({"copy_calibration_bytes": n * 4, "launches": 3}), flush=True)
    return 0


# (M, N, K) of the decoder's projections at the 720p stream shapes: backbone
# QKV, O, gate/up, down; temporal upsampling; refinement QKV, O, gate/up, down;
# pixel head layers 1 and 2
GEMM_SHAPES_720P = [
    ("bb.qkv", 3600, 1920, 1536), ("bb.o", 3600, 1536, 1536), ("bb.w13", 3600, 12288, 1536),
    ("bb.w2", 3600, 1536, 6144), ("tup", 3600, 6144, 1536), ("rf.qkv", 14400, 1920, 1536),
    ("rf.o", 14400, 1536, 1536), ("rf.w13", 14400, 12288, 1536), ("rf.w2", 14400, 1536, 6144),
    ("head1", 14400, 6144, 1536), ("head2", 14400, 768, 6144)]


def reference_probes() -> int:
    """LDS bandwidth of a compute unit (fd_measure_lds_bandwidth), the overlap of
    MFMAs and vector instructions (fd_measure_issue_overlap), and torch.matmul
    (the vendor BLAS) on the decoder's GEMM shapes with random fp16 operands: a
    reference point for the library's own GEMM kernels, never used by them."""
    import torch
    from paper_2607_14898_amd import flashdecoder as fdb
    bpc, ghz = fdb.fd_measure_lds_bandwidth(20000)
    print(json.dumps({"probe": "lds_read_bandwidth", "bytes_per_clock_per_cu": round(bpc, 1),
                      "clock_ghz": round(ghz, 3)}), flush=True)
    for wps in (1, 2):
        cyc = fdb.fd_measure_issue_overlap(wps, 20000)
        print(json.dumps({"probe": "issue_overlap", "waves_per_simd": wps,
                          "cycles_per_slot": {k: round(v, 1) for k, v in cyc.items()}}), flush=True)
    torch.manual_seed(0)
    for name, M, N, K in GEMM_SHAPES_720P:
        a = (torch.randn(M, K, device="cuda") * 0.5).half()
        w = (torch.randn(N, K, device="cuda") * 0.02).half()
        for _ in range(3):
            torch.matmul(a, w.t())
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        reps = 20
        e0.record()
        for _ in range(reps):
            torch.matmul(a, w.t())
        e1.record()
        torch.cuda.synchronize()
        us = e0.elapsed_time(e1) * 1e3 / reps
        tf = 2.0 * M * N * K / (us * 1e-6) / 1e12
        print(json.dumps({"probe": "torch_matmul_f16", "gemm": name, "M": M, "N": N, "K": K,
                          "us": round(us, 2), "tflops": round(tf, 1),
                          "frac_of_2500": round(tf / PEAK_F16_TFLOPS, 3)}), flush=True)
    return 0


def main() -> int:
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=64)
    ap.add_argument("--warmup", type=int, default=8)
    ap.add_argument("--workload", default="xl-720p-stream")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--copy-calibration", type=int, metavar="MIB")
    ap.add_argument("--reference-probes", action="store_true")
    ap.add_argument("--trace-gaps", metavar="CSV",
                    help="idle time between a decode call's kernels in a rocprofv3 kernel trace (host only)")
    ap.add_argument("--cpu-baselines", action="store_true",
                    help="time the CPU oracle on the tiny workloads and per steady stream call")
    ap.add_argument("--streams", type=int, default=1,
                    help="independent streams decoded concurrently per step (fd_decode_chunks)")
    ap.add_argument("--pixels", choices=["f32", "bf16", "u8"], default="f32",
                    help="pixel format of the output store")
    args = ap.parse_args()
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py measures one GPU only: this build has no multi-GPU path "
              "(see DESIGN.md for how the decoder would shard); run with --gpus 1.",
              file=sys.stderr)
        return 2
    if args.copy_calibration:
        return copy_calibration(args.copy_calibration)
    if args.reference_probes:
        return reference_probes()
    if args.trace_gaps:
        return trace_gaps(args.trace_gaps, args.warmup, args.steps)
    if args.cpu_baselines:
        return cpu_baselines()

    import numpy as np
    import torch

    from paper_2607_14898_amd import flashdecoder as fdb
    from paper_2607_14898_amd.flops import call_flops
    from paper_2607_14898_amd.workloads import WORKLOADS

    wl = WORKLOADS[args.workload]
    m = wl.model
    F = wl.frames_per_call
    weights = wl.weights()
    fmt = {"f32": fdb.FD_PIXELS_F32, "bf16": fdb.FD_PIXELS_BF16, "u8": fdb.FD_PIXELS_U8}[args.pixels]
    NS = args.streams
    if NS < 1:
        print("--streams must be >= 1", file=sys.stderr)
        return 2
    dec = fdb.Decoder(m, weights, max_batch=1, max_frames_per_call=F)
    caches = [fdb.KvCache(dec, 1) for _ in range(NS)]
    cache = caches[0]
    z = torch.from_numpy(wl.latents()).cuda()
    chunks = [z[:, :, i * F:(i + 1) * F].contiguous() for i in range(wl.n_calls)]
    outs = [torch.empty(dec.output_shape(1, F), dtype=fdb.pixel_torch_dtype(fmt), device="cuda")
            for _ in range(NS)]
    out = outs[0]
    # stream i starts i * n_calls / NS chunks into the sequence, so the
    # concurrent streams sit at different positions
    pos = [i * wl.n_calls // NS for i in range(NS)]

    def step():
        js = []
        for i in range(NS):
            j = pos[i] % wl.n_calls
            if j == 0:
                caches[i].reset()
            js.append(j)
            pos[i] += 1
        if NS == 1 and fmt == fdb.FD_PIXELS_F32:
            cache.decode_chunk(chunks[js[0]], out)
        elif NS == 1:
            cache.decode_chunk(chunks[js[0]], out, out_format=fmt)
        else:
            fdb.decode_chunks(caches, [chunks[j] for j in js], outs, out_format=fmt)
        return js

    calib_note = None
    if getattr(m, "mlp_precision", "f16") == "fp8s":
        # static-calibrated FP8: maxima of the stream's first chunks, before timing
        amax = np.zeros(fdb.fd_fp8_act_count(dec.handle), np.float32)
        n_cal = min(4, wl.n_calls)
        cal_out = torch.empty(dec.output_shape(1, F), dtype=torch.float32, device="cuda")
        for j in range(n_cal):
            fdb.fd_calibrate_chunk(dec.handle, chunks[j], F, cache.handle, cal_out, amax)
        fdb.fd_set_fp8_act_amax(dec.handle, amax)
        cache.reset()
        calib_note = f"static FP8 amplitudes calibrated on the stream's first {n_cal} chunks"

    for i in range(NS):   # bring every stream to its start position
        for j in range(pos[i]):
            caches[i].decode_chunk(chunks[j], outs[i], out_format=fmt)

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()

    K = args.steps
    ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
          for _ in range(K)]
    fdb.fd_probe_enable(cache.handle, fdb.FD_KC_ATTENTION_REFINE)
    flops = 0.0
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for i in range(K):
        ev[i][0].record()
        js = step()
        ev[i][1].record()
        for j in js:
            g, a = call_flops(m, F, j * F)
            flops += g + a
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    attn_ms, attn_n, attn_work = fdb.fd_probe_read(cache.handle)
    fdb.fd_probe_enable(cache.handle, -1)
    if fmt != fdb.FD_PIXELS_U8:
        assert not any(torch.isnan(o.float()).any().item() for o in outs), "NaN in decoded pixels"

    wall = t1 - t0
    lat = np.array([a.elapsed_time(b) for a, b in ev])

    # per kernel class, after the timed region: device time of every launch of
    # the class (events on the decode stream) against its algorithmic work
    # (2 M N K flops per GEMM, 4 N L_q L_k D_h per attention, bytes read and
    # written per norm / latent unshuffle pass)
    n_probe = max(4, min(16, K))
    kclasses = {}
    for cname, kcl, flops_kind in (("gemm", fdb.FD_KC_GEMM, True), ("attention", fdb.FD_KC_ATTENTION, True),
                                   ("norm", fdb.FD_KC_NORM, False), ("embed_in", fdb.FD_KC_EMBED_IN, False)):
        fdb.fd_probe_enable(cache.handle, kcl)
        for _ in range(n_probe):
            step()
        torch.cuda.synchronize()
        c_ms, c_n, c_work = fdb.fd_probe_read(cache.handle)
        fdb.fd_probe_enable(cache.handle, -1)
        if c_n == 0:
            continue
        ach = c_work / (c_ms * 1e-3) / (1e12 if flops_kind else 1e9)
        pk = PEAK_F16_TFLOPS if flops_kind else PEAK_HBM_GBS
        kclasses[cname] = {
            "bound": "mfma" if flops_kind else "hbm", "unit": "TFLOP/s" if flops_kind else "GB/s",
            "achieved": round(ach, 1), "peak": pk, "frac": round(ach / pk, 4),
            "launches_per_chunk": round(c_n / n_probe, 2), "ms_per_chunk": round(c_ms / n_probe, 4)}
    # sustained dense MFMA throughput of this GPU (after the timed region)
    peak_meas, peak_ghz = fdb.fd_measure_mfma_peak("f16", 100000)
    for v in kclasses.values():
        if v["bound"] == "mfma":
            v["frac_of_measured_peak"] = round(v["achieved"] / peak_meas, 4)
    frames = K * F * m.r_t * NS
    fp8 = getattr(m, "mlp_precision", "f16") in ("fp8", "fp8s")
    achieved = attn_work / (attn_ms * 1e-3) / 1e12
    result = {
        "metric": METRIC,
        "value": round(frames / wall, 3),
        "unit": "frames/s",
        "n_gpus": 1,
        "steps": K,
        "warmup": args.warmup,
        "ms_per_step": round(wall * 1e3 / K, 4),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": (m.compute_dtype + "+fp8") if fp8 else m.compute_dtype,
        "data": "synthetic",
        "config": {
            "workload": wl.name,
            "model": "FlashDecoder-XL (D=1536, 20+2 blocks, 24 heads, 3 KV groups, SwiGLU 6144)",
            "latent_per_chunk": f"{m.latent_channels}x{F}x{m.latent_h}x{m.latent_w}",
            "pixels_per_chunk": f"3x{F * m.r_t}x{m.out_h}x{m.out_w}",
            "chunks_per_stream": wl.n_calls,
            "concurrent_streams": NS,
            "pixel_format": args.pixels,
            "mlp_gemms": ("E4M3 x E4M3 (static per-tensor / per-channel scales)" if m.mlp_precision == "fp8s" else
                          "E4M3 x E4M3 (per-token / per-channel scales)") if fp8 else "fp16",
            "calibration": calib_note,
            "window": m.window,
            "p50_chunk_ms": round(float(np.percentile(lat, 50)), 4),
            "p99_chunk_ms": round(float(np.percentile(lat, 99)), 4),
            "mfma_frac_overall": round(flops / wall / 1e12 / PEAK_F16_TFLOPS, 4),
            "mfma_frac_overall_of_measured_peak": round(flops / wall / 1e12 / peak_meas, 4),
            "algorithmic_tflop_per_step": round(flops / K / 1e12, 4),
            "operands": f"{m.compute_dtype} MFMA operands (bf16-rounded weights/latents), fp32 accumulate",
            "paper_context": "76.1 frames/s, FlashDecoder-XL Wan2.1 720p streaming, 1x H100 (Table 2)",
        },
        "kernel_classes": kclasses,
        "roofline": {
            "kernel": "attn_mfma_kernel<f16, 4 heads, 32 queries/wave> (refinement-stack attention)",
            "bound": "mfma",
            "achieved": round(achieved, 2),
            "peak": PEAK_F16_TFLOPS,
            "unit": "TFLOP/s",
            "frac": round(achieved / PEAK_F16_TFLOPS, 4),
            "traffic": counter_traffic(),
            "measured_peak": round(peak_meas, 1),
            "measured_peak_clock_ghz": round(peak_ghz, 3),
            "frac_of_measured_peak": round(achieved / peak_meas, 4),
            "measured_peak_kind": "sustained f16 32x32x16 MFMA loop, 2 workgroups x 4 waves per CU, "
                                  "changing operands (fd_measure_mfma_peak)",
            "launches": attn_n,
            "avg_launch_us": round(attn_ms * 1e3 / max(attn_n, 1), 2),
        },
    }
    if not args.no_cpu_baseline:
        result["cpu_baseline"] = cpu_baseline(wl, weights)
    print(json.dumps(result), flush=True)
    for c in caches:
        c.close()
    dec.close()
    return 0


if __name__ == "__main__":
    sys.exit(main())
