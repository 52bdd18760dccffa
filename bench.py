#!/usr/bin/env python3
"""Throughput of the MI355X Viterbi decoder on its headline workload.

Workload: 4096 zero-terminated frames x 8192 info bits, K=7 (133,171) rate
1/2, BPSK over AWGN (seeded), soft values already resident in HBM.
A step decodes the whole batch: forward procedure (branch metrics,
add-compare-select, packed survivor decisions) plus traceback.

  value      int8 soft values, radix-4 forward (decoded info Gbit/s)
  variants   the same for float32 radix-2 and int8 radix-2
  roofline   the forward kernel of the headline variant against the vector
             ALU peak at the kernel's data width (packed 16-bit for the int8
             radix-4 kernel): 3 ops per state per stage (add, add,
             compare-select); traffic = HBM bytes per launch from the
             committed counter summary when its kernel source is unchanged
  cpu_baseline  the CPU oracle (exact integers) on the host cores

Prints one JSON line.  --ber adds the equal-BER sweep (0..6 dB).
"""
from __future__ import annotations

import argparse
import hashlib
import json
import math
import os
import re
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "decoded info Gbit/s on 1 MI355X (K=7 r1/2), int8 radix-4 vs fp32 radix-2, at equal BER"
N_FRAMES, N_INFO = 4096, 8192
CUS, LANES, CLOCK_HZ = 256, 64, 2.4e9
VALU32_PEAK_TOPS = CUS * LANES * CLOCK_HZ / 1e12  # 39.32 T lane-ops/s
VALU16_PEAK_TOPS = 2 * VALU32_PEAK_TOPS           # packed 16-bit: 78.64 T ops/s
COPY_BYTES = 512 << 20
# forward kernels whose HBM traffic was counted: profile summary and sources
TRAFFIC_PROFILES = {
    "i8r4": ("fwd_r4q_k7_4096x8192_traffic.md", ["mivit_r4p.hip", "mivit_device.h"]),
    "f32r2": ("fwd_rot_k7_4096x8192_traffic.md", ["mivit_fwd_rot.h", "mivit_device.h"]),
}
# data width of the add-compare-select of each variant's forward kernel
PACKED16 = {"i8r4"}


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=200)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--ebn0", type=float, default=3.0)
    ap.add_argument("--no-cpu", action="store_true", help="skip the CPU-oracle baseline")
    ap.add_argument("--ber", action="store_true", help="run the equal-BER sweep")
    ap.add_argument("--variants", default="i8r4,f32r2,f16r2,i8r2,i8r8")
    ap.add_argument("--configs", action="store_true",
                    help="also measure the single-frame, stream, mixed-batch and backward workloads")
    ap.add_argument("--pcie", action="store_true",
                    help="also time the host pipeline (page-locked host memory in and out)")
    ap.add_argument("--copy-probe", action="store_true",
                    help="also run one device copy of %d MiB (scale for HBM counters)" % (COPY_BYTES >> 20))
    return ap.parse_args()


def source_digest(files):
    h = hashlib.sha256()
    for f in files:
        with open(os.path.join(ROOT, "paper_2011_13579_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def measured_traffic(variant):
    """HBM bytes per forward launch from the committed counter summary, or
    None when the kernel source changed since the counters were taken."""
    prof, files = TRAFFIC_PROFILES.get(variant, (None, None))
    if prof is None:
        return None
    path = os.path.join(ROOT, "profiles", prof)
    if not os.path.exists(path):
        return None
    fields = {}
    with open(path) as fh:
        for ln in fh:
            m = re.match(r"^- (\w+): (\S+)", ln.strip())
            if m:
                fields[m.group(1)] = m.group(2)
    if fields.get("source_sha256") != source_digest(files):
        return None
    try:
        return int(fields["hbm_bytes_per_launch"])
    except (KeyError, ValueError):
        return None


def time_variant(torch, mv, plan, llr, steps, warmup):
    dev = llr.device
    bits, metric, end = plan.empty_outputs(dev)
    st = torch.cuda.current_stream()
    for _ in range(warmup):
        plan.forward(llr, metric, end)
        plan.traceback(bits)
    torch.cuda.synchronize()
    # events on the launch stream: a[k] before step k's forward, b[k] between
    # its forward and traceback; a[steps] closes the last step
    a = [torch.cuda.Event(enable_timing=True) for _ in range(steps + 1)]
    b = [torch.cuda.Event(enable_timing=True) for _ in range(steps)]
    t0 = time.perf_counter()
    for k in range(steps):
        a[k].record(st)
        plan.forward(llr, metric, end)
        b[k].record(st)
        plan.traceback(bits)
    a[steps].record(st)
    torch.cuda.synchronize()
    wall = (time.perf_counter() - t0) / steps
    fwd = float(np.mean([a[k].elapsed_time(b[k]) for k in range(steps)]))
    tb = float(np.mean([b[k].elapsed_time(a[k + 1]) for k in range(steps)]))
    return wall * 1e3, fwd, tb, bits, metric


def cpu_baseline(code, llr_i8_np, gpu_bits):
    """The CPU oracle (exact-integer radix-2, C, -O2, one thread per core over
    frames) on the same int8 soft values: the whole batch, median of 5 runs;
    plus one thread on the first 128 frames.  Its decoded bits are compared
    with the headline variant's bits of the same batch."""
    import oracle
    threads = oracle.default_threads()
    n = llr_i8_np.shape[0]
    oracle.decode_uniform(code, llr_i8_np[:8], N_INFO, True, oracle.I64, n_threads=threads)
    times = []
    for _ in range(5):
        t0 = time.perf_counter()
        ob, _, _ = oracle.decode_uniform(code, llr_i8_np, N_INFO, True, oracle.I64,
                                         n_threads=threads)
        times.append(time.perf_counter() - t0)
    dt = float(np.median(times))
    t0 = time.perf_counter()
    oracle.decode_uniform(code, llr_i8_np[:128], N_INFO, True, oracle.I64, n_threads=1)
    dt1 = time.perf_counter() - t0
    out = {"value": round(n * N_INFO / dt / 1e9, 6), "unit": "Gbit/s", "cores": threads,
           "kind": "oracle",
           "sample": "the whole batch (%d frames x %d bits), exact-integer radix-2 oracle, "
                     "median of 5 runs (%.2f s each)" % (n, N_INFO, dt),
           "single_thread_gbit_s": round(128 * N_INFO / dt1 / 1e9, 6)}
    if gpu_bits is not None:
        out["mismatches"] = int((ob != gpu_bits).sum())
        out["mismatched_frames"] = int((ob != gpu_bits).any(axis=1).sum())
    return out


def ber_sweep(torch, mv, code, frames_plan_i8, frames_plan_f32, frames_plan_f16=None):
    from workload import make_uniform_batch, int8_scale_for
    out = []
    for db in range(0, 7):
        b = make_uniform_batch(code, N_FRAMES, N_INFO, float(db), seed=2000 + db)
        lf = torch.from_numpy(b.llr).to("cuda:0")
        li = mv.quantize_i8(lf, int8_scale_for(float(db), code.beta))
        row = {"ebn0_db": db, "bits": int(b.msg.size)}
        runs = [("f32r2", frames_plan_f32, lf), ("i8r4", frames_plan_i8, li)]
        if frames_plan_f16 is not None:
            runs.append(("f16r2", frames_plan_f16, lf.half()))
        for name, plan, llr in runs:
            bits, _, _ = plan.decode(llr)
            torch.cuda.synchronize()
            dec = mv.unpack_bits(bits.cpu().numpy()[: N_FRAMES * (N_INFO // 32)].reshape(N_FRAMES, -1), N_INFO)
            row[name + "_errors"] = int((dec != b.msg).sum())
            if name == "f32r2":
                ref = dec
            elif name == "i8r4":
                row["paired_differing_bits"] = int((dec != ref).sum())
            else:
                row[name + "_differing_bits"] = int((dec != ref).sum())
        out.append(row)
        del lf, li
    def at(target, key):
        pts = [(r["ebn0_db"], r[key] / r["bits"]) for r in out]
        for (d0, b0), (d1, b1) in zip(pts, pts[1:]):
            if b0 >= target >= b1 and b0 > 0 and b1 > 0:
                x0, x1 = math.log10(b0), math.log10(b1)
                return d0 + (math.log10(target) - x0) * (d1 - d0) / (x1 - x0)
        return None
    # double-precision oracle errors on the same batches, written by
    # tests/golden/make_ber_fp64.py (same seeds, same float32 soft values)
    gold = os.path.join(ROOT, "tests", "golden", "ber_fp64_k7_4096x8192.json")
    have64 = False
    if os.path.exists(gold):
        with open(gold) as fh:
            f64 = {p["ebn0_db"]: p for p in json.load(fh)["points"]}
        have64 = all(r["ebn0_db"] in f64 and f64[r["ebn0_db"]]["bits"] == r["bits"] for r in out)
        if have64:
            for r in out:
                r["f64_oracle_errors"] = f64[r["ebn0_db"]]["f64_errors"]
    for r in out:
        r["valid"] = all(r[k] >= 100 for k in r if k.endswith("_errors"))
    res = {"points": out, "validity": "a point with fewer than 100 errors in any decoder is "
                                      "flagged invalid (the paper's rule)"}
    for tgt in (1e-4, 1e-5):
        a, c = at(tgt, "f32r2_errors"), at(tgt, "i8r4_errors")
        res["ebn0_at_%g" % tgt] = {"f32r2": a, "i8r4": c,
                                   "gap_db": None if a is None or c is None else round(c - a, 4)}
        if have64:
            d = at(tgt, "f64_oracle_errors")
            res["ebn0_at_%g" % tgt]["f64_oracle"] = d
            res["ebn0_at_%g" % tgt]["i8r4_loss_vs_f64_db"] = (None if d is None or c is None
                                                              else round(c - d, 4))
        if frames_plan_f16 is not None:
            h = at(tgt, "f16r2_errors")
            res["ebn0_at_%g" % tgt]["f16r2"] = h
            res["ebn0_at_%g" % tgt]["f16_gap_db"] = (None if a is None or h is None
                                                     else round(h - a, 4))
    return res


def pcie_pipeline(torch, mv, plan, llr_dev, n_batches=8, depth=3):
    """Whole-job rate with the soft values in page-locked host memory and the
    bits returned there: the host pipeline overlaps copy-in, decode and
    copy-out of different batches (all batches hold the same soft values)."""
    pipe = mv.Pipeline(plan, depth)
    one = llr_dev.reshape(-1)[: pipe.llr_elems].cpu()
    h_llr = torch.empty(n_batches * pipe.llr_elems, dtype=one.dtype).pin_memory()
    for b in range(n_batches):
        h_llr[b * pipe.llr_elems:(b + 1) * pipe.llr_elems].copy_(one)
    h_bits = torch.empty(n_batches * pipe.bit_words, dtype=torch.int32).pin_memory()
    pipe.run(h_llr, h_bits, None, n_batches)  # first touch of every host page
    t0 = time.perf_counter()
    pipe.run(h_llr, h_bits, None, n_batches)
    dt = time.perf_counter() - t0
    # plain copy rate of one batch of soft values, for comparison
    d = torch.empty(pipe.llr_elems, dtype=one.dtype, device=llr_dev.device)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    for _ in range(4):
        d.copy_(h_llr[: pipe.llr_elems], non_blocking=True)
    torch.cuda.synchronize()
    h2d = 4 * pipe.llr_elems * one.element_size() / (time.perf_counter() - t1) / 1e9
    pipe.close()
    return {"value": round(n_batches * N_FRAMES * N_INFO / dt / 1e9, 3), "unit": "Gbit/s",
            "batches": n_batches, "depth": depth,
            "bytes_in_per_batch": pipe.llr_elems * one.element_size(),
            "bytes_out_per_batch": pipe.bit_words * 4,
            "host_to_device_gb_s": round(h2d, 2),
            "note": "host pipeline, page-locked host buffers; context, not the headline"}


def _gpu_ms(torch, fn, reps):
    """Median GPU time of fn() in ms (HIP events on the current stream)."""
    fn()
    torch.cuda.synchronize()
    out = []
    for _ in range(reps):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        fn()
        e1.record()
        torch.cuda.synchronize()
        out.append(e0.elapsed_time(e1))
    return float(np.median(out))


def _quantize_per_frame(torch, llr, ebn0, offsets, lengths, betas):
    """int8 soft values with each frame's own scale (16 sigma^2 of its Eb/N0),
    the library quantiser's rule applied on the GPU by torch."""
    from workload import int8_scale_for
    scale = np.repeat(np.array([int8_scale_for(float(e), int(b)) for e, b in zip(ebn0, betas)],
                               np.float32), lengths)
    assert int(offsets[0]) == 0 and scale.size == llr.shape[0]
    x = torch.from_numpy(llr).to("cuda:0") * torch.from_numpy(scale).to("cuda:0")
    return torch.clamp(torch.round(x), -127, 127).to(torch.int8)


def other_configs(torch, mv):
    """The single-frame (latency), 2^26-bit stream, 10000-frame mixed batch and
    backward workloads: GPU times (HIP events, median) and rates."""
    from workload import (CODE_K5, CODE_K7, CODE_K9, make_mixed_batch, make_stream,
                          make_uniform_batch, int8_scale_for)
    out = {}
    dev = "cuda:0"
    # single frame, 1024 bits, 3 dB: latency
    b = make_uniform_batch(CODE_K7, 1, 1024, 3.0, seed=1)
    lf = torch.from_numpy(b.llr).to(dev)
    li = mv.quantize_i8(lf, int8_scale_for(3.0, 2))
    fr = mv.uniform_frames(CODE_K7, 1, 1024, True)
    c1 = {}
    for name, dt, rx, llr in (("f32r2", "f32", 2, lf), ("i8r4", "i8", 4, li)):
        plan = mv.Plan([CODE_K7], fr, dt, rx)
        bits, metric, end = plan.empty_outputs(dev)
        gpu = _gpu_ms(torch, lambda: plan.decode(llr, bits, metric, end), 50)
        t0 = time.perf_counter()
        for _ in range(50):
            plan.decode(llr, bits, metric, end)
            torch.cuda.synchronize()
        c1[name] = {"gpu_us": round(gpu * 1e3, 1),
                    "call_and_sync_us": round((time.perf_counter() - t0) / 50 * 1e6, 1)}
        plan.close()
    out["single_frame_1024"] = c1
    # one 2^26-bit stream, 4 dB, int8, chunks of 2048 with 64 stages of overlap
    n = 1 << 26
    msg, llr = make_stream(CODE_K7, n, 4.0, seed=3)
    ls = mv.quantize_i8(torch.from_numpy(llr).to(dev), int8_scale_for(4.0, 2))
    del llr
    one = np.zeros(1, mv.FRAME_DTYPE)
    one[0] = (0, 0, n, 0, n, 0, mv.MIVIT_START_KNOWN)
    plan = mv.Plan([CODE_K7], one, "i8", 4, 2048, 64)
    bits, metric, end = plan.empty_outputs(dev)
    ms = _gpu_ms(torch, lambda: plan.decode(ls, bits, metric, end), 5)
    ops = 3 * 64 * plan.total_stages
    chunked = mv.unpack_bits(bits.cpu().numpy()[: (n + 31) // 32], n)
    plan.close()
    # the same stream decoded whole (one unchunked frame, start 0, best end):
    # the reference for the chunked decode's BER cost
    whole_plan = mv.Plan([CODE_K7], one, "i8", 4)
    wb, _, _ = whole_plan.decode(ls)
    torch.cuda.synchronize()
    whole = mv.unpack_bits(wb.cpu().numpy()[: (n + 31) // 32], n)
    whole_plan.close()
    out["stream_2p26_chunk2048_ov64"] = {
        "ms": round(ms, 3), "gbit_s": round(n / ms / 1e6, 2), "stages": plan.total_stages,
        "tops": round(ops / ms / 1e9, 2), "frac_packed_peak": round(ops / ms / 1e9 / VALU16_PEAK_TOPS, 3),
        "ber": float((chunked != msg).mean()), "whole_stream_ber": float((whole != msg).mean()),
        "ber_vs_whole_stream": float((chunked != whole).mean()),
        "bits_differing_from_whole_stream": int((chunked != whole).sum())}
    del ls, bits, wb
    # 10000 frames, log-uniform lengths, three codes, Eb/N0 U[1,5]
    codes = [CODE_K5, CODE_K7, CODE_K9]
    F = 10000
    mb = make_mixed_batch(codes, F, 64, 16384, 1.0, 5.0, seed=4)
    nn = mb.n_info.astype(np.int64)
    K = np.array([codes[c].K for c in mb.code_idx])
    beta = np.array([codes[c].beta for c in mb.code_idx])
    S = nn + K - 1
    frm = np.zeros(F, mv.FRAME_DTYPE)
    for f in range(F):
        frm[f] = (mb.llr_offset[f], mb.bit_offset[f], S[f], 0, nn[f], mb.code_idx[f],
                  mv.MIVIT_START_KNOWN | mv.MIVIT_END_ZERO)
    ops = float((3 * (2.0 ** (K - 1)) * S).sum())
    c4 = {"frames": F, "info_bits": int(nn.sum()), "acs_ops": ops,
          "longest_stages": int(S.max())}
    inputs = {"f32": torch.from_numpy(mb.llr).to(dev),
              "i8": _quantize_per_frame(torch, mb.llr, mb.ebn0_db, mb.llr_offset, S * beta, beta)}
    for dt in ("i8", "f32"):
        plan = mv.Plan(codes, frm, dt, 0, autotune=True, graph=True)
        bits, metric, end = plan.empty_outputs(dev)
        ms = _gpu_ms(torch, lambda: plan.decode(inputs[dt], bits, metric, end), 5)
        peak = VALU16_PEAK_TOPS if dt == "i8" else VALU32_PEAK_TOPS
        c4[dt] = {"ms": round(ms, 3), "gbit_s": round(nn.sum() / ms / 1e6, 2),
                  "tops": round(ops / ms / 1e9, 2), "roofline_ms": round(ops / peak / 1e9, 3),
                  "frac": round(ops / ms / 1e9 / peak, 3), "plan": plan.describe()}
        plan.close()
        # each code's frames alone (autotuned): the parts the batch overlaps
        alone = {}
        for ci, cd in enumerate(codes):
            sub = frm[mb.code_idx == ci]
            p1 = mv.Plan(codes, sub, dt, 0, autotune=True, graph=True)
            o1 = p1.empty_outputs(dev)
            alone["K%d" % cd.K] = round(_gpu_ms(torch, lambda: p1.decode(inputs[dt], *o1), 5), 3)
            p1.close()
        c4[dt]["parts_alone_ms"] = alone
    # the longest frame alone (K=9 r1/3, 16346 stages): the float32 bound, as a
    # plan spreads it by itself and over two or four wavefronts
    lf9 = {}
    one9 = frm[int(np.argmax(S)):][:1].copy()
    assert codes[int(one9[0]["code"])] is CODE_K9
    one9["code"] = 0
    for name, dt, var in (("f32_default", "f32", 0), ("f32_2waves", "f32", 6),
                          ("f32_4waves", "f32", 7), ("i8_split", "i8", 0)):
        p1 = mv.Plan([CODE_K9], one9, dt, 2, variant=var)
        o1 = p1.empty_outputs(dev)
        lf9[name] = round(_gpu_ms(torch, lambda: p1.decode(inputs[dt], *o1), 5), 3)
        p1.close()
    c4["longest_frame_ms"] = lf9
    out["mixed_10000"] = c4
    del inputs
    # backward: 2048 x 1024 bits, 2 dB, float32
    b = make_uniform_batch(CODE_K7, 2048, 1024, 2.0, seed=5)
    lf = torch.from_numpy(b.llr).to(dev)
    plan = mv.Plan([CODE_K7], mv.uniform_frames(CODE_K7, 2048, 1024, True), "f32", 2)
    bits, metric, end = plan.empty_outputs(dev)
    g = torch.linspace(0.5, 1.5, 2048, device=dev)
    grad = torch.empty_like(lf)
    fwd = _gpu_ms(torch, lambda: plan.decode(lf, bits, metric, end), 20)
    bwd = _gpu_ms(torch, lambda: plan.decode_grad(bits, g, grad), 20)
    out["backward_2048x1024"] = {"forward_us": round(fwd * 1e3, 1),
                                 "backward_us": round(bwd * 1e3, 1),
                                 "backward_bytes": int(lf.numel() * 4 + bits.numel() * 4),
                                 "backward_tb_s": round((lf.numel() * 4 + bits.numel() * 4)
                                                        / bwd / 1e9, 2)}
    plan.close()
    return out


def main():
    args = parse()
    if args.gpus != 1:
        print("bench.py measures one GPU only: frames are independent, so N GPUs would each "
              "decode their own shard of frames with no exchange; --gpus %d is not supported"
              % args.gpus, file=sys.stderr)
        sys.exit(2)
    import torch
    import paper_2011_13579_amd as mv
    from workload import CODE_K7, make_uniform_batch, int8_scale_for

    code = CODE_K7
    dev = "cuda:0"
    b = make_uniform_batch(code, N_FRAMES, N_INFO, args.ebn0, seed=2000 + int(round(args.ebn0)))
    llr_f32 = torch.from_numpy(b.llr).to(dev)
    llr_i8 = mv.quantize_i8(llr_f32, int8_scale_for(args.ebn0, code.beta))
    llr_f16 = llr_f32.half()
    torch.cuda.synchronize()
    frames = mv.uniform_frames(code, N_FRAMES, N_INFO, True)
    S = N_INFO + code.K - 1
    ops_per_launch = 3 * (1 << (code.K - 1)) * S * N_FRAMES

    if args.copy_probe:
        src = torch.empty(COPY_BYTES // 4, dtype=torch.float32, device=dev).fill_(1.0)
        dst = torch.empty_like(src)
        torch.cuda.synchronize()
        dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst
    # the other workloads first, each plan closed after use: a multi-code
    # plan's parts run concurrently only while the runtime gives their
    # streams distinct hardware queues, which fewer live streams makes likely
    configs = other_configs(torch, mv) if args.configs else None
    plans = {}
    results = {}
    decoded = {}
    for v in args.variants.split(","):
        base, _, kv = v.partition(":")
        dt, radix = {"i8r4": ("i8", 4), "f32r2": ("f32", 2), "f16r2": ("f16", 2),
                     "i8r2": ("i8", 2), "i8r8": ("i8", 8)}[base]
        # suffixes: ":vN" kernel variant N, ":nosplit" frame pairs kept whole
        plans[v] = mv.Plan([code], frames, dt, radix,
                           variant=int(kv[1:]) if kv.startswith("v") else 0,
                           split=kv != "nosplit")
        llr = {"i8": llr_i8, "f32": llr_f32, "f16": llr_f16}[dt]
        ms, fwd, tb, bits, _ = time_variant(torch, mv, plans[v], llr, args.steps, args.warmup)
        dec = mv.unpack_bits(bits.cpu().numpy()[: N_FRAMES * (N_INFO // 32)].reshape(N_FRAMES, -1), N_INFO)
        decoded[v] = dec
        # the packed kernels (variants 0, 4, 5) run 16-bit metrics; the others 32-bit
        peak = (VALU16_PEAK_TOPS if base in PACKED16 and kv in ("", "nosplit", "v4", "v5")
                else VALU32_PEAK_TOPS)
        results[v] = {
            "gbit_s": round(N_FRAMES * N_INFO / (ms * 1e-3) / 1e9, 3),
            "ms_per_step": round(ms, 4), "forward_ms": round(fwd, 4), "traceback_ms": round(tb, 4),
            "forward_tops": round(ops_per_launch / (fwd * 1e-3) / 1e12, 3),
            "forward_peak_tops": round(peak, 2),
            "forward_frac": round(ops_per_launch / (fwd * 1e-3) / 1e12 / peak, 4),
            "end_to_end_frac": round(ops_per_launch / (ms * 1e-3) / 1e12 / peak, 4),
            "bit_errors": int((dec != b.msg).sum()),
        }
    head = results.get("i8r4") or next(iter(results.values()))
    hv = "i8r4" if "i8r4" in results else next(iter(results))
    # the float32 -> int8 quantiser runs once per batch before the timed
    # step; its time, and the rate with it inside the step
    qt = torch.empty_like(llr_i8)
    quant_ms = _gpu_ms(torch, lambda: mv.quantize_i8(llr_f32, int8_scale_for(args.ebn0, code.beta),
                                                      out=qt), 20)
    del qt
    achieved = ops_per_launch / (head["forward_ms"] * 1e-3) / 1e12
    peak = head["forward_peak_tops"]
    line = {
        "metric": METRIC,
        "value": head["gbit_s"],
        "unit": "Gbit/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": head["ms_per_step"],
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "int8" if hv.startswith("i8") else "f32",
        "data": "synthetic (seeded bits, BPSK/AWGN at %.1f dB)" % args.ebn0,
        "config": {"workload": "%d terminated frames x %d info bits, K=7 (133,171) r1/2, %s" %
                   (N_FRAMES, N_INFO, hv), "frames": N_FRAMES, "info_bits": N_INFO,
                   "ebn0_db": args.ebn0, "variant": hv},
        "roofline": {"bound": "alu", "achieved": round(achieved, 3),
                     "peak": peak, "unit": "Tops/s",
                     "frac": round(achieved / peak, 4), "traffic": measured_traffic(hv),
                     "kernel": "forward (%s)" % hv,
                     "peak_basis": "packed 16-bit VALU" if peak > VALU32_PEAK_TOPS else "32-bit VALU",
                     "work": "3 ops x 64 states x %d stages x %d frames per launch (the "
                             "same count for every radix: 2 adds and a compare-select per "
                             "state and stage)" % (S, N_FRAMES),
                     "end_to_end_frac": head["end_to_end_frac"],
                     "binding_kernel": "forward"},
        "quantizer": {"in_timed_step": False, "ms": round(quant_ms, 4),
                      "gbit_s_with_quantizer": round(N_FRAMES * N_INFO /
                                                     ((head["ms_per_step"] + quant_ms) * 1e-3)
                                                     / 1e9, 3),
                      "note": "float32 -> int8 soft values (mivit_quantize_i8) of the whole "
                              "batch; the headline step decodes int8 soft values already in "
                              "HBM"},
        "variants": results,
    }
    if configs is not None:
        line["configs"] = configs
    if args.pcie and "i8r4" in plans:
        line["pcie_inclusive"] = pcie_pipeline(torch, mv, plans["i8r4"], llr_i8)
    if not args.no_cpu:
        line["cpu_baseline"] = cpu_baseline(code, llr_i8.cpu().numpy(), decoded.get("i8r4"))
    if args.ber:
        line["equal_ber"] = ber_sweep(torch, mv, code, plans.get("i8r4"), plans.get("f32r2"),
                                      plans.get("f16r2"))
    print(json.dumps(line), flush=True)


if __name__ == "__main__":
    main()
