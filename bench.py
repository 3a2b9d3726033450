#!/usr/bin/env python3
"""Benchmark of the drafter LM-head hot path on one MI355X.

One step = one call of the low-rank head (down-projection, vocabulary projection with the
fused running log-sum-exp / top-k, cross-workgroup merge) through the C ABI on one batch of
synthetic hidden states, with every input already resident in HBM.  The headline workload is
the single-row latency shape d=4096, r=512, V=128256, k=10 (C2); the other workloads (C3, the
512-row throughput shape C4 with its rank sweep, C5, 16 and 64 rows, the full-head comparator,
a warm-cache run, six calls in one HIP graph) are reported in the "extra" object of the same
JSON line, each with its own roofline entry.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload C2|C3|C4|C5] [--head low_rank|full] [--quick]

Prints exactly one JSON line on stdout (progress goes to stderr).
"""
from __future__ import annotations

import argparse
import glob
import hashlib
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0          # MI355X published HBM3E bandwidth
MFMA_PEAK_TFLOPS = 2500.0      # dense bf16 / fp16 matrix peak
TRAFFIC_FILE = os.path.join(ROOT, "profiles", "hbm_traffic.json")


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def kernel_sources_digest():
    """SHA-256 over the library's kernel sources: names the code a counter run was made on."""
    h = hashlib.sha256()
    csrc = os.path.join(ROOT, "paper_2605_10453_amd", "csrc")
    for path in sorted(glob.glob(os.path.join(csrc, "*.hip")) + glob.glob(os.path.join(csrc, "*.hpp"))):
        h.update(os.path.basename(path).encode())
        h.update(open(path, "rb").read())
    return h.hexdigest()


def measured_traffic(workload):
    """HBM bytes per launch of the dominant kernel from the committed rocprofv3 --pmc summary
    (profiles/hbm_traffic.json); None unless that summary was made on exactly these kernel sources."""
    try:
        rec = json.load(open(TRAFFIC_FILE))
    except (OSError, ValueError):
        return None
    if rec.get("kernel_sources_sha256") != kernel_sources_digest():
        return None
    return rec.get("traffic_bytes_per_launch", {}).get(workload)


def algorithmic_bytes_low_rank(rows, d, r, V, k):
    """Bytes the method must move: every weight once, h once, outputs once."""
    return 2 * (d * r + r * V + rows * d) + rows * k * 8


def projection_kernel(rows, K, V, k, full=False, prepared=False):
    """The kernel that a call's vocabulary projection runs, and the bytes per element of its row operand: the library's
    rules for the shapes timed here (one row, or d of a few thousand; a test holds them against the library's own)."""
    if rows <= (1 if full else 2):
        return "stream_topk_kernel", 4                     # fp32 t or h
    if k > 16 or rows <= (32 if prepared else 48):
        return "rows_topk_kernel", 2 if full else 6        # h, or t as three bf16 pieces
    if not full and rows > 128 and K <= 512 and (k <= 12 or prepared):
        return "head_resident_kernel", 2
    return "head_tile_kernel", 2


def projection_kernel_bytes(rows, K, V, k, full=False, prepared=False):
    """Algorithmic bytes of one launch of the vocabulary-projection kernel: the [K, V] bf16 weight
    matrix once plus its [rows, K] input."""
    return 2 * K * V + projection_kernel(rows, K, V, k, full, prepared)[1] * rows * K


def percentiles(v):
    v = sorted(v)
    n = len(v)
    return {"median": v[n // 2], "p10": v[max(0, (n * 10) // 100)], "p90": v[min(n - 1, (n * 90) // 100)], "mean": sum(v) / n}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=200)
    ap.add_argument("--warmup", type=int, default=20)
    ap.add_argument("--workload", default="C2")
    ap.add_argument("--copies", type=int, default=4,
                    help="distinct device copies of the weights rotated between steps so that every step "
                         "streams them from HBM rather than from the 256 MB last-level cache")
    ap.add_argument("--head", default="low_rank", choices=("low_rank", "full"),
                    help="full: time full_head_topk on the workload's shape instead (a profiling aid: the comparator "
                         "alone in the run; implies --quick)")
    ap.add_argument("--prepared", action="store_true",
                    help="time slimspec_head_topk_prepared (the caller also passes a column-major copy of B, made once "
                         "before the timed region) instead of slimspec_head_topk; the JSON line says so in config")
    ap.add_argument("--quick", action="store_true", help="skip the extra workloads and the CPU baseline")
    ap.add_argument("--no-extra", action="store_true", help="skip the extra workloads only")
    ap.add_argument("--cpu-seconds", type=float, default=12.0)
    ap.add_argument("--copy-probe", action="store_true",
                    help="also launch a plain elementwise copy of 128 MiB a few times: the reference a counter run "
                         "scales its FETCH_SIZE / WRITE_SIZE readings by")
    args = ap.parse_args()

    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py: this build runs on one GPU only (no sharding, no collectives); use --gpus 1",
              file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch
    from paper_2605_10453_amd import binding, synth

    if not torch.cuda.is_available():
        print("bench.py: no GPU visible; the HIP path has no CPU fallback", file=sys.stderr)
        sys.exit(3)
    torch.cuda.set_device(0)
    binding.load_library()
    dev = torch.device("cuda:0")

    def upload(bits):
        return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).to(dev).view(torch.bfloat16)

    def null_event_pair_ms(n=50):
        """Elapsed time between two HIP events recorded back to back on an idle stream position:
        what an event pair reports around an empty interval."""
        pairs = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(n)]
        torch.cuda.synchronize()
        for a, b in pairs:
            a.record()
            b.record()
        torch.cuda.synchronize()
        v = sorted(a.elapsed_time(b) for a, b in pairs)
        return v[len(v) // 2]

    def _event_pairs(n):
        pairs = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(n)]
        for a, b in pairs:      # create the HIP handles
            a.record()
            b.record()
        torch.cuda.synchronize()
        return pairs

    def _timed(step, steps, warmup, with_events=True):
        """Wall-clock time of `steps` back-to-back calls; then, in two more passes over the same steps, the
        per-call durations (an event pair around every call) and the projection kernel's (an event pair
        recorded by the library around that kernel, on the call's stream)."""
        for i in range(warmup):
            step(i)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for i in range(steps):
            step(i)
        torch.cuda.synchronize()
        dt = time.perf_counter() - t0
        kern_ms, call_us = None, None
        if with_events:
            pairs = _event_pairs(steps)
            for i, (a, b) in enumerate(pairs):
                a.record()
                step(i)
                b.record()
            torch.cuda.synchronize()
            call_us = percentiles([a.elapsed_time(b) * 1e3 for a, b in pairs])
            pairs = _event_pairs(steps)
            for i, (a, b) in enumerate(pairs):
                binding.slimspec_set_timing_events(a, b)
                step(i)
            binding.slimspec_set_timing_events(None, None)
            torch.cuda.synchronize()
            kern_ms = sum(a.elapsed_time(b) for a, b in pairs) / steps
        return dt, kern_ms, call_us

    def out_buffers(rows, d, r, V, k):
        ids = torch.empty((rows, k), dtype=torch.int32, device=dev)
        lp = torch.empty((rows, k), dtype=torch.float32, device=dev)
        ws = torch.empty(binding.slimspec_workspace_bytes(rows, d, r, V, k), dtype=torch.uint8, device=dev)
        return ids, lp, ws

    def time_low_rank_tensors(h, As, Bs, k, steps, warmup, with_events=True, prepared=False):
        rows, d = h.shape
        r, V = Bs[0].shape
        ids, lp, ws = out_buffers(rows, d, r, V, k)
        n = len(Bs)
        if prepared:          # weights are prepared once, outside the timed region
            Bts = [binding.slimspec_transpose_weights(b) for b in Bs]
            torch.cuda.synchronize()

            def step(i):
                binding.slimspec_head_topk_prepared(h, As[i % n], Bs[i % n], Bts[i % n], k, out_ids=ids, out_logprobs=lp, workspace=ws)
        else:
            def step(i):
                binding.slimspec_head_topk(h, As[i % n], Bs[i % n], k, out_ids=ids, out_logprobs=lp, workspace=ws)

        return _timed(step, steps, warmup, with_events)

    def time_low_rank(cfg, x, steps, warmup, copies, with_events=True):
        h = upload(x.h)
        As = [upload(x.A)]
        Bs = [upload(x.B)]
        for _ in range(copies - 1):
            As.append(As[0].clone())
            Bs.append(Bs[0].clone())
        return time_low_rank_tensors(h, As, Bs, cfg.k, steps, warmup, with_events, prepared=args.prepared)

    def time_full_tensors(h, Ws, k, steps, warmup, with_events=True):
        rows, d = h.shape
        V = Ws[0].shape[1]
        ids, lp, ws = out_buffers(rows, d, 8, V, k)
        n = len(Ws)

        def step(i):
            binding.full_head_topk(h, Ws[i % n], k, out_ids=ids, out_logprobs=lp, workspace=ws)

        return _timed(step, steps, warmup, with_events)

    def device_inputs(rows, d, r, V, seed, copies, peaked_every=0):
        """Inputs of the same distributions as the seeded host generator, drawn on the device (the extra
        workloads are timed only; their values do not matter beyond their distribution)."""
        g = torch.Generator(device=dev)
        g.manual_seed(seed)
        h = torch.randn((rows, d), generator=g, device=dev, dtype=torch.float32)
        if peaked_every:
            h[::peaked_every] *= 4.0
        h = h.to(torch.bfloat16)
        A = (torch.randn((d, r), generator=g, device=dev, dtype=torch.float32) * d ** -0.5).to(torch.bfloat16)
        B = torch.empty((r, V), device=dev, dtype=torch.bfloat16)
        for j0 in range(0, r, 128):
            j1 = min(r, j0 + 128)
            B[j0:j1] = (torch.randn((j1 - j0, V), generator=g, device=dev, dtype=torch.float32) * r ** -0.5).to(torch.bfloat16)
        return h, [A] + [A.clone() for _ in range(copies - 1)], [B] + [B.clone() for _ in range(copies - 1)]

    def roofline_of(name, rows, K, V, k, kern_ms, null_ms, full=False, prepared=False):
        """Roofline entry of the vocabulary-projection kernel of one call."""
        kbytes = projection_kernel_bytes(rows, K, V, k, full, prepared)
        flops = 2.0 * rows * K * V
        kern_s = kern_ms * 1e-3
        hbm = kbytes / kern_s / 1e9
        mfma = flops / kern_s / 1e12
        # the kernel's arithmetic intensity (about `rows` flop per byte) against the ridge of the two peaks (312 flop/B)
        if flops / kbytes >= MFMA_PEAK_TFLOPS * 1e3 / HBM_PEAK_GBS:
            out = {"bound": "mfma", "achieved": mfma, "peak": MFMA_PEAK_TFLOPS, "unit": "TFLOP/s",
                   "frac": mfma / MFMA_PEAK_TFLOPS, "hbm_frac_same_kernel": hbm / HBM_PEAK_GBS}
        else:
            out = {"bound": "hbm", "achieved": hbm, "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": hbm / HBM_PEAK_GBS,
                   "mfma_frac_same_kernel": mfma / MFMA_PEAK_TFLOPS}
        out.update({"traffic": measured_traffic(name),
                    "kernel": f"vocabulary projection + running log-sum-exp / top-k ({projection_kernel(rows, K, V, k, full, prepared)[0]})",
                    "kernel_us": kern_ms * 1e3,
                    "kernel_us_minus_empty_event_pair": (kern_ms - null_ms) * 1e3,
                    "empty_event_pair_us": null_ms * 1e3,
                    "algorithmic_bytes_per_launch": kbytes,
                    "algorithmic_flops_per_launch": flops})
        return out

    def low_rank_entry(name, rows, d, r, V, k, dt, steps, kern_ms, call_us, null_ms):
        """What is reported for one timed low-rank workload."""
        us = dt / steps * 1e6
        flops = 2.0 * rows * (d * r + r * V)
        return {"shape": {"rows": rows, "d": d, "r": r, "V": V, "k": k},
                "us_per_call": us, "rows_per_s": rows / (us * 1e-6),
                "us_per_call_event_pairs": call_us,
                "call_hbm_frac": algorithmic_bytes_low_rank(rows, d, r, V, k) / (us * 1e-6) / 1e9 / HBM_PEAK_GBS,
                "call_mfma_frac": flops / (us * 1e-6) / 1e12 / MFMA_PEAK_TFLOPS,
                "roofline": roofline_of(name, rows, r, V, k, kern_ms, null_ms)}

    # ------------------------------------------------------------------ headline workload
    cfg = synth.CONFIGS[args.workload]
    log(f"[bench] generating {cfg.name}: rows={cfg.rows} d={cfg.d} r={cfg.r} V={cfg.V} k={cfg.k}")
    x = synth.make_inputs(cfg, seed=0)
    copies = max(1, args.copies)
    null_ms = null_event_pair_ms()
    full_only = args.head == "full"
    if full_only:
        args.quick = True
        log(f"[bench] timing the FULL head on this shape: {args.warmup} warm-up + {args.steps} steps, {copies} weight copies")
        gw_ = torch.Generator(device=dev)
        gw_.manual_seed(1)
        W0 = torch.empty((cfg.d, cfg.V), device=dev, dtype=torch.bfloat16)
        for j0 in range(0, cfg.d, 256):
            W0[j0:j0 + 256] = (torch.randn((min(256, cfg.d - j0), cfg.V), generator=gw_, device=dev) * cfg.d ** -0.5).to(torch.bfloat16)
        dt, kern_ms, call_us = time_full_tensors(upload(x.h), [W0] + [W0.clone() for _ in range(copies - 1)], cfg.k,
                                                 args.steps, args.warmup)
        del W0
    else:
        log(f"[bench] timing low-rank head: {args.warmup} warm-up + {args.steps} steps, {copies} weight copies")
        dt, kern_ms, call_us = time_low_rank(cfg, x, args.steps, args.warmup, copies)
    ms_per_step = dt / args.steps * 1e3
    rows_per_s = cfg.rows * args.steps / dt
    log(f"[bench] {ms_per_step * 1e3:.2f} us/call, {rows_per_s:.1f} rows/s, projection kernel {kern_ms * 1e3:.2f} us "
        f"(empty event pair {null_ms * 1e3:.2f} us)")

    head_name = ("FULL head (comparator, not the headline metric)" if full_only else
                 "low-rank head with the caller's column-major copy of B" if args.prepared else "low-rank head")
    out = {
        "metric": "LM-head rows/s (and us/call) at d=4096,r=512,V=128256; % HBM/MFMA peak",
        "value": rows_per_s, "unit": "rows/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": ms_per_step, "us_per_call": ms_per_step * 1e3,
        "us_per_call_event_pairs": call_us,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "bf16 weights and hidden states, fp32 accumulate",
        "data": "synthetic (seeded host generator for the headline workload; the extra workloads draw the same "
                "distributions on the device)",
        "config": {"workload": f"{cfg.name}: {head_name} "
                               f"rows={cfg.rows} d={cfg.d} r={cfg.r} V={cfg.V} k={cfg.k}, "
                               f"{copies} rotating weight copies (cold last-level cache)",
                   "rows": cfg.rows, "d": cfg.d, "r": cfg.r, "V": cfg.V, "k": cfg.k},
        "roofline": roofline_of(cfg.name + ("_full" if full_only else ""), cfg.rows, cfg.d if full_only else cfg.r, cfg.V,
                                cfg.k, kern_ms, null_ms, full=full_only, prepared=args.prepared),
        "call_hbm_frac": (2.0 * cfg.d * cfg.V if full_only else algorithmic_bytes_low_rank(cfg.rows, cfg.d, cfg.r, cfg.V, cfg.k))
                         / (ms_per_step * 1e-3) / 1e9 / HBM_PEAK_GBS,
        "kernel_sources_sha256": kernel_sources_digest(),
    }

    if args.copy_probe:
        src = torch.ones(32 << 20, dtype=torch.float32, device=dev)
        dst = torch.empty_like(src)
        for _ in range(5):
            torch.mul(src, 1.0, out=dst)       # one elementwise kernel: reads 128 MiB, writes 128 MiB
        torch.cuda.synchronize()
        out["copy_probe"] = {"kernel": "torch elementwise mul by 1.0", "bytes_read": src.numel() * 4,
                             "bytes_written": dst.numel() * 4, "launches": 5}
        del src, dst

    # ------------------------------------------------------------------ CPU baseline (the fp64 checker)
    if not args.quick:
        import oracle
        oracle.build(force=False)
        log("[bench] timing the CPU fp64 checker on the same inputs")
        sub_rows = min(cfg.rows, 8)
        hs = np.ascontiguousarray(x.h[:sub_rows])
        oracle.slimspec_head_topk(hs, x.A, x.B, cfg.k)          # warm the page cache / thread pool
        n, t0 = 0, time.perf_counter()
        while True:
            oracle.slimspec_head_topk(hs, x.A, x.B, cfg.k)
            n += 1
            el = time.perf_counter() - t0
            if el >= args.cpu_seconds and n >= 3:
                break
        out["cpu_baseline"] = {"value": n * sub_rows / el, "unit": "rows/s", "cores": oracle.num_threads(),
                               "kind": "oracle",
                               "sample": f"{n} calls of the fp64 checker on the first {sub_rows} row(s) of the "
                                         f"same inputs, {el:.1f} s of wall time",
                               "us_per_call": el / n * 1e6}
    else:
        out["cpu_baseline"] = None

    # ------------------------------------------------------------------ extra workloads (context)
    if not (args.quick or args.no_extra):
        extra = {}
        # the same workload from a warm last-level cache: one copy of the weights, every call re-reads it
        log("[bench] warm cache (one weight copy)")
        wdt, wk, wcall = time_low_rank(cfg, x, args.steps, args.warmup, 1)
        extra["warm_cache"] = {"us_per_call": wdt / args.steps * 1e6, "projection_kernel_us": wk * 1e3,
                               "us_per_call_event_pairs": wcall, "weight_copies": 1,
                               "note": "the weights (135 MB at C2) stay in the 256 MB last-level cache between calls"}

        # the same workload with the outputs of stochastic decoding (log-sum-exp and one Gumbel-max draw per row)
        try:
            hs_, As_, Bs_ = upload(x.h), [upload(x.A) for _ in range(copies)], [upload(x.B) for _ in range(copies)]
            ws_s = torch.empty(binding.slimspec_workspace_bytes(cfg.rows, cfg.d, cfg.r, cfg.V, cfg.k), dtype=torch.uint8, device=dev)
            sdt, _, scall = _timed(lambda i: binding.slimspec_head_sample(hs_, As_[i % copies], Bs_[i % copies], cfg.k, i, workspace=ws_s),
                                   args.steps, args.warmup, with_events=False)
            extra["with_sampling_outputs"] = {"us_per_call": sdt / args.steps * 1e6,
                                              "note": "slimspec_head_sample: top-k, lse and one draw per row (the binding allocates "
                                                      "five small output tensors per call here)"}
            del hs_, As_, Bs_, ws_s
        except Exception as exc:
            extra["with_sampling_outputs"] = {"error": repr(exc)[:200]}
        log("[bench] full head on the same shape")
        g = torch.Generator(device=dev)
        g.manual_seed(1)
        W = torch.empty((cfg.d, cfg.V), device=dev, dtype=torch.bfloat16)
        for j0 in range(0, cfg.d, 256):
            W[j0:j0 + 256] = (torch.randn((min(256, cfg.d - j0), cfg.V), generator=g, device=dev) * cfg.d ** -0.5).to(torch.bfloat16)
        Ws = [W, W.clone()]
        hdev = upload(x.h)
        nf = max(10, args.steps // 4)
        fdt, fk, fcall = time_full_tensors(hdev, Ws, cfg.k, nf, 5)
        fms = fdt / nf * 1e3
        froof = roofline_of(cfg.name + "_full", cfg.rows, cfg.d, cfg.V, cfg.k, fk, null_ms, full=True)
        extra["full_head"] = {"us_per_call": fms * 1e3, "projection_kernel_us": fk * 1e3,
                              "us_per_call_event_pairs": fcall,
                              "roofline_frac_kernel": froof["frac"], "bound": froof["bound"],
                              "low_rank_speedup": fms / ms_per_step,
                              "ideal_speedup": 1.0 / ((cfg.r / cfg.d) * (1 + cfg.d / cfg.V)),
                              "paper_relative_head_time_r_d8": 0.21,
                              "paper_hardware": "NVIDIA H200, vLLM 0.17.1 (context only; the paper's head time "
                                                "excludes softmax / top-k)"}
        # the static-truncation comparator of Appendix C: the full head over the first V_tr columns with an id map
        try:
            trunc = {}
            for v_tr, nu_paper in ((65536, 0.58), (32768, 0.33), (16384, 0.20)):
                Wt = [w[:, :v_tr].contiguous() for w in Ws]
                idm = torch.arange(v_tr, dtype=torch.int32, device=dev)
                ids_t, lp_t, ws_t = out_buffers(cfg.rows, cfg.d, 8, v_tr, cfg.k)
                step_t = lambda i: binding.truncated_head_topk(hdev, Wt[i % 2], idm, cfg.k, out_ids=ids_t, out_logprobs=lp_t, workspace=ws_t)
                tdt, _, tcall = _timed(step_t, nf, 5, with_events=False)
                trunc[f"V_tr_{v_tr}"] = {"us_per_call": tdt / nf * 1e6, "relative_to_full_head": tdt / fdt,
                                         "paper_relative_head_time": nu_paper}
                del Wt
            trunc["note"] = ("truncated_head_topk on the first V_tr columns; the paper's ratios are VocabTrim / FR-Spec "
                             "on H200 in vLLM without softmax / top-k (context only)")
            extra["truncated_head"] = trunc
        except Exception as exc:
            extra["truncated_head"] = {"error": repr(exc)[:200]}
        # the dynamic-selection comparator of Appendix C: low-rank router, exact full-head logits on the routed ids
        try:
            k_route = 64
            hr_, Ar_, Br_ = upload(x.h), [upload(x.A) for _ in range(2)], [upload(x.B) for _ in range(2)]
            idr, lpr, _ = out_buffers(cfg.rows, cfg.d, cfg.r, cfg.V, cfg.k)
            shape_r = binding.SlimspecShape(cfg.rows, cfg.d, cfg.r, cfg.V)
            import ctypes as _ct
            wsr = torch.empty(int(binding.load_library().routed_workspace_bytes(_ct.byref(shape_r), k_route)), dtype=torch.uint8, device=dev)
            step_r = lambda i: binding.routed_head_topk(hr_, Ar_[i % 2], Br_[i % 2], Ws[i % 2], k_route, cfg.k,
                                                        out_ids=idr, out_logprobs=lpr, workspace=wsr)
            rdt, _, _ = _timed(step_r, nf, 5, with_events=False)
            extra["routed_head"] = {"us_per_call": rdt / nf * 1e6, "k_route": k_route, "relative_to_full_head": rdt / fdt,
                                    "paper_relative_head_time_r_d8": 0.46,
                                    "note": "routed_head_topk: low-rank router (k_route ids per row), exact logits on those, softmax "
                                            "over them; the paper's ratio is SpecVocab at r = d/8 on H200 in vLLM (context only)"}
            # the same head from the token-major full head Wt [V, d] (the layout frameworks store it in)
            Wts = [w.t().contiguous() for w in Ws]
            step_t = lambda i: binding.routed_head_topk_prepared(hr_, Ar_[i % 2], Br_[i % 2], Wts[i % 2], k_route, cfg.k,
                                                                 out_ids=idr, out_logprobs=lpr, workspace=wsr)
            tdt, _, _ = _timed(step_t, nf, 5, with_events=False)
            extra["routed_head"]["token_major_W_us_per_call"] = tdt / nf * 1e6
            extra["routed_head"]["token_major_W_relative_to_full_head"] = tdt / fdt
            del hr_, Ar_, Br_, wsr, Wts
        except Exception as exc:
            extra["routed_head"] = {"error": repr(exc)[:200]}
        # six head calls (the paper's six draft steps, section 5.1) captured in one HIP graph: no host launch jitter
        try:
            hg = upload(x.h)
            Ag = [upload(x.A) for _ in range(2)]
            Bg = [upload(x.B) for _ in range(2)]
            idg, lpg, wsg = out_buffers(cfg.rows, cfg.d, cfg.r, cfg.V, cfg.k)
            binding.slimspec_head_topk(hg, Ag[0], Bg[0], cfg.k, out_ids=idg, out_logprobs=lpg, workspace=wsg)
            torch.cuda.synchronize()
            eager_ids, eager_lp = idg.clone(), lpg.clone()
            side = torch.cuda.Stream()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.stream(side):
                with torch.cuda.graph(graph, stream=side):
                    for i in range(6):
                        binding.slimspec_head_topk(hg, Ag[i % 2], Bg[i % 2], cfg.k, out_ids=idg, out_logprobs=lpg, workspace=wsg)
            ok = True
            for _ in range(3):
                graph.replay()
                torch.cuda.synchronize()
                ok = ok and bool(torch.equal(idg, eager_ids)) and bool(torch.equal(lpg, eager_lp))
            nrep = 40
            t0 = time.perf_counter()
            for _ in range(nrep):
                graph.replay()
            torch.cuda.synchronize()
            extra["graph_of_6_calls"] = {"us_per_call": (time.perf_counter() - t0) / (6 * nrep) * 1e6,
                                         "replays_match_eager": ok, "weight_copies": 2}
            del graph
        except Exception as exc:                      # graph capture is a convenience figure only
            extra["graph_of_6_calls"] = {"error": repr(exc)[:200]}

        if cfg.name == "C2":
            # full head on 512 rows first (it shares W with the run above), then the other low-rank workloads
            c4 = synth.CONFIGS["C4"]
            others = [("C3", 1, 5120, 640, 151936, 10, 0, 4, 100), ("C4_512_rows", 512, 4096, 512, 128256, 10, 10, 2, 50),
                      ("C4_r256", 512, 4096, 256, 128256, 10, 10, 3, 50), ("C4_r1024", 512, 4096, 1024, 128256, 10, 10, 2, 40),
                      ("C5", 256, 8192, 1024, 128256, 16, 0, 2, 40),
                      ("rows_16", 16, 4096, 512, 128256, 10, 0, 3, 60), ("rows_64", 64, 4096, 512, 128256, 10, 0, 3, 60)]
            full512 = None
            try:
                log("[bench] full head, 512 rows")
                h4, _, _ = device_inputs(c4.rows, c4.d, 8, 8, 4, 1, peaked_every=c4.peaked_every)
                sf = 30          # (the first calls after idle run at lower clocks: ten warm-up calls)
                fdt4, fk4, fcall4 = time_full_tensors(h4, Ws, c4.k, sf, 10)
                rf4 = roofline_of("C4_full", c4.rows, c4.d, c4.V, c4.k, fk4, null_ms, full=True)
                full512 = {"us_per_call": fdt4 / sf * 1e6, "projection_kernel_us": fk4 * 1e3, "us_per_call_event_pairs": fcall4,
                           "roofline_frac_kernel": rf4["frac"], "bound": rf4["bound"]}
            except Exception as exc:
                full512 = {"error": repr(exc)[:200]}
            del Ws, W
            torch.cuda.empty_cache()
            for name, rows, d, r, V, k, peaked, ncopies, nsteps in others:
                log(f"[bench] {name}: rows={rows} d={d} r={r} V={V} k={k}")
                try:
                    h, As, Bs = device_inputs(rows, d, r, V, 7, ncopies, peaked_every=peaked)
                    edt, ek, ecall = time_low_rank_tensors(h, As, Bs, k, nsteps, 8)
                    extra[name] = low_rank_entry(name, rows, d, r, V, k, edt, nsteps, ek, ecall, null_ms)
                    extra[name]["weight_copies"] = ncopies
                    if rows >= 5:       # with the caller's column-major copy of B as well (read from 33 rows on)
                        qdt, _, _ = time_low_rank_tensors(h, As, Bs, k, nsteps, 8, with_events=False, prepared=True)
                        extra[name]["prepared_weights_us_per_call"] = qdt / nsteps * 1e6
                    if name == "C4_512_rows":
                        ws_s = torch.empty(binding.slimspec_workspace_bytes(rows, d, r, V, k), dtype=torch.uint8, device=dev)
                        sdt, _, _ = _timed(lambda i: binding.slimspec_head_sample(h, As[i % ncopies], Bs[i % ncopies], k, i, workspace=ws_s),
                                           20, 3, with_events=False)
                        extra[name]["with_sampling_outputs_us_per_call"] = sdt / 20 * 1e6
                        Bts_s = [binding.slimspec_transpose_weights(b_) for b_ in Bs]
                        sdt, _, _ = _timed(lambda i: binding.slimspec_head_sample_prepared(h, As[i % ncopies], Bs[i % ncopies], Bts_s[i % ncopies],
                                                                                           k, i, workspace=ws_s), 20, 3, with_events=False)
                        extra[name]["with_sampling_outputs_prepared_weights_us_per_call"] = sdt / 20 * 1e6
                        del ws_s
                        # the same rows as six drafted positions (section 5.1 drafts six tokens) with a down-projection each
                        n_pos = 6
                        stack = torch.stack([As[0]] + [(torch.randn((d, r), device=dev) * d ** -0.5).to(torch.bfloat16)
                                                       for _ in range(n_pos - 1)]).contiguous()
                        off = [rows * p_ // n_pos for p_ in range(n_pos + 1)]
                        ids_p, lp_p, ws_p = out_buffers(rows, d, r, V, k)
                        pdt, _, _ = _timed(lambda i: binding.slimspec_head_topk_positions(h, stack, off, Bs[i % ncopies], k, out_ids=ids_p,
                                                                                         out_logprobs=lp_p, workspace=ws_p),
                                           20, 3, with_events=False)
                        extra[name]["six_positions_us_per_call"] = pdt / 20 * 1e6
                        pdt, _, _ = _timed(lambda i: binding.slimspec_head_topk_positions_prepared(h, stack, off, Bs[i % ncopies], Bts_s[i % ncopies], k,
                                                                                                  out_ids=ids_p, out_logprobs=lp_p, workspace=ws_p),
                                           20, 3, with_events=False)
                        extra[name]["six_positions_prepared_weights_us_per_call"] = pdt / 20 * 1e6
                        del Bts_s
                        del stack, ids_p, lp_p, ws_p
                        # the router-then-exact head on the same rows, 16 routed ids per row (the router on the matrix cores)
                        k_rt = 16
                        Wr = (torch.randn((d, V), device=dev) * d ** -0.5).to(torch.bfloat16)
                        Wrt = Wr.t().contiguous()
                        Bt0 = binding.slimspec_transpose_weights(Bs[0])
                        import ctypes as _ct2
                        shape_q = binding.SlimspecShape(rows, d, r, V)
                        ws_q = torch.empty(int(binding.load_library().routed_workspace_bytes(_ct2.byref(shape_q), k_rt)), dtype=torch.uint8, device=dev)
                        ids_q, lp_q, _ = out_buffers(rows, d, r, V, k)
                        q1, _, _ = _timed(lambda i: binding.routed_head_topk(h, As[0], Bs[0], Wr, k_rt, k, out_ids=ids_q, out_logprobs=lp_q,
                                                                             workspace=ws_q), 10, 2, with_events=False)
                        q2, _, _ = _timed(lambda i: binding.routed_head_topk_prepared(h, As[0], Bs[0], Wrt, k_rt, k, Bt=Bt0, out_ids=ids_q,
                                                                                      out_logprobs=lp_q, workspace=ws_q), 20, 3, with_events=False)
                        extra[name]["routed_head_k_route_16"] = {"us_per_call": q1 / 10 * 1e6, "token_major_W_and_Bt_us_per_call": q2 / 20 * 1e6,
                                                                 "note": "one copy of the weights (warm last-level cache for B, W read sparsely)"}
                        del Wr, Wrt, Bt0, ws_q, ids_q, lp_q
                    del h, As, Bs
                    torch.cuda.empty_cache()
                except Exception as exc:
                    extra[name] = {"error": repr(exc)[:200]}
            if "us_per_call" in extra.get("C4_512_rows", {}) and full512 and "us_per_call" in full512:
                full512["low_rank_speedup"] = full512["us_per_call"] / extra["C4_512_rows"]["us_per_call"]
            if "C4_512_rows" in extra:
                extra["C4_512_rows"]["full_head"] = full512
        out["extra"] = extra

    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
