#!/usr/bin/env python3
"""Benchmark of the PQk-means iteration on one MI355X.

A "step" is one whole iteration of Alg. 1 (assignment by linear scan, Eq. 5, then the
sparse-voting update, Eq. 7-8), issued through the C ABI.  The headline workload is the largest
configuration, the billion-scale SIFT-like one (configuration 5: N = 1e9 four-byte codes,
K = 1e5 centers, 4e14 table look-ups per step, about 15 s); `--config C` selects another.  The
steps are issued the way the workload runs them: pqkm_fit calls of the configuration's
iteration count (1 for configuration 5, 10 for configuration 2), each from the initial
centers, so whatever pqkm_fit does once per call (it regroups the codes for the scan) is inside
the timed region as often as in the workload.  Inputs are generated on the GPU and are
resident in HBM before the timed region.

Prints ONE JSON line.  `value` is code-center SDC evaluations per second over the whole step
(N*K / time per iteration, update included); `assign_evals_per_s` counts the scan kernel alone.
`roofline` is for the dominant kernel, the LDS-tiled assignment scan: achieved = the bytes its N*K*M
look-ups read from LDS per launch / the kernel's average duration (HIP events recorded by the
library on the stream the kernel runs on), against the LDS gather peak of the chip
(256 CUs x 2.4 GHz x 256 B/clk).  A look-up of the plain scans reads a 4-byte table entry, one of the
scans through lower bounds the entry's one-byte bound (`roofline.bytes_per_lookup`; the fp32 distances of
the few centers that the bounds leave are formed from the tables through the L2 and not counted); where the scan on the
matrix cores did the work, in none of the configurations here, the figures of this bound are null;
`roofline.assign_step_frac` is the same work over the time of the
whole assignment step (tile images and regrouping of the codes included).  `configs` holds the
same figures for the other configurations (a few steps each).  `cpu_baseline` is the CPU
oracle timed on the host cores, once on all of them and once on one thread.

The default command must end within the caller's time limit whatever machine of the pool it
lands on: after the first warm-up step of configuration 5 the total is projected, and if it
would pass --time-budget seconds the headline falls back to configuration 4 (the line says so).

Two things keep a sub-millisecond iteration honest: short-iteration workloads first run untimed
for --prewarm-seconds (the GPU raises its clocks only after tens of milliseconds of load), and
their K steps are timed twice, plain for `value` and once more with the event pairs for the
roofline's kernel time (a pair costs 3-4 us of stream time, 3 % of such an iteration).
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

LDS_PEAK_GBS = 256 * 2.4e9 * 256 / 1e9          # 157286 GB/s: 256 CUs x 2.4 GHz x 256 B/clk (ds_read_b128)
HBM_PEAK_GBS = 8000.0


BF16_MFMA_PEAK_TFLOPS = 2500.0                   # published dense bf16 matrix peak


def encoder_bench(args, w, pq, torch, dev) -> int:
    """PQ encoding of min(N, 2^20) random vectors of the configuration's dimensionality; HIP events on the
    stream the kernel runs on."""
    import workloads as W

    n = min(w.N, 1 << 20)
    Ds = w.D // w.M
    cw = torch.from_numpy(W.codewords(w)).to(dev)
    gen = torch.Generator(device=dev)
    gen.manual_seed(w.seed)
    vectors = torch.randn((n, w.D), generator=gen, device=dev, dtype=torch.float32)
    codes = torch.empty((n, w.M), dtype=torch.uint8, device=dev)
    for _ in range(max(args.warmup, 1)):
        pq.encode(vectors, cw, codes=codes)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    steps = max(1, min(args.steps, 20))
    e0.record()
    for _ in range(steps):
        pq.encode(vectors, cw, codes=codes)
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / steps
    flops = 3 * 2.0 * n * w.D * 256                # three bf16 products per (vector, codeword, dim): two-part splits
    tflops = flops / (ms * 1e-3) / 1e12
    print(json.dumps({
        "metric": "PQ encoding (Sec. 2.2), vectors/s", "value": n / (ms * 1e-3), "unit": "vectors/s", "n_gpus": 1,
        "steps": steps, "ms_per_step": ms, "dtype": "f32", "data": "synthetic",
        "config": {"workload": f"encoder, config {args.config} shape: {n} vectors, D={w.D}, M={w.M}, Ds={Ds}, L=256"},
        "roofline": {"bound": "mfma", "kernel": "encode_mfma_kernel", "achieved": tflops, "peak": BF16_MFMA_PEAK_TFLOPS,
                     "unit": "TFLOP/s", "frac": tflops / BF16_MFMA_PEAK_TFLOPS, "traffic": None},
        "hbm_gbs": n * w.D * 4 / (ms * 1e-3) / 1e9}))
    return 0


def naive_update_bench(args, w, pq, torch, dev) -> int:
    """Update step alone, sparse voting against the naive method, on the assignment of the first iteration."""
    import workloads as W

    n = min(w.N, 1 << 24)
    wl = w if n == w.N else __import__("dataclasses").replace(w, N=n)
    tables = pq.build_tables(torch.from_numpy(W.codewords(wl)).to(dev))
    codes = W.codes_torch(wl, dev)
    centers0 = torch.from_numpy(W.codes_at(wl, W.init_center_indices(wl))).to(dev)
    ws = torch.empty(pq.workspace_bytes(n, wl.M, wl.K), dtype=torch.uint8, device=dev)
    assign, _ = pq.assign(codes, centers0, tables, want_dist=False, workspace=ws)
    hist = torch.empty((wl.K, wl.M, 256), dtype=torch.int32, device=dev)
    steps = max(1, min(args.steps, 20))

    def timed(fn):
        for _ in range(2):
            fn()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(steps):
            fn()
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) / steps

    c1, c2 = centers0.clone(), centers0.clone()
    ms_sparse = timed(lambda: (c1.copy_(centers0), pq.update(codes, assign, tables, c1, hist=hist, workspace=ws)))
    ms_naive = timed(lambda: (c2.copy_(centers0), pq.update_naive(codes, assign, tables, c2, workspace=ws)))
    torch.cuda.synchronize()
    nz = float((hist != 0).sum()) / (wl.K * wl.M)
    print(json.dumps({
        "metric": "update step: sparse voting (Eq. 7-8) vs naive (Eq. 6)", "value": ms_naive / ms_sparse,
        "unit": "x (naive time / sparse-voting time)", "n_gpus": 1, "steps": steps, "dtype": "f32 vote, f64 naive sums",
        "data": "synthetic",
        "config": {"workload": f"config {args.config}: N={n}, M={wl.M}, K={wl.K}; assignment of the first iteration"},
        "ms_sparse_voting": ms_sparse, "ms_naive": ms_naive, "mean_nonzero_bins": nz,
        "same_centers": bool((c1 == c2).all())}))
    return 0


def indexed_bench(args, w, pq, torch, dev) -> int:
    """Alg. 1's two FindNN variants on a stretch of the configuration's codes against all its K centers: the linear
    scan and the search through the exact index over the centers, timed with HIP events, and the verdict of
    Check() (10 trials on 4096 sampled codes, as in Sec. 3.1)."""
    import dataclasses

    import workloads as W

    n = min(w.N, args.indexed_codes)
    wl = dataclasses.replace(w, N=n)
    tables = pq.build_tables(torch.from_numpy(W.codewords(w)).to(dev))
    codes = W.codes_torch(wl, dev)
    centers = torch.from_numpy(W.codes_at(w, W.init_center_indices(w))).to(dev)
    a1 = torch.empty(n, dtype=torch.int32, device=dev)
    a2 = torch.empty(n, dtype=torch.int32, device=dev)
    ws = torch.empty(pq.workspace_bytes(n, w.M, w.K), dtype=torch.uint8, device=dev)

    def timed(fn, reps):
        fn()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(reps):
            fn()
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) / reps

    note(f"linear scan over {n} codes x {w.K} centers")
    ms_scan = timed(lambda: pq.assign(codes, centers, tables, assign=a1, want_dist=False, workspace=ws), 3)
    note("indexed search over the same codes")
    ms_index = timed(lambda: pq.assign_indexed(codes, centers, tables, assign=a2, want_dist=False), 1)
    same = bool(torch.equal(a1, a2))
    note("Check() on 4096 sampled codes")
    g = torch.Generator(device="cpu")
    g.manual_seed(w.seed)
    sample = codes[torch.randperm(n, generator=g)[:4096].to(dev)].contiguous()
    use_index, c_scan, c_index = pq.check(sample, centers, tables, trials=10)
    print(json.dumps({
        "metric": "assignment step: linear scan vs exact index over the centers (Alg. 1, Check)", "value": ms_index / ms_scan,
        "unit": "x (indexed time / scan time)", "n_gpus": 1, "dtype": "f32", "data": "synthetic",
        "config": {"workload": f"config {args.config}: first {n} codes, M={w.M}, all K={w.K} initial centers"},
        "ms_scan": ms_scan, "ms_indexed": ms_index, "same_assignment": same,
        "check": {"sample": 4096, "trials": 10, "scan_ms": c_scan, "index_ms": c_index, "use_index": use_index}}))
    return 0


def microbench(torch) -> int:
    """The microbenchmarks behind the roofline denominators (paper_1709_03708_amd/csrc/microbench.hip): LDS read
    and write rates, VALU issue rates, the scan's instruction mix with and without a tile switch.  Prints a table
    on stderr and one JSON line on stdout."""
    import ctypes
    import os

    path = os.path.join(os.path.dirname(os.path.abspath(__file__)), "paper_1709_03708_amd", "libpqkm_microbench.so")
    if not os.path.exists(path):
        print("bench.py: " + path + " is missing (run __graft_entry__.build())", file=sys.stderr)
        return 2
    lib = ctypes.CDLL(path)
    lib.pqkm_microbench.restype = ctypes.c_int
    lib.pqkm_microbench.argtypes = [ctypes.c_int, ctypes.POINTER(ctypes.c_float), ctypes.POINTER(ctypes.c_double)]
    torch.zeros(1, device="cuda:0")                      # device and context
    clock = 2.4e9
    tests = [(0, "ds_read_b128, lane-consecutive", "lds"), (1, "ds_read_b64, lane-consecutive", "lds"),
             (2, "ds_read_b32, lane-consecutive", "lds"), (5, "ds_read_b128, 8 lanes per 128-byte row, random rows", "lds"),
             (3, "ds_read_b128, 4 lanes per 64-byte row, random rows", "lds"),
             (6, "ds_read_b128, 2 lanes per 32-byte row, random rows", "lds"),
             (7, "ds_read_b128, 1 lane per 16-byte row, random rows", "lds"),
             (4, "ds_write_b128, 128 KB per iteration", "lds"),
             (10, "v_add_f32", "valu"), (11, "v_min_f32", "valu"), (12, "v_min3_f32", "valu"),
             (13, "v_lshlrev_b32 (SDWA)", "valu"), (14, "v_and_b32", "valu"), (15, "v_lshrrev_b32", "valu"),
             (16, "v_fma_f32", "valu"),
             (20, "scan mix, 31 codes per lane-slot", "mix"), (21, "scan mix + two barriers per tile", "mix"),
             (22, "scan mix + two barriers + 128 KB written per tile", "mix"),
             (30, "streaming copy of 1 GiB (HBM read + write)", "hbm")]
    out = {}
    for what, name, kind in tests:
        ms, units = ctypes.c_float(0), ctypes.c_double(0)
        if lib.pqkm_microbench(what, ctypes.byref(ms), ctypes.byref(units)) != 0:
            print(f"bench.py: microbenchmark {what} failed", file=sys.stderr)
            return 1
        clocks = ms.value * 1e-3 * clock
        if kind == "lds":
            v = units.value / clocks
            line = f"{v:7.1f} B/clk/CU"
        elif kind == "valu":
            v = clocks / units.value
            line = f"{v:7.2f} clocks per wave64 instruction per SIMD"
        elif kind == "hbm":
            v = units.value * torch.cuda.get_device_properties(0).multi_processor_count / (ms.value * 1e-3) / 1e12
            line = f"{v:7.2f} TB/s"
        else:
            v = units.value * 4.0 / clocks
            line = f"{100 * v:7.1f} % of the LDS read peak ({clocks / 400:.0f} clocks per tile)"
        out[name] = v
        print(f"{name:52s} {ms.value:8.3f} ms  {line}", file=sys.stderr)
    print(json.dumps({"microbench": out, "clock_hz": clock,
                      "units": {"lds": "B/clk/CU", "valu": "clocks per wave64 instruction per SIMD",
                                "mix": "fraction of 256 B/clk/CU", "hbm": "TB/s"}}))
    return 0


_T0 = time.perf_counter()


def note(msg: str) -> None:
    """Progress on stderr (stdout carries the one JSON line): a long run must not look hung."""
    print(f"bench.py [{time.perf_counter() - _T0:6.1f} s] {msg}", file=sys.stderr, flush=True)


def measure(args, cfg, steps, warmup, pq, W, torch, dev, t_start=None, budget=0.0):
    """Generate configuration `cfg`, run `warmup` untimed and `steps` timed iterations, and return the figures
    (or None if the projected total would pass the time budget).  The scan kernel and the whole assignment
    steps are timed by HIP event pairs the library records on the stream it launches on."""
    w = W.CONFIGS[cfg]
    N, M, K = w.N, w.M, w.K
    note(f"configuration {cfg}: generating {N} codes of {M} bytes on the GPU")
    tables = pq.build_tables(torch.from_numpy(W.codewords(w)).to(dev))
    codes = W.codes_torch(w, dev)
    init_idx = W.init_center_indices(w)
    centers0 = torch.from_numpy(W.codes_at(w, init_idx)).to(dev)
    centers = centers0.clone()
    assign = torch.empty(N, dtype=torch.int32, device=dev)
    ws = torch.empty(pq.workspace_bytes(N, M, K), dtype=torch.uint8, device=dev)
    torch.cuda.synchronize()
    short = float(N) * K * M <= 2e12
    talk = float(N) * K * M >= 1e14                  # iterations of seconds: wait for each and say so

    def run(n: int, what: str = "") -> int:
        """`n` iterations as pqkm_fit calls of w.iters iterations, each from the initial centers."""
        calls, left = 0, n
        while left > 0:
            it = min(left, w.iters)
            centers.copy_(centers0)
            pq.fit(codes, tables, centers, it, assign=assign, workspace=ws)
            left -= it
            calls += 1
            if talk:
                torch.cuda.synchronize()
                note(f"configuration {cfg}: {what} iteration {n - left} of {n} done")
        return calls

    # The GPU raises its clocks only after some tens of milliseconds of load: a handful of sub-millisecond warm-up
    # steps would leave the timed region on the ramp.  Workloads whose iteration is short are therefore run untimed
    # for a fixed wall time first (the W warm-up steps then follow as asked).
    prewarm_s = 0.0
    if args.prewarm_seconds > 0 and short:
        tp = time.perf_counter()
        while time.perf_counter() - tp < args.prewarm_seconds:
            run(w.iters)
            torch.cuda.synchronize()
        prewarm_s = time.perf_counter() - tp

    # An event pair costs 3-4 us of stream time; next to a 0.25 ms iteration that is 3 % of `value`, so for
    # short-iteration workloads the K steps are timed twice: once plain (`value`, `ms_per_step`) and once more with
    # the event pairs (the roofline's kernel time; `ms_per_step_with_events`).  Long iterations are timed once, with
    # the pairs.
    ms_with_events = None
    if short:
        run(warmup)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        fit_calls = run(steps)
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        pq.set_option("profile", 3)
        run(warmup)
        torch.cuda.synchronize()
        pq.profile_read()                               # discard the warm-up launches
        pq.profile_read_steps()
        te0 = time.perf_counter()
        run(steps)
        torch.cuda.synchronize()
        ms_with_events = (time.perf_counter() - te0) * 1e3 / steps
    else:
        pq.set_option("profile", 3)
        if warmup > 0:
            tw = time.perf_counter()
            run(1, "warm-up")
            torch.cuda.synchronize()
            one = time.perf_counter() - tw
            if budget > 0 and t_start is not None:
                projected = (time.perf_counter() - t_start) + one * (warmup - 1 + steps) + args.reserve_seconds
                if projected > budget:
                    pq.set_option("profile", 0)
                    pq.profile_read()
                    pq.profile_read_steps()
                    return {"skipped": True, "first_step_s": one, "projected_s": projected}
            run(warmup - 1, "warm-up")
            torch.cuda.synchronize()
        pq.profile_read()                               # discard the warm-up launches
        pq.profile_read_steps()
        t0 = time.perf_counter()
        fit_calls = run(steps, "timed")
        torch.cuda.synchronize()
        t1 = time.perf_counter()
    scan_ms_total, scan_launches = pq.profile_read()
    step_ms_total, assign_steps = pq.profile_read_steps()
    pq.set_option("profile", 0)

    ms_per_step = (t1 - t0) * 1e3 / steps
    evals = float(N) * K
    scan_ms = scan_ms_total / max(scan_launches, 1)
    lookups_per_launch = evals * M * steps / max(scan_launches, 1)
    bytes_each = bytes_per_lookup(w, pq, ws)
    achieved_gbs = lookups_per_launch * bytes_each / (scan_ms * 1e-3) / 1e9 if scan_ms > 0 and bytes_each else None
    assign_step_ms = step_ms_total / max(assign_steps, 1)
    return {
        "skipped": False, "w": w, "codes": codes, "tables": tables, "centers0": centers0,
        "ms_per_step": ms_per_step, "value": evals / (ms_per_step * 1e-3), "fit_calls": fit_calls,
        "prewarm_s": prewarm_s, "short": short, "ms_with_events": ms_with_events,
        "scan_ms": scan_ms, "scan_ms_total": scan_ms_total, "scan_launches": scan_launches,
        "achieved_gbs": achieved_gbs, "lookups_per_launch": lookups_per_launch,
        "assign_step_ms": assign_step_ms,
        "bytes_per_lookup": bytes_each,
        "assign_step_frac": evals * M * bytes_each / (assign_step_ms * 1e-3) / 1e9 / LDS_PEAK_GBS
        if assign_step_ms > 0 and bytes_each else None,
    }


def bytes_per_lookup(w, pq, workspace) -> float | None:
    """LDS bytes per (code, center, subspace), averaged over the iterations of a fit call: 1 for the scan through lower bounds,
    4 for the others; the library says which of them an iteration runs.  None where the last call in `workspace` was done by
    the scan on the matrix cores, which looks nothing up per pair."""
    dot = pq.dot_scan(w.N, w.M, w.K, workspace)
    if dot["tried"] and not dot["left"]:
        return None
    each = [1.0 if pq.scan_plan(w.N, w.M, w.K, it)["scan"] == 2 else 4.0 for it in range(w.iters)]
    return sum(each) / len(each)


def workload_label(cfg, w) -> str:
    return f"config {cfg} ({w.name}): N={w.N} uint8 codes, M={w.M}, K={w.K}, D={w.D}"


def cpu_baseline(r, oracle) -> dict:
    """The CPU oracle (assign + update) on a bounded sample of the headline workload: the first n codes against all
    K centers, about 10 s on all host threads and about 10 s on one."""
    w = r["w"]
    K = w.K
    h_tables = r["tables"].cpu().numpy()
    cent = r["centers0"].cpu().numpy()
    cores = oracle.max_threads()

    def timed(threads: int, seconds: float):
        note(f"CPU oracle on {threads} thread(s), about {seconds:.0f} s")
        oracle.set_threads(threads)
        n_sub = int(min(w.N, max(2_000, seconds * 1e8 * threads / K)))
        h_codes = r["codes"][:n_sub].cpu().numpy()
        reps, c0 = 0, time.perf_counter()
        while True:
            a, _ = oracle.assign(h_codes, cent, h_tables, want_dist=False)
            oracle.update(h_codes, a, h_tables, cent)
            reps += 1
            t_cpu = time.perf_counter() - c0
            if t_cpu >= seconds or reps >= 200:
                break
        return float(n_sub) * K * reps / t_cpu, (f"{reps} oracle iterations (assign + update) over the first {n_sub} "
                                                 f"codes x all {K} centers, {t_cpu:.1f} s")

    v_all, s_all = timed(cores, 10.0)
    v_one, s_one = timed(1, 8.0)
    oracle.set_threads(cores)
    return {"value": v_all, "unit": "SDC evaluations/s", "cores": cores, "kind": "oracle", "sample": s_all,
            "single_thread": {"value": v_one, "cores": 1, "sample": s_one}}


def main() -> int:
    t_start = time.perf_counter()
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=4)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--config", type=int, default=5,
                    help="headline workload configuration (1-5); 5, the largest, is the benchmark's")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-sub-configs", action="store_true",
                    help="skip the few-step runs of the other configurations (the `configs` array)")
    ap.add_argument("--time-budget", type=float, default=540.0,
                    help="seconds the whole run may take; if configuration 5 would not fit (projected after its first "
                         "warm-up step) the headline falls back to configuration 4; 0 = never fall back")
    ap.add_argument("--reserve-seconds", type=float, default=70.0,
                    help="part of the time budget kept for the other configurations and the CPU baseline")
    ap.add_argument("--prewarm-seconds", type=float, default=0.5,
                    help="untimed run before the warm-up steps so that the GPU clocks have ramped up (short iterations only)")
    ap.add_argument("--encoder", action="store_true",
                    help="time the PQ encoder (Sec. 2.2), the preprocessing step in front of the clustering, on "
                         "random vectors of the configuration's shape instead of the iteration; prints its own line")
    ap.add_argument("--naive-update", action="store_true",
                    help="time the sparse-voting update (Eq. 7-8) against the naive update (Eq. 6) on the "
                         "configuration's first assignment, as in the paper's per-step runtime table; prints its own line")
    ap.add_argument("--indexed", action="store_true",
                    help="time the assignment through the exact index over the centers (Alg. 1's table branch) against "
                         "the linear scan on a stretch of the configuration's codes, and run Check(); prints its own line")
    ap.add_argument("--indexed-codes", type=int, default=1 << 20, help="codes of the --indexed comparison")
    ap.add_argument("--microbench", action="store_true",
                    help="run the microbenchmarks behind the roofline denominators (LDS read and write rates, VALU "
                         "issue rates, the scan's instruction mix with and without a tile switch) and print them")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="run only a plain device copy of 1 GiB (5 times): the known-size kernel against which "
                         "the FETCH_SIZE / WRITE_SIZE counters of rocprofv3 --pmc are scaled")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py: this build runs on ONE GPU (no sharding, no collectives); use --gpus 1", file=sys.stderr)
        return 2

    import numpy as np
    import torch

    import paper_1709_03708_amd as pq
    import workloads as W

    if not torch.cuda.is_available():
        print("bench.py: no GPU visible", file=sys.stderr)
        return 2
    pq.load()                                           # fails loudly if the HIP library is missing
    dev = torch.device("cuda:0")
    if args.microbench:
        return microbench(torch)
    if args.copy_calibration:
        src = torch.full((1 << 28,), 1.0, dtype=torch.float32, device=dev)      # 1 GiB
        dst = torch.empty_like(src)
        for _ in range(5):
            dst.copy_(src)
        torch.cuda.synchronize()
        print(json.dumps({"copy_bytes_read": 1 << 30, "copy_bytes_written": 1 << 30, "copies": 5}))
        return 0
    if args.encoder:
        return encoder_bench(args, W.CONFIGS[args.config], pq, torch, dev)
    if args.naive_update:
        return naive_update_bench(args, W.CONFIGS[args.config], pq, torch, dev)
    if args.indexed:
        return indexed_bench(args, W.CONFIGS[args.config], pq, torch, dev)

    cfg = args.config
    fallback = None
    r = measure(args, cfg, args.steps, args.warmup, pq, W, torch, dev, t_start, args.time_budget if cfg == 5 else 0.0)
    if r["skipped"]:
        fallback = (f"configuration 5 would not fit the time budget of {args.time_budget:.0f} s on this machine (first "
                    f"step {r['first_step_s']:.1f} s, projected {r['projected_s']:.0f} s for {args.warmup} + {args.steps} "
                    f"steps); the headline is configuration 4, the largest that fits")
        print("bench.py: " + fallback, file=sys.stderr)
        r = None
        torch.cuda.empty_cache()
        cfg = 4
        r = measure(args, cfg, args.steps, args.warmup, pq, W, torch, dev)
    w = r["w"]
    N, M, K = w.N, w.M, w.K

    out = {
        "metric": "code-center SDC evaluations/sec in assignment (N*K/s); seconds per PQk-means iter",
        "value": r["value"],
        "unit": "SDC evaluations/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": r["ms_per_step"],
        "sec_per_iter": r["ms_per_step"] * 1e-3,
        "assign_evals_per_s": float(N) * K * args.steps / (r["scan_ms_total"] * 1e-3),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": workload_label(cfg, w),
                   "N": N, "M": M, "K": K, "iterations_timed": args.steps, "fit_calls": r["fit_calls"],
                   "iterations_per_fit_call": w.iters, "prewarm_s": round(r["prewarm_s"], 3)},
        "roofline": {"bound": "lds", "kernel": "assign_filter / assign_scan (LDS-tiled linear scan, Eq. 5)",
                     "bytes_per_lookup": r["bytes_per_lookup"],
                     "achieved": r["achieved_gbs"], "peak": LDS_PEAK_GBS, "unit": "GB/s",
                     "frac": r["achieved_gbs"] / LDS_PEAK_GBS if r["achieved_gbs"] else None, "traffic": None,
                     "avg_kernel_ms": r["scan_ms"], "launches": r["scan_launches"],
                     "timed_in": ("a second pass of the same steps with HIP event pairs around every scan launch"
                                  if r["short"] else "the timed region (HIP event pairs around every scan launch)"),
                     "ms_per_step_with_events": r["ms_with_events"] if r["short"] else r["ms_per_step"],
                     "assign_step_ms": r["assign_step_ms"], "assign_step_frac": r["assign_step_frac"],
                     "lookups_per_s": r["lookups_per_launch"] / (r["scan_ms"] * 1e-3),
                     "hbm_algorithmic_gbs": (N * M + 4 * N) / (r["scan_ms_total"] / args.steps * 1e-3) / 1e9,
                     "hbm_peak_gbs": HBM_PEAK_GBS},
    }
    if fallback:
        out["config"]["fallback"] = fallback

    cpu = None
    if not args.no_cpu_baseline:
        import oracle

        cpu = cpu_baseline(r, oracle)
    r = None
    torch.cuda.empty_cache()

    if not args.no_sub_configs:
        subs = []
        for c in (2, 3, 4):
            if c == cfg:
                continue
            if args.time_budget > 0 and time.perf_counter() - t_start > args.time_budget - 20:
                subs.append({"config": c, "skipped": "time budget"})
                continue
            # whole fit calls of the configuration's iteration count where an iteration is short (configuration 2: 10),
            # so that the regrouping pass per call weighs as it does in the workload
            sub_steps = W.CONFIGS[c].iters if W.CONFIGS[c].N * W.CONFIGS[c].K < 1e10 else 3
            sr = measure(args, c, sub_steps, 1, pq, W, torch, dev)
            sw = sr["w"]
            subs.append({"config": c, "workload": workload_label(c, sw), "steps": sub_steps, "warmup": 1,
                         "ms_per_step": sr["ms_per_step"], "value": sr["value"],
                         "avg_kernel_ms": sr["scan_ms"], "launches": sr["scan_launches"],
                         "frac": sr["achieved_gbs"] / LDS_PEAK_GBS if sr["achieved_gbs"] else None,
                         "assign_step_ms": sr["assign_step_ms"],
                         "assign_step_frac": sr["assign_step_frac"]})
            sr = None
            torch.cuda.empty_cache()
        out["configs"] = subs
    if cpu is not None:
        out["cpu_baseline"] = cpu
    print(json.dumps(out))
    return 0


if __name__ == "__main__":
    sys.exit(main())
