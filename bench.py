#!/usr/bin/env python3
"""Benchmark of the APH predistorter on one MI355X.

Headline workload: one stream of N = 2^24 complex64 OFDM-like samples (16-QAM
on 1200 of 2048 subcarriers, RMS 0.25), odd orders {1,3,5,7} in the main and
the conjugate branch, L = 4 taps, DC term; FP32 arithmetic.  One step = one
forward apply of the whole stream (every step of Eq. 1 / Algorithm 1) on
inputs already resident in HBM.  Input/output buffers rotate over >= 2 GiB so
the 256 MB last-level cache cannot serve repeated steps.

Prints ONE JSON line: throughput, the HBM roofline of the kernel (algorithmic
bytes / kernel time from HIP events on the launch stream), the FP64 oracle
timed on the host (which also gates accuracy) and, under "secondary", the
other workloads: the launch-bound N = 65,536 stream, the two-carrier N = 2^26
stream (orders to 9, L = 8), the 256-stream batch (persistent launch vs
per-stream launches), the adjoint, the coefficient-learning step (fused
kernels vs autograd vs plain-ops autograd), least-squares estimation and
indirect learning, the paper's Table 2 configuration and host ingestion.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--main-only] [--only-leg NAME]
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import sys
import time
import traceback

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "DPD Msamples/s + % HBM roofline at NMSE≤-110 dB vs oracle; grad-step time"
HBM_PEAK_GBS = 8000.0
VALU_FP32_PEAK_TFLOPS = 157.3      # 1024 SIMDs x 32 FMAs a cycle at 2.4 GHz: by two waves of a SIMD, one alone half
MFMA_BF16_TFLOPS = 2500.0          # dense bf16 matrix-core peak of MI355X
BYTES_PER_SAMPLE = 16              # 8 B complex64 read + 8 B written
ROTATE_BYTES = 2 << 30
PMC_FILE = os.path.join(ROOT, "profiles", "dpd_fwd_n2p24_P7_L4_pmc.txt")
KERNEL_SOURCES = ["paper_1612_09001_amd/csrc/dpd_fwd_kernels.h",
                  "paper_1612_09001_amd/csrc/dpd_internal.h"]


def kernel_hash() -> str:
    h = hashlib.sha256()
    for rel in KERNEL_SOURCES:
        with open(os.path.join(ROOT, rel), "rb") as f:
            h.update(f.read())
    return h.hexdigest()[:16]


def traffic_from_profile(n: int):
    """HBM bytes per launch from the committed rocprofv3 --pmc summary
    (FETCH_SIZE and WRITE_SIZE, each scaled by the same counter read on a plain
    copy of known size); None when the kernel sources changed since then."""
    try:
        kv = {}
        with open(PMC_FILE) as f:
            for line in f:
                if ":" in line and not line.startswith("#"):
                    k, v = line.split(":", 1)
                    kv[k.strip()] = v.strip()
    except OSError:
        return None
    if kv.get("kernel_sources_sha256_16") != kernel_hash() or kv.get("n") != str(n):
        return None
    try:
        return int(float(kv["traffic_bytes_per_launch"]))
    except (KeyError, ValueError):
        return None


STATS_FILE = os.path.join(ROOT, "profiles", "dpd_fwd_n2p24_P7_L4_stats.txt")


def kernel_ns_from_profile(n: int):
    """Average duration (ns) of the headline kernel in the committed rocprofv3
    --stats summary; None when the kernel sources changed since then."""
    kv = {}
    try:
        with open(STATS_FILE) as f:
            for line in f:
                if ":" in line and not line.startswith("#"):
                    k, v = line.split(":", 1)
                    kv[k.strip()] = v.strip()
    except OSError:
        return None
    if kv.get("kernel_sources_sha256_16") != kernel_hash() or kv.get("n", str(n)) != str(n):
        return None
    try:
        return float(kv["stats_average_ns"])
    except (KeyError, ValueError):
        return None


_ORC = None


def _oracle():
    """The FP64 oracle (test infrastructure), loaded once for the accuracy
    gates and the CPU baseline."""
    global _ORC
    if _ORC is None:
        import oracle
        _ORC = oracle.Oracle()
    return _ORC


def _metrics():
    sys.path.insert(0, os.path.join(ROOT, "tests"))
    import metrics
    return metrics


def gate(z_gpu, z_ref) -> dict:
    """NMSE and max relative error of a GPU output against the FP64 oracle."""
    m = _metrics()
    nm, mr = m.nmse_db(z_gpu, z_ref), m.max_rel(z_gpu, z_ref)
    return {"nmse_db": round(nm, 2), "max_rel": float("%.3g" % mr),
            "pass": bool(nm <= m.NMSE_DB_MAX and mr <= m.MAX_REL_MAX)}


def gate_dcoef(g_gpu, g_ref, entry_max=None, rel_max=None) -> dict:
    m = _metrics()
    entry_max = m.DCOEF_ENTRY_MAX if entry_max is None else entry_max
    rel_max = m.DCOEF_REL_MAX if rel_max is None else rel_max
    ee = m.entry_err(g_gpu, g_ref)
    rel = float(np.linalg.norm(np.asarray(g_gpu) - g_ref) / np.linalg.norm(g_ref))
    return {"entry_err": float("%.3g" % ee), "rel_l2": float("%.3g" % rel),
            "pass": bool(ee <= entry_max and rel <= rel_max)}


def _timed(fn):
    t0 = time.perf_counter()
    r = fn()
    return r, time.perf_counter() - t0


CPU_BUDGET_S = 10.0   # host time spent timing the oracle on each thread count


def _repeat_timed(fn, budget_s, min_runs=3):
    """Runs fn until `budget_s` seconds (and at least min_runs runs) have
    passed; returns the median run time and the number of runs."""
    times = []
    t_all = time.perf_counter()
    while len(times) < min_runs or time.perf_counter() - t_all < budget_s:
        t = time.perf_counter()
        fn()
        times.append(time.perf_counter() - t)
    return float(np.median(times)), len(times)


def cpu_baseline(x_host, z_gpu, mo, co, L, h):
    """FP64 oracle on the host cores over the whole headline workload, repeated
    for about CPU_BUDGET_S seconds (median run); also gates the GPU output
    against it."""
    orc = _oracle()
    z = orc.forward(x_host, mo, co, L, h)
    t, runs = _repeat_timed(lambda: orc.forward(x_host, mo, co, L, h), CPU_BUDGET_S)
    n = x_host.size
    acc = gate(z_gpu, z)
    threads = orc.threads()
    # the same oracle on one thread, over the first 2^21 samples
    m = min(n, 1 << 21)
    orc.set_threads(1)
    t1, runs1 = _repeat_timed(lambda: orc.forward(x_host[:m], mo, co, L, h), CPU_BUDGET_S)
    orc.set_threads(threads)
    base = {"value": round(n / t / 1e6, 3), "unit": "Msamples/s", "cores": threads,
            "kind": "oracle",
            "sample": "whole headline workload: %d samples through the FP64 C oracle "
                      "(gcc -O2, OpenMP), median of %d runs over about %g s" % (n, runs, CPU_BUDGET_S),
            "single_thread_value": round(m / t1 / 1e6, 3),
            "single_thread_sample": "first %d samples of the same workload, one thread, median of %d runs over "
                                    "about %g s" % (m, runs1, CPU_BUDGET_S),
            "cpu_model": _cpu_model()}
    return base, acc


# oracle timings of the secondary workloads, filled in by their legs
CPU_EXTRA = {}


def _cpu_model() -> str:
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def _rotating(torch, x_host, total_bytes=ROTATE_BYTES):
    n = x_host.size
    nbuf = max(2, total_bytes // (2 * 8 * n))
    xs = [torch.from_numpy(x_host).cuda() for _ in range(nbuf)]
    zs = [torch.empty_like(xs[0]) for _ in range(nbuf)]
    return xs, zs


WARM_S = 0.05   # the GPU clocks settle after ~30 ms of load (and drop again while the host works)


def _time_launches(torch, launch, nbuf, steps, warmup):
    """Back-to-back launches between one pair of HIP events on the launch
    stream (torch's current stream); returns wall seconds and mean ms per
    launch (kernel time plus the inter-launch gap of a busy queue).  Before
    timing: `warmup` launches, repeated until at least WARM_S of load has
    run, so every leg is timed at settled clocks."""
    t0 = time.perf_counter()
    while True:
        for i in range(max(1, warmup)):
            launch(i % nbuf)
        torch.cuda.synchronize()
        if time.perf_counter() - t0 >= WARM_S:
            break
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    t0 = time.perf_counter()
    e0.record()
    for i in range(steps):
        launch(i % nbuf)
    e1.record()
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    return wall, e0.elapsed_time(e1) / steps


def leg_config1(torch, dpd, signals, steps=2000, graph_len=100, singles=200):
    """The small configuration: one stream of N = 65,536 samples, the headline
    basis (orders {1,3,5,7} both branches, L = 4, DC).  Its 1 MiB of traffic
    takes 0.13 us at HBM peak, so launch overhead bounds it: back-to-back
    launches, the same launches replayed from one hipGraph, and the latency of
    one launch followed by a stream synchronisation."""
    from paper_1612_09001_amd import autotune

    orders, L, n = [1, 3, 5, 7], 4, 65536
    plan = dpd.Plan(orders, orders, L, signals.aph_coeffs(orders, orders, L, config_id=1))
    x = torch.from_numpy(signals.ofdm_16qam(n, config_id=1)).cuda()
    z = torch.empty_like(x)
    st = dpd.current_stream()
    default_ms = _time_launches(
        torch, lambda i: dpd.dpd_apply(plan.handle, st, x.data_ptr(), z.data_ptr(), n), 1, steps, 200)[1]
    tune = autotune.tune_plan(plan, x, out=z)
    wall, launch_ms = _time_launches(
        torch, lambda i: dpd.dpd_apply(plan.handle, st, x.data_ptr(), z.data_ptr(), n), 1, steps, 200)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        sc = dpd.current_stream()
        for _ in range(graph_len):
            dpd.dpd_apply(plan.handle, sc, x.data_ptr(), z.data_ptr(), n)
    for _ in range(5):
        g.replay()
    torch.cuda.synchronize()
    reps = max(1, steps // graph_len)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(reps):
        g.replay()
    e1.record()
    torch.cuda.synchronize()
    graph_us = e0.elapsed_time(e1) * 1e3 / (reps * graph_len)
    lat = []
    for _ in range(singles):
        t0 = time.perf_counter()
        dpd.dpd_apply(plan.handle, st, x.data_ptr(), z.data_ptr(), n)
        torch.cuda.current_stream().synchronize()
        lat.append(time.perf_counter() - t0)
    lat_us = float(np.median(lat)) * 1e6
    orc = _oracle()
    x_host = x.cpu().numpy()
    h = signals.aph_coeffs(orders, orders, L, config_id=1)
    ref = orc.forward(x_host, orders, orders, L, h)
    reps_cpu = []
    for _ in range(20):
        t0 = time.perf_counter()
        orc.forward(x_host, orders, orders, L, h)
        reps_cpu.append(time.perf_counter() - t0)
    CPU_EXTRA["config1_forward"] = {"msamples_per_s": round(n / float(np.median(reps_cpu)) / 1e6, 2),
                                    "sample": "the whole N=65536 stream, median of 20", "cores": orc.threads()}
    return {"workload": "single stream N=65536, orders {1,3,5,7} main+conj, L=4, DC (launch-bound)",
            "accuracy": gate(z.cpu().numpy(), ref),
            "tune": tune, "back_to_back_us_per_apply_default_tune": round(default_ms * 1e3, 2),
            "back_to_back_us_per_apply": round(launch_ms * 1e3, 2),
            "back_to_back_msamples_per_s": round(n / (launch_ms * 1e-3) / 1e6, 1),
            "graph_us_per_apply": round(graph_us, 2),
            "graph_msamples_per_s": round(n / (graph_us * 1e-6) / 1e6, 1),
            "launch_plus_sync_latency_us_median": round(lat_us, 1),
            "hbm_time_at_peak_us": round(BYTES_PER_SAMPLE * n / (HBM_PEAK_GBS * 1e9) * 1e6, 3)}


def leg_config3(torch, dpd, signals, steps=50):
    """N = 2^26 two-carrier stream, orders {1..9} both branches, L = 8."""
    orders = [1, 3, 5, 7, 9]
    L, n = 8, 1 << 26
    x_host = signals.two_carrier(n, config_id=3)
    h = signals.aph_coeffs(orders, orders, L, config_id=3)
    plan = dpd.Plan(orders, orders, L, h)
    xs, zs = _rotating(torch, x_host)
    st = dpd.current_stream()
    ptrs = [(a.data_ptr(), b.data_ptr()) for a, b in zip(xs, zs)]
    wall, kmean = _time_launches(
        torch, lambda i: dpd.dpd_apply(plan.handle, st, ptrs[i][0], ptrs[i][1], n), len(xs), steps, 50)
    flops = 8 * len(orders) * L + 3           # widely-linear FIR + |x|^2 per sample
    tfl = flops * n / (kmean * 1e-3) / 1e12
    gbs = BYTES_PER_SAMPLE * n / (kmean * 1e-3) / 1e9
    z_last = zs[(steps - 1) % len(xs)].cpu().numpy()
    del xs, zs
    orc = _oracle()
    ref, t_cpu = _timed(lambda: orc.forward(x_host, orders, orders, L, h))
    CPU_EXTRA["config3_forward"] = {"msamples_per_s": round(n / t_cpu / 1e6, 2), "cores": orc.threads(),
                                    "sample": "the whole 2^26-sample two-carrier stream, one run"}
    acc = gate(z_last, ref)
    del ref, z_last
    return {"workload": "two-carrier N=2^26, orders {1,3,5,7,9} main+conj, L=8, DC", "accuracy": acc,
            "msamples_per_s": round(n * steps / wall / 1e6, 1), "kernel_ms": round(kmean, 4),
            "hbm_gbs": round(gbs, 1), "hbm_frac": round(gbs / HBM_PEAK_GBS, 4),
            "valu_tflops": round(tfl, 2), "flops_per_sample": flops,
            "valu_frac": round(tfl / VALU_FP32_PEAK_TFLOPS, 4), "tune": plan.get_tune()}


def _steady_us(fn, rounds=5, warmup=10, iters=30):
    """Median over `rounds` of the mean time per call of `iters` back-to-back
    calls after `warmup` untimed ones (HIP events), the first round after at
    least WARM_S of load: the steady-state time of a launch long enough that
    the clock state of the first calls matters."""
    import torch
    from paper_1612_09001_amd import autotune

    t0 = time.perf_counter()
    while time.perf_counter() - t0 < WARM_S:
        for _ in range(warmup):
            fn()
        torch.cuda.synchronize()
    return float(np.median([autotune.time_us(fn, warmup=warmup, iters=iters) for _ in range(rounds)]))


def leg_config4(torch, dpd, signals):
    """256 streams, lengths U[2^14, 2^20], own coefficients, P_max in {5,7,9},
    L in {2..8}: one persistent launch (graph-replayed) vs 256 launches."""
    from paper_1612_09001_amd import autotune, batch

    wl = batch.BatchWorkload(signals.batch_specs(), config_id=4)
    tune, b = autotune.tune_batch(wl)
    total = wl.samples()
    t_direct = _steady_us(b.apply)
    t_each = _steady_us(b.apply_each)
    g = torch.cuda.CUDAGraph()
    b.apply()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        b.apply()
    t_graph = _steady_us(g.replay)
    ge = torch.cuda.CUDAGraph()
    with torch.cuda.graph(ge):
        b.apply_each()
    t_graph_each = _steady_us(ge.replay)
    gbs = BYTES_PER_SAMPLE * total / (t_graph * 1e-6) / 1e9
    # every output of every stream (from the last graph replay) against the oracle
    torch.cuda.synchronize()
    z = wl.z.cpu().numpy()
    orc = _oracle()
    worst = None
    for s_, (n_, pmax, L_) in enumerate(wl.specs):
        orders_ = signals.odd_orders(pmax)
        g = gate(z[wl.offsets[s_]:wl.offsets[s_] + n_],
                 orc.forward(wl.stream_input(s_), orders_, orders_, L_, wl.coeffs_host[s_]))
        if worst is None or g["nmse_db"] > worst["nmse_db"]:
            worst = dict(g, stream=s_)
        worst["pass"] = bool(worst["pass"] and g["pass"])
    # widely-linear FIR + |x|^2 per sample, per stream (both branches hold orders 1..P_max)
    flops = sum(n * (8 * ((pmax + 1) // 2) * L + 3) for n, pmax, L in wl.specs)
    t_hbm = BYTES_PER_SAMPLE * total / (HBM_PEAK_GBS * 1e9) * 1e6
    t_valu = flops / (VALU_FP32_PEAK_TFLOPS * 1e12) * 1e6
    # each stream at the larger of its own two times: the bound when streams
    # of different classes do not overlap memory and ALU work with each other
    t_cls = sum(max(BYTES_PER_SAMPLE * n / (HBM_PEAK_GBS * 1e9),
                    n * (8 * ((pmax + 1) // 2) * L + 3) / (VALU_FP32_PEAK_TFLOPS * 1e12))
                for n, pmax, L in wl.specs) * 1e6
    return {"workload": "256 streams, n~U[2^14,2^20] (seeded), P_max in {5,7,9}, L in {2..8}, conj+DC",
            "accuracy_worst_stream": worst,
            "samples": total, "tune": tune, "chunks_blocks": list(b.info()),
            "persistent_graph_us": round(t_graph, 1), "persistent_us": round(t_direct, 1),
            "per_stream_launches_us": round(t_each, 1), "per_stream_graph_us": round(t_graph_each, 1),
            "msamples_per_s": round(total / t_graph, 1), "hbm_frac": round(gbs / HBM_PEAK_GBS, 4),
            "flops_per_sample": round(flops / total, 1),
            "valu_frac": round(flops / (t_graph * 1e-6) / 1e12 / VALU_FP32_PEAK_TFLOPS, 4),
            "bound_us": round(max(t_hbm, t_valu), 1), "bound_frac": round(max(t_hbm, t_valu) / t_graph, 4),
            "per_stream_bound_us": round(t_cls, 1), "per_stream_bound_frac": round(t_cls / t_graph, 4),
            "speedup_vs_per_stream": round(t_each / t_graph, 2),
            "speedup_vs_per_stream_graph": round(t_graph_each / t_graph, 2)}


def leg_batch_classes(torch, dpd, signals, reps=20):
    """The 256-stream workload class by class (the streams of one (P_max, L)
    class as a batch of their own, in the persistent kernel), against one
    stream of the same class and total length through the single-stream
    kernel; for per-class counters under a profiler (one batch_kernel dispatch
    group per class, in the printed order).  Not part of the default run."""
    from paper_1612_09001_amd import autotune, batch

    specs = signals.batch_specs()
    wl = batch.BatchWorkload(specs, config_id=4)
    classes = sorted({(pm, L) for _, pm, L in specs}, key=lambda c: (-(c[0] + 1) // 2 * c[1], c))
    st = dpd.current_stream()
    out = []
    for pm, L in classes:
        idx = [i for i, (_, p_, l_) in enumerate(specs) if (p_, l_) == (pm, L)]
        streams = [wl.streams()[i] for i in idx]
        total = int(sum(specs[i][0] for i in idx))
        b = batch.Batch(streams, tune={"samples_per_thread": 8, "grid_mult": 16})
        t_b = autotune.time_us(b.apply, warmup=3, iters=reps)
        orders = signals.odd_orders(pm)
        plan = dpd.Plan(orders, orders, L, signals.aph_coeffs(orders, orders, L, config_id=4))
        x = torch.from_numpy(signals.ofdm_16qam(total, config_id=4, stream_id=1000 + pm * 10 + L)).cuda()
        z = torch.empty_like(x)
        t_s = autotune.time_us(lambda: dpd.dpd_apply(plan.handle, st, x.data_ptr(), z.data_ptr(), total),
                               warmup=3, iters=reps)
        ni = (pm + 1) // 2
        fl = 8 * ni * L + 3
        bound = max(BYTES_PER_SAMPLE * total / (HBM_PEAK_GBS * 1e9), fl * total / (VALU_FP32_PEAK_TFLOPS * 1e12))
        out.append({"P_max": pm, "L": L, "streams": len(idx), "samples": total, "batch_us": round(t_b, 1),
                    "single_stream_us": round(t_s, 1), "batch_over_single": round(t_b / t_s, 3),
                    "bound_us": round(bound * 1e6, 1), "batch_frac_of_bound": round(bound * 1e6 / t_b, 3),
                    "single_frac_of_bound": round(bound * 1e6 / t_s, 3)})
        b.close()
        del x, z
    return {"workload": "the 256-stream batch split by (P_max, L) class", "classes": out,
            "sum_batch_us": round(sum(c["batch_us"] for c in out), 1),
            "sum_single_us": round(sum(c["single_stream_us"] for c in out), 1),
            "sum_bound_us": round(sum(c["bound_us"] for c in out), 1)}


def leg_backward(torch, dpd, signals, steps=50):
    """Adjoint of the headline forward (N = 2^24, orders {1,3,5,7} both
    branches, L = 4): input and coefficient gradients in one call."""
    orders, L, n = [1, 3, 5, 7], 4, 1 << 24
    h = signals.aph_coeffs(orders, orders, L, config_id=1)
    plan = dpd.Plan(orders, orders, L, h)
    x = torch.from_numpy(signals.ofdm_16qam(n, config_id=1)).cuda()
    g = torch.from_numpy(signals.ofdm_16qam(n, config_id=1, stream_id=1)).cuda()
    gx = torch.empty_like(x)
    gc = torch.empty(plan.K, dtype=torch.complex64, device="cuda")
    wsb = dpd.dpd_backward_ws_size(plan.handle, 1, n)
    ws = torch.empty(max(wsb, 1), dtype=torch.uint8, device="cuda")
    st = dpd.current_stream()
    wall, kmean = _time_launches(
        torch, lambda i: dpd.dpd_backward(plan.handle, st, 0, x.data_ptr(), g.data_ptr(), gx.data_ptr(),
                                          gc.data_ptr(), 1, n, n, ws.data_ptr(), wsb), 1, steps, 20)
    ni = (orders[-1] + 1) // 2
    # dx: transposed filter 8*NI*L + basis Jacobian ~12*NI; dcoef: outer products 8*NI*L + basis 2*NI
    flops = 16 * ni * L + 14 * ni
    nbytes = 24 * n                         # x and G read, dx written
    orc = _oracle()
    (rx, rc), t_cpu = _timed(lambda: orc.backward(x.cpu().numpy(), orders, orders, L, h, g.cpu().numpy()))
    CPU_EXTRA["backward"] = {"msamples_per_s": round(n / t_cpu / 1e6, 2), "cores": orc.threads(),
                             "sample": "dx and dcoef of the whole 2^24-sample stream, one run"}
    acc = {"dx": gate(gx.cpu().numpy(), rx), "dcoef": gate_dcoef(gc.cpu().numpy(), rc)}
    return {"workload": "adjoint of the headline: N=2^24, orders {1,3,5,7} main+conj, L=4; dx and dcoef",
            "accuracy": acc,
            "kernel_ms": round(kmean, 4), "msamples_per_s": round(n / (kmean * 1e-3) / 1e6, 1),
            "hbm_frac": round(nbytes / (kmean * 1e-3) / 1e9 / HBM_PEAK_GBS, 4), "flops_per_sample": flops,
            "valu_frac": round(flops * n / (kmean * 1e-3) / 1e12 / VALU_FP32_PEAK_TFLOPS, 4)}


# The paper's Table 4 peak throughputs for the Table 2 configuration (32-bit
# float; mobile SoCs of 2014-2015): context for the table2 leg, not a target.
PAPER_TABLE4_MSPS = {"Tegra K1 GPU (Kepler, 852 MHz)": 153.5, "Tegra X1 GPU (Maxwell, 998 MHz)": 221.8,
                     "TK1 4x Cortex-A15 NEON+OpenMP": 214.4, "TX1 4x Cortex-A57 NEON+OpenMP": 200.1}


def leg_table2(torch, dpd, signals, steps=200):
    """The paper's Table 2 configuration (section 3.4): P = 5 main, Q = 3
    conjugate, L = 5, DC term, on N = 2^24 OFDM-like samples."""
    mo, co, L, n = [1, 3, 5], [1, 3], 5, 1 << 24
    x_host = signals.ofdm_16qam(n, config_id=2)
    plan = dpd.Plan(mo, co, L, signals.aph_coeffs(mo, co, L, config_id=2))
    xs, zs = _rotating(torch, x_host)
    st = dpd.current_stream()
    ptrs = [(a.data_ptr(), b.data_ptr()) for a, b in zip(xs, zs)]
    wall, kmean = _time_launches(
        torch, lambda i: dpd.dpd_apply(plan.handle, st, ptrs[i][0], ptrs[i][1], n), len(xs), steps, 200)
    msps = n / (kmean * 1e-3) / 1e6
    gbs = BYTES_PER_SAMPLE * n / (kmean * 1e-3) / 1e9
    z_last = zs[(steps - 1) % len(xs)].cpu().numpy()
    del xs, zs
    best = max(PAPER_TABLE4_MSPS.values())
    acc = gate(z_last, _oracle().forward(x_host, mo, co, L, signals.aph_coeffs(mo, co, L, config_id=2)))
    return {"workload": "Table 2 configuration: orders {1,3,5} main, {1,3} conjugate, L=5, DC; N=2^24",
            "accuracy": acc,
            "kernel_ms": round(kmean, 4), "msamples_per_s": round(msps, 1),
            "hbm_frac": round(gbs / HBM_PEAK_GBS, 4), "tune": plan.get_tune(),
            "paper_table4_msamples_per_s": PAPER_TABLE4_MSPS,
            "ratio_to_best_paper_number": round(msps / best, 1)}


def leg_ingest(torch, dpd, signals, reps=3):
    """Host ingestion: 2^25 samples from pinned host memory through the
    headline predistorter back to pinned host memory (chunks of 2^20 to 2^22
    on three streams, copies overlapped with filtering), and the zero-copy form (one
    launch on the buffers' device mappings); host-link-bound rates, never the
    headline value."""
    from paper_1612_09001_amd import ingest

    orders, L, n = [1, 3, 5, 7], 4, 1 << 25
    plan = dpd.Plan(orders, orders, L, signals.aph_coeffs(orders, orders, L, config_id=1))
    xh = torch.from_numpy(signals.ofdm_16qam(n, config_id=1)).pin_memory()
    zh = torch.empty(n, dtype=torch.complex64).pin_memory()
    out = {"workload": "pinned host -> predistorter (headline basis) -> pinned host, 2^25 samples"}
    for chunk in (1 << 20, 1 << 21, 1 << 22):
        pipe = ingest.HostPipeline(plan, chunk=chunk, nbuf=3)
        pipe.run(xh, zh)
        ts = []
        for _ in range(reps):
            pipe.reset()
            t0 = time.perf_counter()
            pipe.run(xh, zh)
            ts.append(time.perf_counter() - t0)
        t = float(np.median(ts))
        out["chunk_2^%d" % (chunk.bit_length() - 1)] = {
            "ms": round(t * 1e3, 2), "msamples_per_s": round(n / t / 1e6, 1),
            "host_link_gbs_each_way": round(8 * n / t / 1e9, 2)}
        del pipe
    # the same copies with no filtering (the host-link ceiling of this pattern)
    chunk = 1 << 21
    ss = [torch.cuda.Stream() for _ in range(3)]
    bufs = [torch.empty(chunk, dtype=torch.complex64, device="cuda") for _ in ss]

    def copies():
        for i, t0 in enumerate(range(0, n, chunk)):
            with torch.cuda.stream(ss[i % 3]):
                bufs[i % 3].copy_(xh[t0:t0 + chunk], non_blocking=True)
                zh[t0:t0 + chunk].copy_(bufs[i % 3], non_blocking=True)
        for q in ss:
            q.synchronize()

    copies()
    ts = []
    for _ in range(reps):
        t0 = time.perf_counter()
        copies()
        ts.append(time.perf_counter() - t0)
    t = float(np.median(ts))
    out["copies_only_chunk_2^21"] = {"ms": round(t * 1e3, 2), "host_link_gbs_each_way": round(8 * n / t / 1e9, 2)}
    # zero copy: one launch that reads and writes the pinned buffers in place
    zc = ingest.ZeroCopy(plan)
    zc.run(xh, zh)
    ts = []
    for _ in range(reps):
        t0 = time.perf_counter()
        zc.run(xh, zh)
        ts.append(time.perf_counter() - t0)
    t = float(np.median(ts))
    out["zero_copy"] = {"ms": round(t * 1e3, 2), "msamples_per_s": round(n / t / 1e6, 1),
                        "host_link_gbs_each_way": round(8 * n / t / 1e9, 2)}
    ref = _oracle().forward(xh.numpy(), orders, orders, L, signals.aph_coeffs(orders, orders, L, config_id=1))
    out["accuracy_zero_copy"] = gate(zh.numpy(), ref)
    pipe = ingest.HostPipeline(plan)
    zh.fill_(0)
    pipe.run(xh, zh)
    out["accuracy_pipeline"] = gate(zh.numpy(), ref)
    return out


def leg_ls(torch, dpd, signals, reps=5):
    """Least-squares estimation (section 2.2, Eq. 2) with the headline basis
    (orders {1,3,5,7} both branches, L = 4, K = 33): the matrix-core normal
    equations over 2^20 and 2^24 samples, the FP64 Cholesky solve, and the
    indirect-learning loop on the synthetic PA (2^18 samples, RMS 0.2)."""
    from paper_1612_09001_amd import autotune, ila

    orders, L = [1, 3, 5, 7], 4
    plan = dpd.Plan(orders, orders, L, signals.aph_coeffs(orders, orders, L, config_id=1))
    K = plan.K
    D = 2 * K + 2
    Dp = (D + 15) // 16 * 16
    nt = Dp // 16
    useful = D * (D + 1)                     # upper triangle of the real Gram, flops per sample
    # bf16 matrix operations issued per sample: every 16x16 tile pair takes a
    # 16x16x32 product per 8 samples (each FP32 feature as a bf16 high and low
    # part, the four cross products summed in FP32)
    issued = nt * (nt + 1) // 2 * 16 * 16 * 32 * 2 // 8
    st = dpd.current_stream()
    out = {"workload": "normal equations of the K=33 headline basis; Cholesky solve; indirect learning",
           "K": K, "real_features": D, "useful_flops_per_sample": useful, "mfma_bf16_flops_per_sample": issued}
    m = _metrics()
    orc = _oracle()
    for lg in (20, 24):
        n = 1 << lg
        y_host = signals.ofdm_16qam(n, config_id=1)
        t_host = signals.ofdm_16qam(n, config_id=1, stream_id=2)
        y = torch.from_numpy(y_host).cuda()
        t = torch.from_numpy(t_host).cuda()
        A = torch.empty((K, K), dtype=torch.complex128, device="cuda")
        b = torch.empty(K, dtype=torch.complex128, device="cuda")
        wsb = dpd.dpd_ls_ws_size(plan.handle, 1, n)
        ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
        us = autotune.time_us(lambda: dpd.dpd_ls_normal(plan.handle, st, y.data_ptr(), t.data_ptr(), 1, n, n, 1.0,
                                                        ws.data_ptr(), wsb, A.data_ptr(), b.data_ptr()),
                              warmup=20, iters=4 * reps)   # steady clocks: ~30 ms of work at 2^24
        out["normal_2^%d_us" % lg] = round(us, 1)
        out["normal_2^%d_useful_tflops" % lg] = round(useful * n / (us * 1e-6) / 1e12, 2)
        out["normal_2^%d_mfma_bf16_tflops" % lg] = round(issued * n / (us * 1e-6) / 1e12, 2)
        out["normal_2^%d_mfma_bf16_frac" % lg] = round(issued * n / (us * 1e-6) / 1e12 / MFMA_BF16_TFLOPS, 4)
        (Ar, br), t_cpu = _timed(lambda: orc.ls_normal(y_host, orders, orders, L, t_host))
        ea, eb, ma, mb = m.ls_errors(A.cpu().numpy(), b.cpu().numpy(), Ar, br,
                                     float(np.sum(np.abs(t_host.astype(np.complex128)) ** 2)))
        out["normal_2^%d_accuracy" % lg] = {"A_scaled_frob": float("%.3g" % ea), "b_scaled_frob": float("%.3g" % eb),
                                            "A_scaled_entry_max": float("%.3g" % ma),
                                            "b_scaled_entry_max": float("%.3g" % mb),
                                            "pass": bool(max(ea, eb, ma, mb) <= m.LS_REL_MAX)}
        CPU_EXTRA["ls_normal_2^%d" % lg] = {"msamples_per_s": round(n / t_cpu / 1e6, 3), "cores": orc.threads(),
                                           "sample": "the whole 2^%d-sample fit, one run" % lg}
        del y, t, ws
    h, info = dpd.ls_solve(A, b, 1e-9)
    swsb = dpd.dpd_ls_solve_ws_size(K)
    sws = torch.empty(swsb, dtype=torch.uint8, device="cuda")
    out["solve_us"] = round(autotune.time_us(
        lambda: dpd.dpd_ls_solve(st, K, A.data_ptr(), b.data_ptr(), 1e-9, sws.data_ptr(), swsb, h.data_ptr(),
                                 info.data_ptr()), warmup=2, iters=max(reps, 20)), 1)
    from paper_1612_09001_amd import spectral

    x = torch.from_numpy(signals.ofdm_16qam(1 << 18, config_id=5, rms=0.2)).cuda()
    est = ila.ILA(x, orders, orders, L)
    xh = x.cpu().numpy()

    def regrowth():
        _, y = est.transmit()
        return round(spectral.distortion_regrowth_db(y.cpu().numpy() / est.pa.gain, xh), 2)

    out["guard_band_distortion_db_no_dpd"] = regrowth()
    warm = ila.ILA(x, orders, orders, L)   # first launches of every kernel on the way
    warm.step()
    torch.cuda.synchronize()
    del warm
    e = [est.nmse_db()]
    times = []
    for _ in range(3):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        est.step()
        torch.cuda.synchronize()
        times.append(time.perf_counter() - t0)
        e.append(est.nmse_db())
    out["ila_iteration_ms_2^18"] = round(float(np.median(times)) * 1e3, 3)
    out["ila_nmse_db_iters_0_to_3"] = [round(v, 2) for v in e]
    out["guard_band_distortion_db_after_3_iters"] = regrowth()
    out["ila_solve_info"] = int(est.info.item())
    # the same three iterations composed from FP64 oracle calls
    import oracle.ila as oila
    ref, _ = oila.run(orc, xh, (orders, orders), L, signals.identity_coeffs(orders, orders, L), 3, ridge=est.ridge)
    out["ila_fp64_nmse_db_iters_0_to_3"] = [round(v, 2) for v in ref]
    out["ila_max_abs_diff_db_vs_fp64"] = round(float(np.max(np.abs(np.array(e) - np.array(ref)))), 3)
    # the non-contiguous two-carrier signal (gap between the carriers)
    x2h = signals.two_carrier(1 << 18, config_id=3, stream_id=5, rms=0.2)
    est2 = ila.ILA(torch.from_numpy(x2h).cuda(), orders, orders, L)

    def regrowth2():
        _, y2 = est2.transmit()
        return round(spectral.distortion_regrowth_db(y2.cpu().numpy() / est2.pa.gain, x2h,
                                                     bands=spectral.TWO_CARRIER), 2)

    out["two_carrier_gap_distortion_db_no_dpd"] = regrowth2()
    for _ in range(3):
        est2.step()
    out["two_carrier_gap_distortion_db_after_3_iters"] = regrowth2()
    out["two_carrier_ila_solve_info"] = int(est2.info.item())
    _, y2 = oila.transmit(orc, x2h, (orders, orders), L, est2.h.cpu().numpy())
    out["two_carrier_gap_distortion_db_after_3_iters_fp64_chain"] = round(
        spectral.distortion_regrowth_db(y2[0] / oila.GAIN, x2h, bands=spectral.TWO_CARRIER), 2)
    return out


def learn_step_work(NI, L, NIB=3, LB=3):
    """Arithmetic (flops, a multiply-add counted as two) and HBM bytes per
    sample of one learning step as one pass: the predistorter (NI power levels,
    L taps), the memoryless I/Q stage, the PA (NIB levels, LB taps) and the loss
    forward; the two stage adjoints and the predistorter's coefficient gradient
    backward.  Bytes: x read, z and dE/dy written."""
    fwd = ((8 * NI * L + 3)                  # predistorter: 2x2 matrices by Horner in |x|^2, and |x|^2
           + (8 + 3)                         # I/Q stage (one level) and |u|^2
           + (8 * NIB * LB + 3)              # PA and the |u|^2 it reads
           + 10)                             # residual, squared error, dE/dy
    bwd = (8 * NIB * LB                      # U_j = sum_k M^T g for the PA
           + 10 * (NIB - 1) + 4              # P + 2 Q u by Horner
           + 8                               # I/Q stage transpose
           + 8 * NI * L + 6 * (NI - 1) + 4)  # coefficient gradient, powers of |x|^2 times v, sum of G
    return fwd, bwd, 24


def _learn_roofline(samples, ms, orders, L):
    ni = (max(orders) + 1) // 2
    fwd, bwd, nbytes = learn_step_work(ni, L)
    t = ms * 1e-3
    return {"flops_per_sample": fwd + bwd, "bytes_per_sample": nbytes,
            "valu_tflops": round(samples * (fwd + bwd) / t / 1e12, 2),
            "valu_frac": round(samples * (fwd + bwd) / t / 1e12 / VALU_FP32_PEAK_TFLOPS, 4),
            "hbm_frac": round(samples * nbytes / t / 1e9 / HBM_PEAK_GBS, 4),
            "note": "the whole step (two launches) against the FP32 VALU peak at 2.4 GHz and HBM peak"}


def leg_config5(torch, dpd, signals, steps=200, plain_steps=20):
    """64 x 2^18 samples, DPD orders {1,3,5,7} both branches, L = 6, identity
    start, synthetic PA, loss mean|y/10 - x|^2, Adam lr 1e-3: the fused step
    (transmitter, loss, adjoint and gradient in one kernel, Adam in another), the
    same step with the transmitter as separate launches per stage, autograd over
    DPDFunction nodes and plain-ops autograd."""
    from paper_1612_09001_amd.baselines import PlainTrainer
    from paper_1612_09001_amd.train import AutogradTrainer, FusedTrainer

    orders, L, rows, n = [1, 3, 5, 7], 6, 64, 1 << 18
    x = np.stack([signals.ofdm_16qam(n, config_id=5, stream_id=r) for r in range(rows)])
    xd = torch.from_numpy(x).cuda()
    h0 = signals.identity_coeffs(orders, orders, L)

    def run(tr, k):
        ms, losses = [], []
        for _ in range(k):
            e0 = torch.cuda.Event(enable_timing=True)
            e1 = torch.cuda.Event(enable_timing=True)
            e0.record()
            loss = tr.step()
            e1.record()
            losses.append(loss.clone())
            ms.append((e0, e1))
        torch.cuda.synchronize()
        run.total_ms = ms[0][0].elapsed_time(ms[-1][1])   # first step's start to the last one's end
        ms = [a.elapsed_time(b) for a, b in ms]
        return ms, [float(v.item()) for v in losses]

    # the fused step's loss and coefficient gradient at the identity against the FP64 chain (all 64 rows)
    import oracle.pa as opa
    tr0 = FusedTrainer(xd, orders, orders, L, h0, lr=0.0)
    loss0 = float(tr0.step().item())
    gc0 = tr0.gc.cpu().numpy()
    orc = _oracle()
    (E_ref, g_ref), t_cpu = _timed(lambda: opa.chain_loss_and_gradient(orc, x, (orders, orders), L, h0))
    CPU_EXTRA["config5_chain_gradient"] = {"msamples_per_s": round(rows * n / t_cpu / 1e6, 3), "cores": orc.threads(),
                                           "sample": "loss and coefficient gradient of the whole 64 x 2^18 batch "
                                                     "through the FP64 chain, one run"}
    acc = {"loss_rel": float("%.3g" % (abs(loss0 - E_ref) / E_ref)),
           "gradient": gate_dcoef(gc0, g_ref, entry_max=1e-4, rel_max=1e-4)}
    acc["pass"] = bool(acc["loss_rel"] <= 1e-5 and acc["gradient"]["pass"])
    # settle the clocks before each timed run: steps of the throwaway trainer
    # (learning rate 0) for WARM_S
    def settle():
        t0 = time.perf_counter()
        while time.perf_counter() - t0 < WARM_S:
            for _ in range(20):
                tr0.step()
            torch.cuda.synchronize()

    settle()
    trf = FusedTrainer(xd, orders, orders, L, h0)
    fused_ms, fused_loss = run(trf, steps)
    fused_b2b_ms = run.total_ms / steps
    h_fused = trf.coeffs.cpu().numpy()
    del trf
    # the same steps replayed from a graph: 20 captured dpd_learn_step_dev
    # calls (Adam's step count on the device), replayed steps / 20 times
    settle()
    trg = FusedTrainer(xd, orders, orders, L, h0, device_step=True)
    gph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(gph):
        for _ in range(20):
            trg.step()
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(steps // 20):
        gph.replay()
    e1.record()
    torch.cuda.synchronize()
    graph_ms = e0.elapsed_time(e1) / (steps // 20 * 20)
    graph_dev = float(np.max(np.abs(trg.coeffs.cpu().numpy() - h_fused)))
    del trg, gph
    settle()
    stage_ms, stage_loss = run(FusedTrainer(xd, orders, orders, L, h0, fused_transmitter=False), 50)
    settle()
    auto_ms, auto_loss = run(AutogradTrainer(xd, orders, orders, L, h0), plain_steps)
    settle()
    plain_ms, plain_loss = run(PlainTrainer(xd, orders, orders, L, h0), plain_steps)
    del tr0
    k = min(plain_steps, steps)
    agree = float(np.max(np.abs(np.array(plain_loss[:k]) - np.array(fused_loss[:k])) /
                         np.array(fused_loss[:k])))
    med = lambda v: float(np.median(v[10:] if len(v) > 12 else v[2:]))
    # suppression after the gradient-learned predistorter: the same procedure at
    # the indirect-learning drive level (RMS 0.2) with Adam lr 0.03
    from paper_1612_09001_amd import spectral
    from paper_1612_09001_amd.pa import SyntheticPA
    import oracle.ila as oila
    x2 = np.stack([signals.ofdm_16qam(n, config_id=5, stream_id=r, rms=0.2) for r in range(rows)])
    x2d = torch.from_numpy(x2).cuda()
    tr2 = FusedTrainer(x2d, orders, orders, L, h0, lr=0.03)
    for _ in range(steps):
        tr2.step()
    h2 = tr2.coeffs.cpu().numpy()
    spa = SyntheticPA()

    def guard(hh, xx=x2d, xh=x2[0]):
        pl = dpd.Plan(orders, orders, L, hh)
        _, yy = spa.forward(pl.apply(xx[0].contiguous()))
        return round(spectral.distortion_regrowth_db(yy.cpu().numpy() / spa.gain, xh), 2)

    _, y64 = oila.transmit(orc, x2[0], (orders, orders), L, h2)
    sup = {"workload": "64x2^18 OFDM-like at RMS 0.2, the same 200 Adam steps with lr 0.03",
           "guard_band_distortion_db_no_dpd": guard(h0), "guard_band_distortion_db_learned": guard(h2),
           "guard_band_distortion_db_learned_fp64_chain": round(
               spectral.distortion_regrowth_db(y64[0] / oila.GAIN, x2[0]), 2),
           "at_rms_0.25_lr_1e-3": {"guard_band_distortion_db_no_dpd": guard(h0, xd, x[0]),
                                   "guard_band_distortion_db_learned": guard(h_fused, xd, x[0])}}
    del tr2, x2d
    # the same on two non-contiguous carriers: distortion in the gap between them
    x3 = np.stack([signals.two_carrier(n, config_id=3, stream_id=r, rms=0.2) for r in range(rows)])
    x3d = torch.from_numpy(x3).cuda()
    tr3 = FusedTrainer(x3d, orders, orders, L, h0, lr=0.03)
    for _ in range(steps):
        tr3.step()
    h3 = tr3.coeffs.cpu().numpy()

    def gap(hh):
        pl = dpd.Plan(orders, orders, L, hh)
        _, yy = spa.forward(pl.apply(x3d[0].contiguous()))
        return round(spectral.distortion_regrowth_db(yy.cpu().numpy() / spa.gain, x3[0], bands=spectral.TWO_CARRIER), 2)

    _, y64 = oila.transmit(orc, x3[0], (orders, orders), L, h3)
    sup["two_carrier_gap_distortion_db_no_dpd"] = gap(h0)
    sup["two_carrier_gap_distortion_db_learned"] = gap(h3)
    sup["two_carrier_gap_distortion_db_learned_fp64_chain"] = round(
        spectral.distortion_regrowth_db(y64[0] / oila.GAIN, x3[0], bands=spectral.TWO_CARRIER), 2)
    del tr3, x3d
    return {"workload": "64x2^18 OFDM-like, DPD {1,3,5,7} main+conj L=6, synthetic PA, Adam 1e-3",
            "accuracy_step0": acc, "suppression": sup,
            "grad_step_ms_fused": round(med(fused_ms), 4),
            "grad_step_ms_fused_back_to_back": round(fused_b2b_ms, 4),
            "grad_step_ms_graph_replay": round(graph_ms, 4),
            "graph_vs_eager_coeffs_max_abs_after_%d_steps" % steps: float("%.3g" % graph_dev),
            "grad_step_roofline": _learn_roofline(rows * n, med(fused_ms), orders, L),
            "grad_step_ms_fused_transmitter_per_stage": round(med(stage_ms), 4),
            "per_stage_vs_fused_loss_rel_max_first_50": float("%.3g" % float(np.max(
                np.abs(np.array(stage_loss) - np.array(fused_loss[:50])) / np.array(fused_loss[:50])))),
            "grad_step_ms_autograd_dpdfunction": round(med(auto_ms), 4),
            "grad_step_ms_plain_ops_autograd": round(med(plain_ms), 4),
            "speedup_vs_plain_ops": round(med(plain_ms) / med(fused_ms), 2),
            "speedup_vs_autograd_dpdfunction": round(med(auto_ms) / med(fused_ms), 2),
            "loss_db_step0": round(10 * np.log10(fused_loss[0]), 2),
            "loss_db_final": round(10 * np.log10(fused_loss[-1]), 2), "steps": steps,
            "plain_vs_fused_loss_rel_max_first_%d" % k: float("%.3g" % agree)}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    # the GPU clocks need ~500 launches (~30 ms) of load to settle
    ap.add_argument("--steps", type=int, default=1000)
    ap.add_argument("--warmup", type=int, default=1000)
    ap.add_argument("--log2n", type=int, default=24)
    ap.add_argument("--no-cpu", action="store_true", help="skip the oracle leg")
    ap.add_argument("--main-only", action="store_true", help="skip the secondary workloads")
    ap.add_argument("--tune", default="", help="S,LDS[,GRID_MULT] override, e.g. 8,1,16")
    ap.add_argument("--calibrate-copy", action="store_true",
                    help="also run one plain device copy of the same bytes (counter calibration)")
    ap.add_argument("--only-leg", default="",
                    help="run only these secondary workloads (comma-separated: config1, config3, config4, "
                         "backward, config5, ls, table2, ingest, batch_classes) and print their results, "
                         "e.g. under a profiler")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py: measures one GPU only; --gpus %d is not supported (the forward map, the "
              "batch and the training step shard without cross-GPU traffic in the hot path)" % args.gpus,
              file=sys.stderr)
        sys.exit(2)

    import torch
    from paper_1612_09001_amd import dpd, signals
    legs = {"config1": leg_config1, "config3": leg_config3, "config4": leg_config4, "backward": leg_backward, "config5": leg_config5,
            "ls": leg_ls, "table2": leg_table2, "ingest": leg_ingest}
    extra_legs = {"batch_classes": leg_batch_classes}
    if args.only_leg:
        known = dict(legs, **extra_legs)
        for name in args.only_leg.split(","):
            if name not in known:
                print("bench.py: unknown workload %r (known: %s)" % (name, ", ".join(known)), file=sys.stderr)
                sys.exit(2)
            print(json.dumps({name: known[name](torch, dpd, signals)}), flush=True)
        return

    n = 1 << args.log2n
    mo = co = [1, 3, 5, 7]
    L = 4
    x_host = signals.ofdm_16qam(n, config_id=2)
    h = signals.aph_coeffs(mo, co, L, config_id=2)
    plan = dpd.Plan(mo, co, L, h)
    if args.tune:
        vals = [int(v) for v in args.tune.split(",")]
        plan.set_tune(samples_per_thread=vals[0], stage_lds=vals[1],
                      grid_mult=vals[2] if len(vals) > 2 else 16)
    tune = plan.get_tune()

    xs, zs = _rotating(torch, x_host)
    nbuf = len(xs)
    stream = dpd.current_stream()
    ptrs = [(a.data_ptr(), b.data_ptr()) for a, b in zip(xs, zs)]
    handle = plan.handle
    if args.calibrate_copy:
        zs[0].copy_(xs[0])
        torch.cuda.synchronize()

    # Warm the clocks with the one-shot variant of the filter (a different
    # kernel symbol), so a profiler's per-kernel average of the timed kernel
    # covers exactly the timed launches.
    plan.set_tune(samples_per_thread=tune["samples_per_thread"], stage_lds=0)
    for i in range(args.warmup):
        dpd.dpd_apply(handle, stream, ptrs[i % nbuf][0], ptrs[i % nbuf][1], n)
    plan.set_tune(samples_per_thread=tune["samples_per_thread"], stage_lds=tune["stage_lds"],
                  grid_mult=tune["grid_mult"])
    # a plain device copy of the same bytes over the same buffers through the
    # runtime (torch copy_ = hipMemcpyAsync), on warm clocks (the timed launches
    # then rewrite every output)
    _, copy_ms = _time_launches(torch, lambda i: zs[i].copy_(xs[i]), nbuf, min(args.steps, 200), 20)
    copy_gbs = BYTES_PER_SAMPLE * n / (copy_ms * 1e-3) / 1e9
    # the forward kernel's own memory walk without the filter (dpd_copy): the
    # practical ceiling of this access pattern
    _, walk_ms = _time_launches(torch, lambda i: dpd.dpd_copy(stream, ptrs[i][0], ptrs[i][1], n), nbuf,
                                min(args.steps, 500), 50)
    walk_gbs = BYTES_PER_SAMPLE * n / (walk_ms * 1e-3) / 1e9
    wall, kern_ms = _time_launches(
        torch, lambda i: dpd.dpd_apply(handle, stream, ptrs[i][0], ptrs[i][1], n), nbuf,
        args.steps, 1)
    ms_per_step = wall * 1e3 / args.steps
    value = n * args.steps / wall / 1e6
    achieved = BYTES_PER_SAMPLE * n / (kern_ms * 1e-3) / 1e9
    prof_ns = kernel_ns_from_profile(n)

    out = {
        "metric": METRIC,
        "value": round(value, 1),
        "unit": "Msamples/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms_per_step, 5),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic (seeded OFDM-like 16-QAM, 1200/2048 subcarriers, RMS 0.25)",
        "config": {"workload": "single stream N=2^%d complex64, orders {1,3,5,7} main+conj, "
                               "L=4, DC term, FP32 forward apply" % args.log2n,
                   "n": n, "L": L, "orders": mo, "tune": tune, "rotating_buffers": nbuf},
        "roofline": {"bound": "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS,
                     "unit": "GB/s", "frac": round(achieved / HBM_PEAK_GBS, 4),
                     "traffic": traffic_from_profile(n),
                     "kernel_ms": round(kern_ms, 5),
                     "algorithmic_bytes_per_launch": BYTES_PER_SAMPLE * n,
                     "frac_wall": round(BYTES_PER_SAMPLE * n / (ms_per_step * 1e-3) / 1e9 / HBM_PEAK_GBS, 4),
                     "frac_rocprof": (round(BYTES_PER_SAMPLE * n / (prof_ns * 1e-9) / 1e9 / HBM_PEAK_GBS, 4)
                                      if prof_ns else None),
                     "rocprof_kernel_us": round(prof_ns / 1e3, 2) if prof_ns else None,
                     "runtime_copy_gbs": round(copy_gbs, 1),
                     "frac_of_runtime_copy": round(achieved / copy_gbs, 4),
                     "copy_walk_gbs": round(walk_gbs, 1), "copy_walk_us": round(walk_ms * 1e3, 2),
                     "frac_of_copy_walk": round(achieved / walk_gbs, 4)},
    }
    z_last = zs[(args.steps - 1) % nbuf]
    if not args.main_only:
        del xs
        sec = {}
        for name, fn in legs.items():
            try:
                sec[name] = fn(torch, dpd, signals)
            except Exception as e:  # a failing secondary leg must not hide the headline
                traceback.print_exc(file=sys.stderr)
                sec[name] = {"error": "%s: %s" % (type(e).__name__, e)}
            torch.cuda.empty_cache()
        out["secondary"] = sec
    if not args.no_cpu:
        base, acc = cpu_baseline(x_host, z_last.cpu().numpy(), mo, co, L, h)
        if CPU_EXTRA:
            base["other_workloads"] = CPU_EXTRA
        out["cpu_baseline"] = base
        out["accuracy"] = acc
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
