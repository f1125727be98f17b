#!/usr/bin/env python3
"""Benchmark: chromatic Gibbs sweeps of a 2048 x 2048 lattice GMRF on one MI355X.

Workload (one "step" = one full sweep: all 4 colors, fused q / sse reductions,
posterior accumulators and the device-side tau / lam Gamma draws):
2048 x 2048 pixel lattice, 8-neighbour intrinsic CAR prior, 2x2-parity
4-coloring, y = 8x8-block piecewise-constant image + N(0, 0.1^2) noise,
Gamma(1, 1) priors on tau and lam, FP32 state / draws / neighbour sums with
FP64 accumulators and reductions, burn-in 0 (every sweep accumulates).

Prints ONE JSON line.  ``value`` is site-updates/s of the FP32 path with all
inputs resident in HBM; the line also carries the FP64 path, p50 / p99 solve
latency (1000-sweep solves) for both precisions, the roofline of the sweep
kernel, the same sweep on an 8192 x 8192 lattice (a working set far beyond
the 256 MB Infinity Cache) next to a device copy measured in the same run,
the irregular 1,000,000-site workload, the 512-instance batch, and the CPU
oracle timed on bounded samples.
"""
from __future__ import annotations

import argparse
import json
import os
import platform
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

ROWS = COLS = 2048
BIG = 8192
STENCIL = 8
HBM_PEAK_GBS = 8000.0
# algorithmic bytes per site update, accumulating sweeps: lattice x read + x
# write + y read + its share of the S1 / S2 read-modify-write and of the fields
# read back for it, once per five FP32 sweeps (12 + (32 + 16) / 5) or three
# FP64 sweeps (24 + (32 + 16) / 3); a general graph has x, y, S1 / S2 in every
# sweep, its CSR row (row offset + column indices at mean degree ~6) and the
# slab-to-id map
BYTES_PER_SITE = {"fp32_acc": 21.6, "fp64_acc": 40}
GRAPH_PROBE_SITES = 1_000_000       # sites of the Delaunay counter probe
BURN_IN_BYTES_PER_SITE = 12          # FP32 burn-in sweep: x read + x write + y read
CSR_BYTES_PER_SITE = {"fp32_acc": 72, "fp64_acc": 84}
METRIC = ("site-updates/s + HBM GB/s fraction per sweep; p50/p99 solve latency "
          "(FP32 vs FP64)")
SWEEP_KERNEL = "lattice_sweep_kernel<float, LatCfg<8, 64, 64, 512>, false, false>"
# rocprofv3 summaries of the dominant kernel (committed under profiles/):
# its average duration in the kernel trace of this benchmark's command, and
# its HBM traffic per launch from FETCH_SIZE / WRITE_SIZE scaled by a device
# copy's readings.  Each holds a "json:" line with the figures and the
# SHA-256 of the kernel sources it was taken from; a figure is reported only
# while the sources are unchanged.
PROFILES = os.path.join(ROOT, "profiles")
TRACE_SUMMARY = os.path.join(PROFILES, "lattice_sweep_2048x2048_s8_kernel_trace.md")
TRAFFIC_SUMMARY = os.path.join(PROFILES, "lattice_sweep_2048x2048_s8_fp32_traffic.md")
TRAFFIC_SUMMARY_BIG = os.path.join(PROFILES, "lattice_sweep_8192x8192_s8_fp32_traffic.md")
TRAFFIC_SUMMARY_GRAPH = os.path.join(PROFILES, "chunked_sweep_delaunay1m_traffic.md")
KERNEL_SOURCES = [os.path.join(ROOT, "paper_1702_05518_amd", "csrc", f)
                  for f in ("gmrf.hip", "rng.hpp")]


def log(msg):
    print(msg, file=sys.stderr, flush=True)


def kernel_sources_sha256() -> str:
    import hashlib

    h = hashlib.sha256()
    for f in KERNEL_SOURCES:
        with open(f, "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()


def profile_figures(path):
    """The "json:" line of a committed profile summary, if it was taken from
    the current kernel sources (else None)."""
    try:
        with open(path) as fh:
            for line in fh:
                if line.startswith("json:"):
                    d = json.loads(line[5:])
                    return d if d.get("kernel_sources_sha256") == kernel_sources_sha256() else None
    except OSError:
        pass
    return None


def _csv_rows(path):
    import csv

    with open(path, newline="") as fh:
        return list(csv.DictReader(fh))


def _short(name, width=110):
    name = name.replace("gmrf::", "")
    return name if len(name) <= width else name[:width - 3] + "..."


def trace_summary(trace_csv, commands):
    """Markdown summary of a rocprofv3 kernel trace (kernel_trace.csv): one
    row per kernel and launch size (workgroups), durations in ns, and a
    "json:" line with the sweep kernel's figures at the benchmark's size."""
    groups = {}
    total = 0
    for r in _csv_rows(trace_csv):
        if r["Kind"] != "KERNEL_DISPATCH":
            continue
        wg = int(r["Workgroup_Size_X"]) * int(r["Workgroup_Size_Y"]) * int(r["Workgroup_Size_Z"])
        blocks = int(r["Grid_Size_X"]) * int(r["Grid_Size_Y"]) * int(r["Grid_Size_Z"]) // wg
        d = int(r["End_Timestamp"]) - int(r["Start_Timestamp"])
        total += d
        groups.setdefault((r["Kernel_Name"], blocks, wg), []).append(d)
    rows = sorted(groups.items(), key=lambda kv: -sum(kv[1]))
    out = ["# Kernel trace: " + commands[0].split(" -- ", 1)[-1], "",
           "Commands (from the repository root):", "", "```", *commands, "```", "",
           "Per kernel and launch size (workgroups x threads), durations in ns:", "",
           "| Kernel | Workgroups x threads | Calls | Average | Min | Max | % of GPU time |",
           "|---|---|---|---|---|---|---|"]
    for (name, blocks, wg), ds in rows[:16]:
        out.append(f"| `{_short(name)}` | {blocks} x {wg} | {len(ds)} | {np.mean(ds):.0f} | "
                   f"{min(ds)} | {max(ds)} | {100.0 * sum(ds) / total:.2f} |")
    key = [k for k in groups if SWEEP_KERNEL.replace(" ", "") in
           k[0].replace("gmrf::", "").replace(" ", "") and k[1] == (ROWS // 64) * (COLS // 64)]
    fig = None
    if key:
        ds = groups[key[0]]
        fig = {"kernel": SWEEP_KERNEL, "workgroups": key[0][1], "calls": len(ds),
               "avg_ns": float(np.mean(ds)), "kernel_sources_sha256": kernel_sources_sha256()}
    return "\n".join(out), fig


def traffic_summary(fetch_csv, write_csv, dram_csv, side, commands):
    """Markdown summary of the counter probes (bench.py --probe): FETCH_SIZE
    and WRITE_SIZE of the sweep kernel at side x side, each scaled by the
    counter's reading for the probe's 512 MiB device copy, and, from a third
    run, the share of the L2's read and write requests that went to DRAM."""
    def per_kernel(path, counter):
        copy, sweep = [], []
        for r in _csv_rows(path):
            if r["Counter_Name"] != counter:
                continue
            v = float(r["Counter_Value"])
            if r["Kernel_Name"] == "__amd_rocclr_copyBuffer":
                copy.append(v)
            elif _sweep_variant(r["Kernel_Name"]) == "fp32 v1":
                sweep.append(v)
        return max(copy), sweep

    copy_kib = 512 * 1024
    f_copy, f_sweep = per_kernel(fetch_csv, "FETCH_SIZE")
    w_copy, w_sweep = per_kernel(write_csv, "WRITE_SIZE")
    f_scale, w_scale = copy_kib / f_copy, copy_kib / w_copy
    fetch_b = float(np.mean(f_sweep)) * f_scale * 1024
    write_b = float(np.mean(w_sweep)) * w_scale * 1024
    n = side * side
    alg = BYTES_PER_SITE["fp32_acc"] * n
    out = [f"# HBM traffic counters: FP32 lattice sweep kernel, {side}x{side}, 8 neighbours", "",
           "Commands (from the repository root):", "", "```", *commands, "```", "",
           "`bench.py --probe` first copies 512 MiB device-to-device (one dispatch of the "
           "runtime's `__amd_rocclr_copyBuffer`), which must read and write exactly 524288 "
           "KiB: its readings give each counter's scale.", "",
           "| Quantity | FETCH_SIZE (KiB) | WRITE_SIZE (KiB) |", "|---|---|---|",
           f"| 512 MiB copy, counter | {f_copy:.1f} | {w_copy:.1f} |",
           f"| scale factor = 524288 / counter | {f_scale:.3f} | {w_scale:.3f} |",
           f"| sweep kernel, counter, mean of {len(f_sweep)} launches | "
           f"{np.mean(f_sweep):.1f} | {np.mean(w_sweep):.1f} |",
           f"| sweep kernel, scaled, MB per launch | {fetch_b / 1e6:.1f} | {write_b / 1e6:.1f} |",
           "", f"Scaled traffic per launch: {(fetch_b + write_b) / 1e6:.1f} MB, against "
           f"{alg / 1e6:.1f} MB of algorithmic bytes (21.6 B per site).", ""]
    fig = {"kernel": SWEEP_KERNEL, "side": side, "bytes_per_launch": fetch_b + write_b,
           "fetch_bytes": fetch_b, "write_bytes": write_b, "fetch_scale": f_scale,
           "write_scale": w_scale, "kernel_sources_sha256": kernel_sources_sha256()}
    if dram_csv:
        tot = {}
        for r in _csv_rows(dram_csv):
            if _sweep_variant(r["Kernel_Name"]) == "fp32 v1":
                tot.setdefault(r["Counter_Name"], []).append(float(r["Counter_Value"]))
        rd = np.mean(tot["TCC_EA0_RDREQ_DRAM_sum"]) / np.mean(tot["TCC_EA0_RDREQ_sum"])
        wr = np.mean(tot["TCC_EA0_WRREQ_DRAM_sum"]) / np.mean(tot["TCC_EA0_WRREQ_sum"])
        out += ["Requests from the L2 to the fabric that went to DRAM (TCC_EA0_RDREQ_DRAM_sum / "
                "TCC_EA0_RDREQ_sum, TCC_EA0_WRREQ_DRAM_sum / TCC_EA0_WRREQ_sum, means over the "
                "sweep launches):", "",
                "| | L2 requests | to DRAM | share | DRAM bytes (share x scaled bytes) |",
                "|---|---|---|---|---|",
                f"| reads | {np.mean(tot['TCC_EA0_RDREQ_sum']):.0f} | "
                f"{np.mean(tot['TCC_EA0_RDREQ_DRAM_sum']):.0f} | {rd:.3f} | "
                f"{rd * fetch_b / 1e6:.1f} MB |",
                f"| writes | {np.mean(tot['TCC_EA0_WRREQ_sum']):.0f} | "
                f"{np.mean(tot['TCC_EA0_WRREQ_DRAM_sum']):.0f} | {wr:.3f} | "
                f"{wr * write_b / 1e6:.1f} MB |", ""]
        fig.update(dram_read_share=float(rd), dram_write_share=float(wr),
                   dram_bytes=float(rd * fetch_b + wr * write_b))
    return "\n".join(out), fig


def _fused_variant(name):
    """'fp32' / 'fp64' for the chunked general-graph sweep kernel without an
    intercept, else None."""
    n = name.replace("gmrf::", "").replace(" ", "")
    for real, tag in (("float", "fp32"), ("double", "fp64")):
        if f"csr_fused_kernel<{real},false,false>" in n:
            return tag
    return None


def graph_traffic_summary(fetch_csv, write_csv, commands):
    """Markdown summary of the counter probes of the 1,000,000-site Delaunay
    workload (bench.py --probe --probe-graph): FETCH_SIZE and WRITE_SIZE of the
    chunked sweep kernel, FP32 and FP64, each scaled by the counter's reading
    for the probe's 512 MiB device copy, against the algorithmic bytes."""
    def per_kernel(path, counter):
        copy, sweep = [], {}
        for r in _csv_rows(path):
            if r["Counter_Name"] != counter:
                continue
            v = float(r["Counter_Value"])
            if r["Kernel_Name"] == "__amd_rocclr_copyBuffer":
                copy.append(v)
            else:
                tag = _fused_variant(r["Kernel_Name"])
                if tag:
                    sweep.setdefault(tag, []).append(v)
        return max(copy), sweep

    copy_kib = 512 * 1024
    f_copy, f_sweep = per_kernel(fetch_csv, "FETCH_SIZE")
    w_copy, w_sweep = per_kernel(write_csv, "WRITE_SIZE")
    f_scale, w_scale = copy_kib / f_copy, copy_kib / w_copy
    n = GRAPH_PROBE_SITES
    out = ["# HBM traffic counters: chunked general-graph sweep kernel, Delaunay graph of "
           "1,000,000 sites", "",
           "Commands (from the repository root):", "", "```", *commands, "```", "",
           "`bench.py --probe --probe-graph` first copies 512 MiB device-to-device (one dispatch "
           "of the runtime's `__amd_rocclr_copyBuffer`), which must read and write exactly "
           "524288 KiB: its readings give each counter's scale.", "",
           f"Scale factors: FETCH_SIZE {f_scale:.3f} (the copy's reading {f_copy:.1f} KiB), "
           f"WRITE_SIZE {w_scale:.3f} (the copy's reading {w_copy:.1f} KiB).", "",
           "| Kernel | launches | FETCH_SIZE, scaled MB | WRITE_SIZE, scaled MB | total MB | "
           "B per site | algorithmic B per site |", "|---|---|---|---|---|---|---|"]
    fig = {"sites": n, "fetch_scale": f_scale, "write_scale": w_scale,
           "kernel_sources_sha256": kernel_sources_sha256()}
    for tag, prec in (("fp32", "fp32_acc"), ("fp64", "fp64_acc")):
        if tag not in f_sweep or tag not in w_sweep:
            continue
        fb = float(np.mean(f_sweep[tag])) * f_scale * 1024
        wb = float(np.mean(w_sweep[tag])) * w_scale * 1024
        out.append(f"| `csr_fused_kernel` {tag} | {len(f_sweep[tag])} | {fb / 1e6:.1f} | "
                   f"{wb / 1e6:.1f} | {(fb + wb) / 1e6:.1f} | {(fb + wb) / n:.1f} | "
                   f"{CSR_BYTES_PER_SITE[prec]} |")
        fig[tag] = {"fetch_bytes": fb, "write_bytes": wb, "bytes_per_site": (fb + wb) / n}
    out += ["", "The algorithmic bytes count each site's value, y, accumulators and CSR "
            "adjacency (4-byte column indices) once per sweep.  The kernel reads instead its "
            "chunk tables (16-bit local rows and neighbours, slab positions, original ids) "
            "and re-reads the values of each chunk's halo and recomputed closure.  The "
            "counters measure the L2's traffic to the fabric, Infinity Cache hits included.",
            ""]
    return "\n".join(out), fig


def _sweep_variant(name):
    """'fp32 v1' etc. for a 64 x 64 8-neighbour lattice sweep kernel without
    an intercept, else None."""
    n = name.replace("gmrf::", "").replace(" ", "")
    for real, tag in (("float", "fp32"), ("double", "fp64")):
        for v2, ver in (("false", "v1"), ("true", "v2")):
            if f"lattice_sweep_kernel<{real},LatCfg<8,64,64,512>,false,{v2}>" in n:
                return f"{tag} {ver}"
    return None


def counter_summary(csvs, commands):
    """Markdown summary of counter probes (bench.py --probe): the mean of
    every counter over each sweep kernel's launches (FP32 / FP64, random-number
    contract 1 / 2), per launch and per wave (SQ_WAVES)."""
    vals = {}
    for path in csvs:
        for r in _csv_rows(path):
            k = _sweep_variant(r["Kernel_Name"])
            if k:
                vals.setdefault(k, {}).setdefault(r["Counter_Name"], []).append(
                    float(r["Counter_Value"]))
    kinds = sorted(vals)
    out = [f"# Counters: lattice sweep kernels, {ROWS}x{COLS}, 8 neighbours", "",
           "Commands (from the repository root):", "", "```", *commands, "```", "",
           "Mean over each kernel's launches in the probe (" +
           ", ".join(f"{k}: {len(next(iter(vals[k].values())))}" for k in kinds) +
           "), per wave (SQ_WAVES per launch in the last row):", "",
           "| Counter | " + " | ".join(kinds) + " |", "|---|" + "---|" * len(kinds)]
    names = sorted({c for k in kinds for c in vals[k]} - {"SQ_WAVES"})
    for c in names:
        cells = []
        for k in kinds:
            w = np.mean(vals[k]["SQ_WAVES"]) if "SQ_WAVES" in vals[k] else None
            m = float(np.mean(vals[k][c])) if c in vals[k] else None
            cells.append("" if m is None else (f"{m / w:.1f}" if w else f"{m:.0f} (launch)"))
        out.append(f"| {c} | " + " | ".join(cells) + " |")
    out.append("| SQ_WAVES | " + " | ".join(
        f"{np.mean(vals[k]['SQ_WAVES']):.0f}" if "SQ_WAVES" in vals[k] else "" for k in kinds) +
        " |")
    return "\n".join(out), None


def timed_sweeps(torch, chain, steps, capture):
    """Run `steps` sweeps bracketed by events on torch's current stream (the
    stream the library launches on); returns elapsed seconds."""
    s = torch.cuda.current_stream()
    torch.cuda.synchronize()
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    e0.record(s)
    chain.sweep(steps, hyper=True, capture=capture)
    e1.record(s)
    torch.cuda.synchronize()
    return e0.elapsed_time(e1) / 1e3


def dispatch_timed(torch, chain, steps):
    """`steps` sweeps in which every sweep kernel is bracketed by HIP events
    that its dispatch records (a diagnostic: an event on a dispatch makes the
    kernel write its caches back at its end, which lengthens it).  Returns
    the average duration in seconds of the sweep kernel."""
    torch.cuda.synchronize()
    k_ms = chain.sweep_timed(steps, hyper=True)
    return k_ms / steps / 1e3


def solve_latencies(torch, chain, sweeps, reps):
    """Wall time of `reps` solves: `sweeps` sweeps + posterior mean/variance
    into device buffers, each bracketed by events."""
    n = chain.n
    m = torch.empty(n, dtype=torch.float64, device="cuda")
    v = torch.empty_like(m)
    s = torch.cuda.current_stream()
    out = []
    for _ in range(reps):
        a = torch.cuda.Event(enable_timing=True)
        b = torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        a.record(s)
        chain.sweep(sweeps, hyper=True, capture=True)
        chain.posterior_stats_device(m, v)
        b.record(s)
        torch.cuda.synchronize()
        out.append(a.elapsed_time(b))
    return out


def host_to_host_solve(torch, gmrf, graph, y, sweeps):
    """One solve from host arrays to host arrays, for the rate that includes
    the transfers over PCIe: chain creation (device workspace, upload of y,
    the state's layout), `sweeps` sweeps with plain launches (a fresh chain
    has no recorded graph), and the posterior mean / variance copied back to
    host memory.  Returns seconds."""
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    ch = gmrf.Chain(graph, y, precision=gmrf.FP32_ACC64, seed=7)
    ch.sweep(sweeps, hyper=True)
    mean, var, nacc = ch.posterior_stats()        # host pointers: synchronises
    dt = time.perf_counter() - t0
    if nacc != sweeps or not np.isfinite(mean).all():
        print("bench.py: host-to-host solve failed", file=sys.stderr)
        sys.exit(1)
    del ch
    return dt


def graph_seconds(torch, run, steps, reps=3):
    """Best of `reps` timed replays of a captured graph of `steps` sweeps
    (`run(capture)` enqueues them; the first call records the graph)."""
    run(True)
    torch.cuda.synchronize()
    s = torch.cuda.current_stream()
    best = float("inf")
    for _ in range(reps):
        e0 = torch.cuda.Event(enable_timing=True)
        e1 = torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        e0.record(s)
        run(True)
        e1.record(s)
        torch.cuda.synchronize()
        best = min(best, e0.elapsed_time(e1) / 1e3)
    return best


def copy_gbs(torch, nbytes=1 << 30, reps=5):
    """A plain device copy of nbytes (read + write counted) at its best of reps."""
    src = torch.ones(nbytes // 4, dtype=torch.float32, device="cuda")
    dst = torch.empty_like(src)
    dst.copy_(src)
    torch.cuda.synchronize()
    s = torch.cuda.current_stream()
    best = float("inf")
    for _ in range(reps):
        e0 = torch.cuda.Event(enable_timing=True)
        e1 = torch.cuda.Event(enable_timing=True)
        e0.record(s)
        dst.copy_(src)
        e1.record(s)
        torch.cuda.synchronize()
        best = min(best, e0.elapsed_time(e1) / 1e3)
    del src, dst
    torch.cuda.empty_cache()
    return 2.0 * nbytes / best / 1e9


def rng_v2_row(torch, gmrf, graph, y, args):
    """The same workload under the paired random-number contract (version 2:
    one Philox block and one Box-Muller radius per rank pair of a color), FP32
    and FP64, timed like the headline."""
    n = ROWS * COLS
    out = {"covers": "lattice 2048x2048 8-neighbour, rng_version 2 (pairs (r, c), (r, c + 2) "
                     "of a color share one Philox block: cosine and sine branches)"}
    for name, prec in (("fp32_acc", gmrf.FP32_ACC64), ("fp64_acc", gmrf.FP64)):
        if name == "fp64_acc" and args.no_fp64:
            continue
        chain = gmrf.Chain(graph, y, precision=prec, seed=1, rng_version=2)
        chain.sweep(args.warmup, hyper=True)
        chain.sweep(args.steps, hyper=True, capture=True)
        torch.cuda.synchronize()
        t = min(timed_sweeps(torch, chain, args.steps, capture=False),
                timed_sweeps(torch, chain, args.steps, capture=True))
        k_disp = dispatch_timed(torch, chain, args.steps)
        x, tau, lam, _ = chain.get_state()
        if not (np.isfinite(tau) and np.isfinite(lam)):
            print("bench.py: non-finite result (rng_version 2)", file=sys.stderr)
            sys.exit(1)
        bps = BYTES_PER_SITE[name]
        out[name] = {"value": n * args.steps / t, "unit": "site-updates/s",
                     "ms_per_step": t / args.steps * 1e3,
                     "hbm_frac": bps * n / (t / args.steps) / 1e9 / HBM_PEAK_GBS,
                     "kernel_us_dispatch_events": k_disp * 1e6}
        log(f"[bench] rng v2 {name}: {t / args.steps * 1e6:.1f} us/sweep "
            f"({out[name]['hbm_frac']:.3f} of peak)")
        del chain
        torch.cuda.synchronize()
    return out


def big_lattice_row(torch, gmrf, inputs, args):
    """The same FP32 accumulating sweep on an 8192 x 8192 lattice (about 2.9 GB
    per sweep), beyond the 256 MB Infinity Cache, with a 1 GiB device copy
    timed in the same run as the practical ceiling."""
    log(f"[bench] {BIG}x{BIG} lattice (out of cache)")
    copy = copy_gbs(torch)
    nb = BIG * BIG
    wl = inputs.lattice_workload(BIG, BIG, STENCIL, noise_sd=0.1, data_seed=1, with_csr=False)
    g = gmrf.Graph(lattice=(BIG, BIG, STENCIL))
    ch = gmrf.Chain(g, wl["y"], precision=gmrf.FP32_ACC64, seed=1)
    del wl
    ch.sweep(args.warmup, hyper=True)
    steps = max(args.steps, 10)
    t = graph_seconds(torch, lambda cap: ch.sweep(steps, hyper=True, capture=cap), steps)
    _, tau, lam, _ = ch.get_state()
    if not (np.isfinite(tau) and np.isfinite(lam)):
        print("bench.py: non-finite result (8192 lattice)", file=sys.stderr)
        sys.exit(1)
    launch_s = t / steps
    gbs = BYTES_PER_SITE["fp32_acc"] * nb / launch_s / 1e9
    del ch
    torch.cuda.empty_cache()
    row = {"workload": f"lattice {BIG}x{BIG}, 8-neighbour, FP32 with FP64 accumulators, "
                       f"accumulating sweeps (working set ~2.9 GB)",
           "sites": nb, "steps": steps, "site_updates_per_s": nb / launch_s,
           "ms_per_step": launch_s * 1e3, "achieved_gbs": gbs,
           "frac": gbs / HBM_PEAK_GBS, "copy_gbs": copy, "frac_of_copy": gbs / copy,
           "bytes_per_site": BYTES_PER_SITE["fp32_acc"]}
    traffic = profile_figures(TRAFFIC_SUMMARY_BIG)
    row["traffic"] = traffic["bytes_per_launch"] if traffic else None
    row["traffic_unit"] = ("bytes/launch (rocprofv3 FETCH_SIZE + WRITE_SIZE scaled by a device "
                           "copy's reading; every such request goes to the memory side)")
    log(f"[bench] {BIG}x{BIG}: {launch_s * 1e6:.1f} us per sweep, {gbs:.0f} GB/s "
        f"({gbs / HBM_PEAK_GBS:.3f} of peak, {gbs / copy:.3f} of a {copy:.0f} GB/s copy)")
    return row


def delaunay_row(torch, gmrf, inputs, args, wl):
    """The irregular workload at 1,000,000 sites (Delaunay, proper CAR rho
    0.95, greedy coloring), FP32 with FP64 accumulators and FP64."""
    log("[bench] Delaunay 1M")
    color, k = gmrf.greedy_coloring(wl["row_ptr"], wl["col"])
    g = gmrf.Graph(row_ptr=wl["row_ptr"], col_idx=wl["col"], color=color, num_colors=k, rho=0.95)
    n = wl["n"]
    row = {"workload": "Delaunay graph of 1,000,000 uniform points, proper CAR rho 0.95, "
                       f"greedy coloring ({k} colors), accumulating sweeps",
           "sites": n, "colors": int(k)}
    steps = max(args.steps, 10)
    traffic = profile_figures(TRAFFIC_SUMMARY_GRAPH)
    for name, prec in (("fp32_acc", gmrf.FP32_ACC64), ("fp64_acc", gmrf.FP64)):
        ch = gmrf.Chain(g, wl["y"], precision=prec, seed=5, instance=1)
        ch.sweep(args.warmup, hyper=True)
        t = graph_seconds(torch, lambda cap: ch.sweep(steps, hyper=True, capture=cap), steps)
        sweep_s = t / steps
        gbs = CSR_BYTES_PER_SITE[name] * n / sweep_s / 1e9
        row[name] = {"site_updates_per_s": n / sweep_s, "us_per_sweep": sweep_s * 1e6,
                     "achieved_gbs": gbs, "frac": gbs / HBM_PEAK_GBS,
                     "bytes_per_site": CSR_BYTES_PER_SITE[name], "shape": ch.tile[0]}
        tag = name[:4]
        if traffic and traffic["sites"] == n and tag in traffic:
            t = traffic[tag]
            row[name]["traffic"] = t["fetch_bytes"] + t["write_bytes"]
            row[name]["traffic_unit"] = ("bytes/launch of csr_fused_kernel (rocprofv3 FETCH_SIZE + "
                                         "WRITE_SIZE scaled by a device copy's reading)")
        log(f"[bench] Delaunay 1M {name}: {sweep_s * 1e6:.1f} us per sweep "
            f"({gbs / HBM_PEAK_GBS:.3f} of peak)")
        del ch
    return row


def batch_row(torch, gmrf, inputs, args, steps=None):
    """512 independent instances (256 lattices with side U{32..512}, 4
    neighbours; 256 Delaunay graphs with n U{1k..50k}, proper CAR rho 0.95),
    FP32 state with FP64 accumulators, advanced together by shared launches in
    a captured graph of sweeps."""
    steps = max(args.steps, 10) if steps is None else steps
    t0 = time.perf_counter()
    mix = inputs.batch_mix(512, data_seed=4, workers=min(16, os.cpu_count() or 1))
    log(f"[bench] batch inputs built in {time.perf_counter() - t0:.1f} s")
    chains, sites, nbytes = [], 0, 0
    for i, wl in enumerate(mix):
        if wl["kind"] == "lattice":
            g = gmrf.Graph(lattice=(wl["rows"], wl["cols"], wl["stencil"]))
            nbytes += BYTES_PER_SITE["fp32_acc"] * wl["n"]
        else:
            color, k = gmrf.greedy_coloring(wl["row_ptr"], wl["col"])
            g = gmrf.Graph(row_ptr=wl["row_ptr"], col_idx=wl["col"], color=color, num_colors=k,
                           rho=wl["rho"])
            nbytes += CSR_BYTES_PER_SITE["fp32_acc"] * wl["n"]
        chains.append(gmrf.Chain(g, wl["y"], precision=gmrf.FP32_ACC64, seed=1 + i, instance=i))
        sites += wl["n"]
    batch = gmrf.Batch(chains)
    tile, tile_us = batch.autotune(reps=10)
    batch.sweep(args.warmup, capture=False)
    t_batch = graph_seconds(torch, lambda cap: batch.sweep(steps, capture=cap), steps)
    for c in chains[:: len(chains) // 8]:
        _, tau, lam, _ = c.get_state()
        if not (np.isfinite(tau) and np.isfinite(lam)):
            print("bench.py: non-finite result (batch)", file=sys.stderr)
            sys.exit(1)
    sweep_s = t_batch / steps
    gbs = nbytes / sweep_s / 1e9
    log(f"[bench] batch512: {sweep_s * 1e3:.3f} ms per sweep of all chains, "
        f"{sites / sweep_s:.3e} site-updates/s ({gbs / HBM_PEAK_GBS:.3f} of peak)")
    return {"workload": "512 instances: 256 lattices side U{32..512} 4-neighbour, 256 Delaunay "
                        "graphs n U{1k..50k}, FP32 with FP64 accumulators, one captured graph "
                        "of shared launches",
            "instances": len(chains), "sites_per_sweep": sites, "steps": steps,
            "site_updates_per_s": sites / sweep_s, "ms_per_sweep": sweep_s * 1e3,
            "achieved_gbs": gbs, "frac": gbs / HBM_PEAK_GBS,
            "lattice_tile_autotune": {"chosen_shape": tile, "us_per_pass_64x64": tile_us[0],
                                      "us_per_pass_32x32": tile_us[1]}, "_chains": chains}


def cpu_baseline(wl, seconds_budget=10.0, wl1m=None):
    """The oracle (C, FP64) on bounded samples: the 2048 x 2048 workload with
    every host thread (up to 16) and with one, the 64 x 64 workload in full,
    the irregular 15,000-site workload in full (2000 sweeps) and, given the
    1,000,000-site workload, a bounded number of its sweeps."""
    import oracle

    oracle.build(force=False)
    threads = min(16, os.cpu_count() or 1)
    model = ""
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                model = line.split(":", 1)[1].strip()
                break
    except OSError:
        pass

    def timed(ch, n, budget, nthreads, cap=2000):
        t0 = time.perf_counter()
        ch.sweeps(1, nthreads=nthreads)
        one = time.perf_counter() - t0
        reps = max(1, min(cap, int(budget / max(one, 1e-4))))
        t0 = time.perf_counter()
        ch.sweeps(reps, nthreads=nthreads)
        dt = time.perf_counter() - t0
        return n * reps / dt, reps, dt

    n = wl["n"]
    ch = oracle.Chain(wl["row_ptr"], wl["col"], wl["color"], wl["y"], rho=1.0, seed=1)
    rate, reps, dt = timed(ch, n, seconds_budget, threads)
    ch1 = oracle.Chain(wl["row_ptr"], wl["col"], wl["color"], wl["y"], rho=1.0, seed=1)
    rate1, reps1, dt1 = timed(ch1, n, seconds_budget / 2, 1)
    from paper_1702_05518_amd import inputs

    c1 = inputs.lattice_workload(64, 64, 4, noise_sd=0.1, data_seed=1)
    o1 = oracle.Chain(c1["row_ptr"], c1["col"], c1["color"], c1["y"], seed=1)
    t0 = time.perf_counter()
    o1.sweeps(1000, nthreads=1)
    t_c1 = time.perf_counter() - t0
    c3 = inputs.delaunay_workload(15000, data_seed=3, rho=0.95)
    color, _ = oracle.greedy_coloring(c3["row_ptr"], c3["col"])
    o3 = oracle.Chain(c3["row_ptr"], c3["col"], color, c3["y"], rho=0.95, seed=3)
    t0 = time.perf_counter()
    o3.sweeps(2000, nthreads=threads)
    t_c3 = time.perf_counter() - t0
    bps = BYTES_PER_SITE["fp64_acc"]
    big = None
    if wl1m is not None:
        color1m, _ = oracle.greedy_coloring(wl1m["row_ptr"], wl1m["col"])
        o4 = oracle.Chain(wl1m["row_ptr"], wl1m["col"], color1m, wl1m["y"], rho=0.95, seed=3)
        r4, reps4, dt4 = timed(o4, wl1m["n"], seconds_budget / 2, threads)
        big = {"site_updates_per_s": r4, "sweeps": reps4, "seconds": dt4, "threads": threads,
               "gbs": r4 * CSR_BYTES_PER_SITE["fp64_acc"] / 1e9}
    return {"value": rate, "unit": "site-updates/s", "cores": threads, "kind": "oracle",
            "sample": f"{reps} FP64 sweeps (+1 untimed) of the same 2048x2048 8-neighbour "
                      f"lattice workload, C oracle with {threads} OpenMP threads on "
                      f"'{model or platform.processor()}'",
            "seconds": dt, "gbs": rate * bps / 1e9,
            "single_thread": {"value": rate1, "sweeps": reps1, "seconds": dt1,
                              "gbs": rate1 * bps / 1e9},
            "lattice64_1000_sweeps": {"seconds": t_c1, "threads": 1,
                                      "site_updates_per_s": 4096 * 1000 / t_c1},
            "delaunay15k_2000_sweeps": {"seconds": t_c3, "threads": threads,
                                        "site_updates_per_s": 15000 * 2000 / t_c3,
                                        "gbs": 15000 * 2000 / t_c3 *
                                        CSR_BYTES_PER_SITE["fp64_acc"] / 1e9},
            "delaunay1m_sample": big}


def probe(torch, gmrf, inputs, steps, side=ROWS, variants=False, on_graph=False):
    """A plain device copy of 512 MiB (its counters give the scale factor of
    FETCH_SIZE / WRITE_SIZE), then warm-up and `steps` FP32 sweeps, one launch
    each, of the benchmark workload (side x side, 8 neighbours).  variants:
    then the same for FP32 under rng_version 2 and FP64 under both.  on_graph:
    instead the 1,000,000-site Delaunay workload's chunked sweeps, FP32 then
    FP64."""
    src = torch.ones(128 * 1024 * 1024, dtype=torch.float32, device="cuda")
    dst = torch.empty_like(src)
    dst.copy_(src)
    torch.cuda.synchronize()
    del src, dst
    if on_graph:
        wl = inputs.delaunay_workload(GRAPH_PROBE_SITES, data_seed=3, rho=0.95)
        color, k = gmrf.greedy_coloring(wl["row_ptr"], wl["col"])
        graph = gmrf.Graph(row_ptr=wl["row_ptr"], col_idx=wl["col"], color=color, num_colors=k,
                           rho=0.95)
        runs = [(gmrf.FP32_ACC64, 1), (gmrf.FP64, 1)]
    else:
        wl = inputs.lattice_workload(side, side, STENCIL, noise_sd=0.1, data_seed=1,
                                     with_csr=False)
        graph = gmrf.Graph(lattice=(side, side, STENCIL))
        runs = [(gmrf.FP32_ACC64, 1)]
        if variants:
            runs += [(gmrf.FP32_ACC64, 2), (gmrf.FP64, 1), (gmrf.FP64, 2)]
    for prec, v in runs:
        chain = gmrf.Chain(graph, wl["y"], precision=prec, seed=1, rng_version=v)
        # whole groups of sweeps (five FP32, three FP64) that share a pass over
        # the accumulators, as in the benchmark's calls
        chain.sweep(15, hyper=True)
        chain.sweep(steps, hyper=True)
        torch.cuda.synchronize()
        del chain
    print(json.dumps({"probe": "copy 512 MiB + sweeps", "workload": "delaunay1m" if on_graph
                      else f"lattice {side}x{side}", "sweeps": steps + 15, "chains": len(runs)}),
          flush=True)


def bench_batch(torch, gmrf, inputs, args):
    """The batched workload alone (batch_row), with the same chains swept one
    by one for comparison.  Prints one JSON line."""
    row = batch_row(torch, gmrf, inputs, args, steps=args.steps)
    chains = row.pop("_chains")
    solo_sweeps = 5
    s = torch.cuda.current_stream()
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    e0.record(s)
    for c in chains:
        c.sweep(solo_sweeps)
    e1.record(s)
    torch.cuda.synchronize()
    t_solo = e0.elapsed_time(e1) / 1e3 / solo_sweeps
    line = {
        "metric": "site-updates/s (batched instances)", "value": row["site_updates_per_s"],
        "unit": "site-updates/s", "n_gpus": 1, "steps": row["steps"], "warmup": args.warmup,
        "ms_per_step": row["ms_per_sweep"], "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": row["workload"], "sites_per_sweep": row["sites_per_sweep"],
                   "instances": row["instances"]},
        "roofline": {"bound": "hbm", "achieved": row["achieved_gbs"], "peak": HBM_PEAK_GBS,
                     "unit": "GB/s", "frac": row["frac"], "traffic": None},
        "unbatched_site_updates_per_s": row["sites_per_sweep"] / t_solo,
        "batching_speedup": t_solo / (row["ms_per_sweep"] / 1e3),
        "lattice_tile_autotune": row["lattice_tile_autotune"],
    }
    print(json.dumps(line), flush=True)


def bench_serve(torch, gmrf, inputs, args):
    """Serving: Poisson arrivals of 1000-sweep jobs on Delaunay graphs of the
    irregular workload's sizes (n = 15,000 with probability 0.98, n =
    1,000,000 with probability 0.02), FP32 with FP64 accumulators, continuous
    batching; arrival rates 50 .. 1600 jobs/s, 2 s of arrivals each, for the
    latency-against-load curve (the 200/s point is the headline); against the
    FP64 plain form (one standalone chain at a time, plain launches) on the
    whole 200/s stream.  Prints one JSON line."""
    from paper_1702_05518_amd import serve

    pool = []
    for n, ds in [(15000, 11), (15000, 12), (15000, 13), (1_000_000, 14)]:
        wl = inputs.delaunay_workload(n, data_seed=ds, rho=0.95)
        color, k = gmrf.greedy_coloring(wl["row_ptr"], wl["col"])
        pool.append((gmrf.Graph(row_ptr=wl["row_ptr"], col_idx=wl["col"], color=color,
                                num_colors=k, rho=0.95), wl["y"]))
    log("[bench] serve: graph pool ready")

    def arrivals(rate, seed):
        rng = np.random.Generator(np.random.PCG64(seed))
        t, jobs = 0.0, []
        while True:
            t += rng.exponential(1.0 / rate)
            if t > 2.0:
                return jobs
            g, y = pool[3] if rng.random() < 0.02 else pool[int(rng.integers(0, 3))]
            jobs.append(serve.Job(len(jobs), g, y, seed=1000 + len(jobs), instance=len(jobs),
                                  nsweeps=1000, arrival=t, precision=gmrf.FP32_ACC64))

    curve, head, head_jobs = [], None, None
    for rate in (50, 100, 200, 400, 800, 1600):
        jobs = arrivals(rate, 7 if rate == 200 else 7 + rate)
        offered = sum(j.sites * j.nsweeps for j in jobs) / 2.0
        free, _ = torch.cuda.mem_get_info()
        server = serve.Server(budget_bytes=int(0.5 * free), step_sweeps=10, max_active=1024,
                              overlap=True)
        wall = server.run(jobs, realtime=True)
        sites = sum(j.sites * j.nsweeps for j in server.finished)
        point = dict(serve.latency_summary(server.finished), rate_per_s=rate,
                     offered_site_updates_per_s=offered, site_updates_per_s=sites / wall,
                     wall_s=wall, batch_rebuilds=server.rebuilds)
        curve.append(point)
        log(f"[bench] serve {rate}/s: {len(jobs)} jobs in {wall:.2f} s, p50 "
            f"{point['p50_ms']:.1f} ms, p99 {point['p99_ms']:.1f} ms")
        if rate == 200:
            head, head_jobs = point, jobs
    plain_jobs = [serve.Job(j.job_id, j.graph, j.y, j.seed, j.instance, j.nsweeps, j.arrival,
                            gmrf.FP64) for j in head_jobs]
    log(f"[bench] serve: FP64 plain form on the {len(plain_jobs)} jobs of the 200/s stream")
    wall_plain = serve.serve_plain(plain_jobs, precision=gmrf.FP64, realtime=True)
    plain = serve.latency_summary(plain_jobs)
    plain_sites = sum(j.sites * j.nsweeps for j in plain_jobs)
    line = {
        "metric": "p50/p99 solve latency (served, continuous batching)",
        "value": head["site_updates_per_s"], "unit": "site-updates/s", "n_gpus": 1,
        "steps": 1000, "warmup": 0, "ms_per_step": None, "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": "Poisson arrivals 200/s for 2 s of 1000-sweep jobs, Delaunay "
                               "n=15k (p 0.98) or 1M (p 0.02), FP32 + FP64 accumulators, "
                               "continuous batching every 10 sweeps, host work overlapped "
                               "with the queued sweeps",
                   "jobs": head["jobs"], "batch_rebuilds": head["batch_rebuilds"]},
        "served_fp32": {k: head[k] for k in ("p50_ms", "p99_ms", "mean_ms", "jobs")},
        "load_curve": curve,
        "plain_fp64_200_per_s": dict(plain, site_updates_per_s=plain_sites / wall_plain,
                                     wall_s=wall_plain),
    }
    print(json.dumps(line), flush=True)


def run_captured(chain, total):
    """`total` sweeps with every draw, as captured graphs of 1000 sweeps (and
    one graph for the remainder)."""
    for _ in range(total // 1000):
        chain.sweep(1000, hyper=True, capture=True)
    if total % 1000:
        chain.sweep(total % 1000, hyper=True, capture=True)


def bench_image(torch, gmrf, inputs, args):
    """The paper's image example on the GPU (Sec. 3.1, Table 1 setting):
    p x p Gaussian-bump truth plus N(0, 1) (and N(0, 50^2)) noise, 8-neighbour
    intrinsic prior with an intercept, Gamma(0.001, 0.001) priors on both
    precisions, 10,000 sweeps of which the last 2,000 are retained.  T is the
    wall time of the whole run (sweeps as captured 1000-sweep graphs, capture
    included, plus the posterior statistics); the tau^2 = 1/tau chain comes
    from the device trace and gives IAT, ESS and CES = IAT T / N.  Prints one
    JSON line; the paper's CPU figures are context only."""
    from paper_1702_05518_amd import diagnostics

    total = args.iterations
    burn = total * 4 // 5                 # 8,000 of 10,000 in Table 1
    prior = dict(a_tau=0.001, b_tau=0.001, a_lam=0.001, b_lam=0.001)
    rows = []
    for p, noise in [(50, 1.0), (50, 50.0), (128, 1.0), (512, 1.0), (2048, 1.0)]:
        wl = inputs.bump_image_workload(p, noise_sd=noise)
        graph = gmrf.Graph(lattice=(p, p, 8))
        for name, prec in (("fp64", gmrf.FP64), ("fp32_acc", gmrf.FP32_ACC64)):
            ch = gmrf.Chain(graph, wl["y"], precision=prec, seed=1, intercept=True,
                            burn_in=burn, **prior)
            ch.enable_trace(total)
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            run_captured(ch, total)
            mean, var, nacc = ch.posterior_stats()
            torch.cuda.synchronize()
            T = time.perf_counter() - t0
            tr = ch.trace()
            if nacc != total - burn or not np.isfinite(tr).all():
                print("bench.py: image run failed", file=sys.stderr)
                sys.exit(1)
            tau2 = 1.0 / tr[burn:, 0]
            d = diagnostics.summary(tau2, T)
            row = {"p": p, "noise_sd": noise, "precision": name, "seconds": T,
                   "site_updates_per_s": p * p * total / T, "iat_tau2": d["iat"],
                   "ess_tau2": d["ess"], "ces_s": d["ces_s"],
                   "posterior_mean_rmse_vs_truth": float(np.sqrt(np.mean(
                       (mean - wl["truth"]) ** 2))),
                   "sigma2_mean": float(np.mean(1.0 / tr[burn:, 1])),
                   "beta0_mean": float(np.mean(tr[burn:, 2]))}
            rows.append(row)
            log(f"[bench] image p={p} noise={noise} {name}: T {T:.3f} s, IAT {d['iat']:.2f}, "
                f"CES {d['ces_s']:.2e} s")
            ch.disable_trace()
            del ch
    head = rows[0]
    line = {
        "metric": "CES (cost per effective sample) of the tau^2 chain, 50x50 image",
        "value": head["ces_s"], "unit": "s", "n_gpus": 1, "steps": total, "warmup": 0,
        "ms_per_step": head["seconds"] / total * 1e3, "higher_is_better": False,
        "scaling": "weak", "vs_baseline": None, "dtype": "f64", "data": "synthetic",
        "config": {"workload": "p x p Gaussian-bump image + N(0, noise^2), 8-neighbour "
                               "intrinsic CAR with intercept, Gamma(0.001, 0.001) priors, "
                               "10,000 sweeps, 8,000 burn-in, one chain per run",
                   "p": 50, "noise_sd": 1.0},
        "rows": rows,
        "context_paper_table1_chromatic_cpu": {"seconds": 10.99, "iat": 30.42, "ess": 65.74,
                                               "ces_s": 0.17,
                                               "hardware": "Xeon @ 4.10 GHz, R, FP64"},
    }
    print(json.dumps(line), flush=True)


def bench_binomial(torch, gmrf, inputs, args):
    """The paper's binomial example on the GPU (Sec. 3.2, Table 2 setting):
    n = 14,926 areas with a Delaunay adjacency (greedy coloring), counts of
    lognormal trial numbers (median 250, 2.2% areas without data), proper CAR
    rho = 0.995, beta0 ~ N(0, 1000), tau ~ Gamma(1, 1) (InvGam(1, 1) on
    tau^2), 10,000 iterations of which the last 5,000 are retained.  T is the
    wall time of the whole run; IAT / ESS / CES of the beta0 and tau^2
    chains come from the device trace.  The oracle is timed on a bounded
    number of iterations of the same workload.  Prints one JSON line."""
    from paper_1702_05518_amd import diagnostics

    total, n = args.iterations, 14_926
    burn = total // 2                     # 5,000 of 10,000 in Table 2
    wl = inputs.binomial_workload(n, data_seed=5)
    color, k = gmrf.greedy_coloring(wl["row_ptr"], wl["col"])
    graph = gmrf.Graph(row_ptr=wl["row_ptr"], col_idx=wl["col"], color=color, num_colors=k,
                       rho=0.995)
    rows = []
    for name, prec in (("fp64", gmrf.FP64), ("fp32_acc", gmrf.FP32_ACC64)):
        ch = gmrf.Chain(graph, wl["y"], precision=prec, seed=1, trials=wl["trials"],
                        intercept=True, beta0_var=1000.0, burn_in=burn)
        ch.enable_trace(total)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        run_captured(ch, total)
        mean, var, nacc = ch.posterior_stats()
        torch.cuda.synchronize()
        T = time.perf_counter() - t0
        tr = ch.trace()
        if nacc != total - burn or not np.isfinite(tr).all():
            print("bench.py: binomial run failed", file=sys.stderr)
            sys.exit(1)
        b0 = diagnostics.summary(tr[burn:, 2], T)
        t2 = diagnostics.summary(1.0 / tr[burn:, 0], T)
        rows.append({"precision": name, "seconds": T, "site_updates_per_s": n * total / T,
                     "ms_per_sweep": T / total * 1e3,
                     "beta0": {"iat": b0["iat"], "ess": b0["ess"], "ces_s": b0["ces_s"]},
                     "tau2": {"iat": t2["iat"], "ess": t2["ess"], "ces_s": t2["ces_s"]},
                     "eta_corr_vs_truth": float(np.corrcoef(mean, wl["truth"])[0, 1])})
        log(f"[bench] binomial {name}: T {T:.2f} s, CES beta0 {b0['ces_s']:.2e} s, "
            f"tau2 {t2['ces_s']:.2e} s")
        ch.disable_trace()
        del ch
    line = {
        "metric": "CES of the beta0 and tau^2 chains, binomial model n=14,926",
        "value": rows[0]["beta0"]["ces_s"], "unit": "s", "n_gpus": 1, "steps": total,
        "warmup": 0, "ms_per_step": rows[0]["ms_per_sweep"], "higher_is_better": False,
        "scaling": "weak", "vs_baseline": None, "dtype": "f64", "data": "synthetic",
        "config": {"workload": "binomial logit, Polya-Gamma augmentation, Delaunay n=14,926, "
                               "greedy coloring, trials lognormal median 250 (2.2% empty), "
                               "proper CAR rho 0.995, beta0 ~ N(0, 1000), 10,000 iterations, "
                               "5,000 burn-in",
                   "colors": int(k), "trials_total": int(wl["trials"].sum())},
        "rows": rows,
        "context_paper_table2_chromatic_cpu": {"seconds": 222.06, "beta0_ces_s": 0.0935,
                                               "tau2_ces_s": 0.1155,
                                               "hardware": "Core i5-3570, R, FP64"},
    }
    if not args.no_cpu:
        import oracle

        oracle.build(force=False)
        threads = min(16, os.cpu_count() or 1)
        oc = oracle.Chain(wl["row_ptr"], wl["col"], color, wl["y"], rho=0.995,
                          trials=wl["trials"], intercept=True, beta0_var=1000.0, seed=1)
        t0 = time.perf_counter()
        oc.sweeps(1, nthreads=threads)
        one = time.perf_counter() - t0
        reps = max(1, min(200, int(10.0 / max(one, 1e-3))))
        t0 = time.perf_counter()
        oc.sweeps(reps, nthreads=threads)
        dt = time.perf_counter() - t0
        line["cpu_baseline"] = {"value": n * reps / dt, "unit": "site-updates/s",
                                "cores": threads, "kind": "oracle",
                                "sample": f"{reps} FP64 iterations of the same binomial "
                                          f"workload, C oracle with {threads} OpenMP threads"}
    print(json.dumps(line), flush=True)


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=200)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--no-cpu", action="store_true", help="skip the CPU oracle baseline")
    ap.add_argument("--no-fp64", action="store_true", help="skip the FP64 comparison run")
    ap.add_argument("--no-big", action="store_true", help="skip the 8192 x 8192 lattice row")
    ap.add_argument("--no-graph", action="store_true",
                    help="skip the 1,000,000-site Delaunay row")
    ap.add_argument("--no-batch", action="store_true", help="skip the 512-instance batch row")
    ap.add_argument("--no-v2", action="store_true",
                    help="skip the paired random-number contract (rng_version 2) row")
    ap.add_argument("--reps", type=int, default=10, help="solves for p50/p99 latency")
    ap.add_argument("--workload", default="lattice2048",
                    choices=["lattice2048", "batch512", "serve", "image", "binomial"],
                    help="lattice2048: the 2048x2048 lattice line (default); batch512: the "
                         "batched many-instance workload; serve: the serving workload; "
                         "image: the paper's image example with IAT / ESS / CES; "
                         "binomial: the paper's binomial example with IAT / ESS / CES "
                         "(each a separate JSON line)")
    ap.add_argument("--iterations", type=int, default=10_000,
                    help="image / binomial: iterations of the paper's example (default 10,000, "
                         "with the paper's burn-in fractions 4/5 and 1/2)")
    ap.add_argument("--summarize", nargs="+", metavar="ARG",
                    help="print a profiles/ summary: 'trace KERNEL_TRACE_CSV', 'traffic SIDE "
                         "FETCH_CSV WRITE_CSV [DRAM_CSV]', 'traffic-graph FETCH_CSV WRITE_CSV' or "
                         "'counters CSV...' (rocprofv3 "
                         "outputs; no GPU needed)")
    ap.add_argument("--command", action="append", default=[],
                    help="with --summarize: a command line to record in the summary")
    ap.add_argument("--probe-side", type=int, default=ROWS,
                    help="lattice side of --probe (8 neighbours, FP32)")
    ap.add_argument("--probe-variants", action="store_true",
                    help="with --probe: also FP32 under rng_version 2 and FP64 under both")
    ap.add_argument("--probe-graph", action="store_true",
                    help="with --probe: the 1,000,000-site Delaunay workload (chunked sweeps, "
                         "FP32 then FP64) instead of the lattice")
    ap.add_argument("--probe", action="store_true",
                    help="counter probe for rocprofv3 --pmc: a 512 MiB device copy (the "
                         "scale reference for FETCH_SIZE / WRITE_SIZE), then --steps sweeps")
    args = ap.parse_args()
    if args.summarize:
        kind, rest = args.summarize[0], args.summarize[1:]
        if kind == "trace":
            text, fig = trace_summary(rest[0], args.command)
        elif kind == "counters":
            text, fig = counter_summary(rest, args.command)
        elif kind == "traffic-graph":
            text, fig = graph_traffic_summary(rest[0], rest[1], args.command)
        else:
            text, fig = traffic_summary(rest[1], rest[2], rest[3] if len(rest) > 3 else None,
                                        int(rest[0]), args.command)
        print(text)
        if fig:
            print("\njson: " + json.dumps(fig))
        return
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py: the benchmark runs on exactly one GPU (independent chains shard across "
              "GPUs without communication); --gpus must be 1", file=sys.stderr)
        sys.exit(2)

    import torch

    from paper_1702_05518_amd import gmrf, inputs

    if not torch.cuda.is_available():
        print("bench.py: no GPU visible", file=sys.stderr)
        sys.exit(1)
    gmrf.lib()
    n = ROWS * COLS
    if args.probe:
        probe(torch, gmrf, inputs, args.steps, args.probe_side, args.probe_variants,
              args.probe_graph)
        return
    if args.workload == "batch512":
        bench_batch(torch, gmrf, inputs, args)
        return
    if args.workload == "serve":
        bench_serve(torch, gmrf, inputs, args)
        return
    if args.workload == "image":
        bench_image(torch, gmrf, inputs, args)
        return
    if args.workload == "binomial":
        bench_binomial(torch, gmrf, inputs, args)
        return
    log(f"[bench] building workload {ROWS}x{COLS} stencil {STENCIL}")
    wl = inputs.lattice_workload(ROWS, COLS, STENCIL, noise_sd=0.1, data_seed=1,
                                 with_csr=not args.no_cpu)
    graph = gmrf.Graph(lattice=(ROWS, COLS, STENCIL))
    results = {}
    for name, prec in (("fp32_acc", gmrf.FP32_ACC64), ("fp64_acc", gmrf.FP64)):
        if name == "fp64_acc" and args.no_fp64:
            continue
        log(f"[bench] {name}: warmup {args.warmup}")
        chain = gmrf.Chain(graph, wl["y"], precision=prec, seed=1)
        chain.sweep(args.warmup, hyper=True)
        chain.sweep(args.steps, hyper=True, capture=True)      # record the graph once
        torch.cuda.synchronize()
        log(f"[bench] {name}: timing {args.steps} sweeps")
        t_plain = timed_sweeps(torch, chain, args.steps, capture=False)
        t_graph = timed_sweeps(torch, chain, args.steps, capture=True)
        k_disp = dispatch_timed(torch, chain, args.steps)
        lat = solve_latencies(torch, chain, 1000, args.reps)
        mean, var, nacc = chain.posterior_stats()
        x, tau, lam, sw = chain.get_state()
        if not (np.isfinite(mean).all() and np.isfinite(tau) and np.isfinite(lam)):
            print("bench.py: non-finite result", file=sys.stderr)
            sys.exit(1)
        results[name] = dict(t_plain=t_plain, t_graph=t_graph, kernel_disp_s=k_disp,
                             p50_ms=float(np.percentile(lat, 50)),
                             p99_ms=float(np.percentile(lat, 99)), tau=tau, lam=lam,
                             sweeps_done=sw)
        log(f"[bench] {name}: plain {t_plain * 1e3:.3f} ms, graph {t_graph * 1e3:.3f} ms, "
            f"dispatch-event kernel {k_disp * 1e6:.2f} us, p50 {results[name]['p50_ms']:.2f} ms")
        del chain
        torch.cuda.synchronize()

    # burn-in sweeps (no accumulator update): x read and written, y read
    burn = gmrf.Chain(graph, wl["y"], precision=gmrf.FP32_ACC64, seed=1, burn_in=1 << 40)
    burn.sweep(args.warmup, hyper=True)
    t_burn = graph_seconds(torch, lambda cap: burn.sweep(args.steps, hyper=True, capture=cap),
                           args.steps) / args.steps
    del burn
    burn_gbs = BURN_IN_BYTES_PER_SITE * n / t_burn / 1e9
    log(f"[bench] burn-in sweep: {t_burn * 1e6:.1f} us ({burn_gbs / HBM_PEAK_GBS:.3f} of peak)")
    log("[bench] host-to-host solve (FP32, 1000 sweeps)")
    host_solve_s = min(host_to_host_solve(torch, gmrf, graph, wl["y"], 1000) for _ in range(3))
    r = results["fp32_acc"]
    t_best = min(r["t_plain"], r["t_graph"])
    value = n * args.steps / t_best
    bytes_launch = BYTES_PER_SITE["fp32_acc"] * n
    # One launch of the sweep kernel per sweep (it also ends the previous
    # sweep); the call adds one commit launch and one unit-variate launch.
    # The kernel's average launch duration is the timed region's length over
    # its launches, so the figure includes every gap and the small launches.
    launch_s = t_best / args.steps
    achieved = bytes_launch / launch_s / 1e9
    prof = profile_figures(TRACE_SUMMARY)
    traffic = profile_figures(TRAFFIC_SUMMARY)
    line = {
        "metric": METRIC,
        "value": value,
        "unit": "site-updates/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": t_best / args.steps * 1e3,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": "lattice 2048x2048, 8-neighbour intrinsic CAR, 2x2-parity "
                               "4-coloring, FP32 state/draws/neighbour sums, FP64 "
                               "accumulators and q/sse reductions, Gamma(1,1) priors, "
                               "accumulating sweeps",
                   "sites": n, "colors": 4, "sweep_launch": "hipGraph" if r["t_graph"] <=
                   r["t_plain"] else "stream"},
        "roofline": {"bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": achieved / HBM_PEAK_GBS,
                     "traffic": traffic["bytes_per_launch"] if traffic else None,
                     "traffic_unit": "bytes/launch (rocprofv3 FETCH_SIZE + WRITE_SIZE, each "
                                     "scaled by a device copy's reading)",
                     "algorithmic_bytes": bytes_launch,
                     "kernel": SWEEP_KERNEL,
                     "bytes_per_site": BYTES_PER_SITE["fp32_acc"],
                     "launch_us": launch_s * 1e6,
                     "launch_us_basis": "timed region / launches (HIP events around the "
                                        "K sweeps, one sweep-kernel launch each)",
                     "kernel_us_rocprof": prof["avg_ns"] / 1e3 if prof else None,
                     "frac_kernel_rocprof": (bytes_launch / (prof["avg_ns"] * 1e-9) / 1e9 /
                                             HBM_PEAK_GBS) if prof else None,
                     "kernel_us_dispatch_events": r["kernel_disp_s"] * 1e6},
        "burn_in_sweep": {"us": t_burn * 1e6, "bytes_per_site": BURN_IN_BYTES_PER_SITE,
                          "achieved_gbs": burn_gbs, "frac": burn_gbs / HBM_PEAK_GBS,
                          "covers": "FP32 sweeps before burn-in ends (no S1/S2 update), "
                                    "graph replay"},
        "sweep_ms": {"fp32_stream": r["t_plain"] / args.steps * 1e3,
                     "fp32_graph": r["t_graph"] / args.steps * 1e3},
        "solve_latency_ms_1000_sweeps": {"fp32": {"p50": r["p50_ms"], "p99": r["p99_ms"]}},
        "host_to_host_1000_sweeps": {"value": n * 1000 / host_solve_s, "unit": "site-updates/s",
                                     "ms": host_solve_s * 1e3,
                                     "covers": "chain creation with the upload of y, 1000 "
                                               "plain-launch sweeps, mean/variance to host "
                                               "(best of 3)"},
    }
    if "fp64_acc" in results:
        d = results["fp64_acc"]
        t64 = min(d["t_plain"], d["t_graph"])
        line["fp64"] = {"value": n * args.steps / t64, "unit": "site-updates/s",
                        "ms_per_step": t64 / args.steps * 1e3,
                        "hbm_frac": BYTES_PER_SITE["fp64_acc"] * n / (t64 / args.steps) / 1e9 /
                        HBM_PEAK_GBS,
                        "kernel_us_dispatch_events": d["kernel_disp_s"] * 1e6}
        line["solve_latency_ms_1000_sweeps"]["fp64"] = {"p50": d["p50_ms"], "p99": d["p99_ms"]}
    if not args.no_v2:
        line["rng_v2"] = rng_v2_row(torch, gmrf, graph, wl["y"], args)
    if not args.no_big:
        line["lattice8192_out_of_cache"] = big_lattice_row(torch, gmrf, inputs, args)
    wl1m = None
    if not (args.no_graph and args.no_cpu):
        wl1m = inputs.delaunay_workload(1_000_000, data_seed=3, rho=0.95)
    if not args.no_graph:
        line["delaunay1m"] = delaunay_row(torch, gmrf, inputs, args, wl1m)
    if not args.no_batch:
        row = batch_row(torch, gmrf, inputs, args)
        del row["_chains"]
        line["batch512"] = row
    if not args.no_cpu:
        log("[bench] cpu baseline (oracle)")
        line["cpu_baseline"] = cpu_baseline(wl, wl1m=wl1m)
    print(json.dumps(line), flush=True)


if __name__ == "__main__":
    main()
