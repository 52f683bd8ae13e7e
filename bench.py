#!/usr/bin/env python3
"""Throughput of the basketised EM-shower stepping on one MI355X.

Workload (default): 10,000 events on a 50-layer Pb/lAr sampling calorimeter
(2.3 mm Pb + 5.7 mm lAr, 40x40 cm) in a 4 T field along y; one primary per
event, e-/e+/gamma by event mod 3, kinetic energy log-uniform in
100 MeV..100 GeV, 1 mrad Gaussian angular spread.  One benchmark step = one
full transport of that batch (every stage of every step of every track,
scoring included) through the C ABI, the primaries already resident on the
device (gv_stage outside the timed region), the deposit buffer a torch tensor
on torch's current stream.

Reported: track steps/s and primaries/s of the batched mixed-precision path
(value), beside the plain FP64 per-stage path on the same batch and seed; the
per-layer deposits of the two are checked with a paired test; the dominant
kernel's HBM roofline fraction from HIP-event timing inside the library; the
FP64 CPU oracle timed on a bounded sample of the same batch.
"""
from __future__ import annotations

import argparse
import json
import math
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "steps/s & primaries/s on 1 MI355X, FP32 batched vs FP64 plain, matched edep"
HBM_PEAK = 8.0e12
TRAFFIC_FILE = os.path.join(ROOT, "profiles", "hbm_traffic_c4.json")


def kernel_source_hash():
    """SHA-1 over the HIP sources and build flags of the library."""
    import hashlib
    h = hashlib.sha1()
    pkg = os.path.join(ROOT, "paper_2005_00949_amd")
    files = sorted(os.listdir(os.path.join(pkg, "csrc")))
    for f in files:
        with open(os.path.join(pkg, "csrc", f), "rb") as fh:
            h.update(f.encode() + b"\0" + fh.read())
    with open(os.path.join(pkg, "build.py"), "rb") as fh:
        h.update(fh.read())
    return h.hexdigest()


def measured_traffic(steps_per_launch, workload, knobs):
    """HBM bytes per launch from the recorded FETCH_SIZE / WRITE_SIZE counters of
    the transport's kernels (per step, calibrated against a plain copy), or None when the kernel
    sources changed since they were taken, the workload differs, or no
    recorded entry has these knobs (basket, occupancy, inner steps)."""
    try:
        with open(TRAFFIC_FILE) as f:
            t = json.load(f)
    except (OSError, ValueError):
        return None
    if t.get("source_sha1") != kernel_source_hash() or t.get("workload") != workload:
        return None
    for e in t.get("entries", []):
        if e.get("knobs") == list(knobs):
            return e["bytes_per_step"] * steps_per_launch
    return None


def shower_roofline(res):
    """Algorithmic bytes per second of the kernels outside the tail: the
    transport's algorithmic bytes less 108 B per tail step
    (mixed-precision slot read and moving fields written; the tail's loopers
    have no secondaries), over the kernel time outside the tail."""
    t = (sum(res["kern_ms"]) - sum(res["tail_ms"])) * 1e-3
    b = res["alg_bytes"] - 108.0 * res["tail_steps"]
    if t <= 0.0:
        return None
    return {"achieved": b / t / 1e9, "frac": b / t / HBM_PEAK, "kernel_ms_per_transport": t * 1e3 / len(res["kern_ms"])}


def log(msg):
    print(msg, file=sys.stderr, flush=True)


def paired_layers(x, y, gate=True):
    """Per-layer paired comparison of deposits X (tested) vs Y (reference):
    mean difference within 3 sigma of the paired differences and within 0.5%
    on layers that hold at least 1% of the mean total deposit.  With
    gate=False (two different samplers, whose histories decorrelate) the
    statistics are reported without a verdict, together with the 3-sigma
    resolution of the sample on the big layers."""
    import numpy as np
    d = x - y
    n = len(d)
    m = y.mean(0)
    delta = d.mean(0)
    sig = d.std(0, ddof=1) / math.sqrt(n) if n > 1 else np.zeros_like(m)
    big = m >= 0.01 * m.sum()
    ok3 = np.abs(delta) <= 3 * sig + 1e-9 * np.abs(m)
    ok05 = ~big | (np.abs(delta) <= 0.005 * np.abs(m))
    worst = float(np.max(np.abs(delta[big]) / m[big])) if big.any() else 0.0
    out = dict(worst_rel_big_layers=worst, layers_outside_3sigma=int((~ok3).sum()), layers=int(len(m)),
               three_sigma_rel_median_big_layers=float(np.median(3 * sig[big] / m[big])) if big.any() else 0.0,
               events=int(n))
    if gate:
        out["pass_"] = bool(ok05.all() and (~ok3).sum() <= max(1, len(m) // 20))
    return out


def run_gpu(args):
    import numpy as np
    import torch

    import gv_inputs
    import paper_2005_00949_amd as gv

    torch.cuda.set_device(0)
    geom, prim, seed = gv_inputs.workload(args.workload, args.events)
    n_events = int(prim["event"].max()) + 1
    stream = torch.cuda.current_stream()
    eng = gv.Engine(geom, driver=gv.DRIVER_BATCHED, precision=gv.PMIX, edep_on_device=1,
                    hip_stream=stream.cuda_stream, basket=args.basket, occupancy=args.occupancy,
                    inner_steps=args.inner, graph_steps=args.graph_steps)
    edep = torch.zeros((n_events, eng.n_cells), dtype=torch.float64, device="cuda:0")
    eng.stage(prim)
    log(f"[bench] workload {args.workload}: {len(prim)} primaries, {n_events} events, "
        f"{eng.n_cells} cells; warmup {args.warmup}, steps {args.steps}")
    tune_ms = 0.0
    warm_ms = []
    for w in range(args.warmup):
        eng.transport_staged(seed, edep.data_ptr())
        st = eng.stats()
        tune_ms += st["autotune_ms"]
        warm_ms.append(round(st["transport_ms"], 2))
        log(f"[bench] warmup {w}: {st['transport_ms']:.1f} ms ({st['autotune_ms']:.1f} ms autotuning), "
            f"{st['total_steps']} steps, basket {st['basket']} occupancy {st['occupancy']} "
            f"inner {st['inner_steps']}")
    torch.cuda.synchronize()
    steps = prims = 0
    lane_slots = 0
    kernel_ms = 0.0
    launches = 0
    alg_bytes = 0.0
    edep_first = None
    per_ms, tail_ms = [], []
    tail_steps, kern_ms = 0, []
    helper_steps = 0
    t0 = time.perf_counter()
    for k in range(args.steps):
        eng.transport_staged(seed + k, edep.data_ptr())
        st = eng.stats()
        steps += st["total_steps"]
        lane_slots += st["lane_slots"]
        prims += len(prim)
        kernel_ms += st["kernel_ms"]
        launches += st["kernel_launches"]
        alg_bytes += st["alg_bytes"]
        per_ms.append(st["transport_ms"])
        tail_ms.append(st["tail_kernel_ms"])
        tail_steps += st["tail_steps"]
        helper_steps += st["helper_steps"]
        kern_ms.append(st["kernel_ms"])
        if k == 0:
            edep_first = edep.cpu().numpy()
            st0 = st
        log(f"[bench] step {k}: {st['transport_ms']:.1f} ms ({st['tail_kernel_ms']:.1f} ms in the tail), "
            f"{st['total_steps']} steps")
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    res = dict(steps=steps, primaries=prims, elapsed=elapsed, kernel_ms=kernel_ms, launches=launches,
               alg_bytes=alg_bytes, stats0=st0, n_events=n_events, median_ms=float(np.median(per_ms)),
               autotune_ms=tune_ms, tail_ms=tail_ms, per_ms=per_ms, lane_slots=lane_slots, warm_ms=warm_ms,
               tail_steps=tail_steps, kern_ms=kern_ms, edep_first=edep_first, helper_steps=helper_steps)

    # the same transport through gv_transport with host primaries and a host
    # edep_out (PCIe both ways); reported beside value, never as value
    res["pcie_inclusive_ms"] = res["pcie_inclusive_steps_per_s"] = None
    if not args.no_pcie:
        eng.configure(edep_on_device=0)
        t = time.perf_counter()
        eng.transport(prim, seed)
        res["pcie_inclusive_ms"] = (time.perf_counter() - t) * 1e3
        res["pcie_inclusive_steps_per_s"] = eng.stats()["total_steps"] / (res["pcie_inclusive_ms"] * 1e-3)
        eng.configure(edep_on_device=1)
        eng.stage(prim)

    # the same batch with every final state sampled from the alias tables
    # (the second sampling method of the paper's physics library)
    tables = None
    if args.table_steps > 0:
        eng.configure(fs_alias=gv.FS_ALL)
        eng.transport_staged(seed, edep.data_ptr())          # warm-up (graph capture)
        edep_tab = edep.cpu().numpy()
        tt, ttail, tsteps = [], [], 0
        for k in range(args.table_steps):
            torch.cuda.synchronize()
            t = time.perf_counter()
            eng.transport_staged(seed + k, edep.data_ptr())
            torch.cuda.synchronize()
            tt.append(time.perf_counter() - t)
            st = eng.stats()
            tsteps += st["total_steps"]
            ttail.append(round(st["tail_kernel_ms"], 2))
        tables = dict(steps_per_s=tsteps / sum(tt), median_ms_per_transport=float(np.median(tt)) * 1e3,
                      ms_per_transport=[round(x * 1e3, 2) for x in tt], tail_ms_per_transport=ttail,
                      edep_vs_rejection=paired_layers(edep_tab, edep_first, gate=False),
                      note="table and rejection sampling draw different final states from the same "
                           "streams, so the histories decorrelate after the first interaction: the "
                           "per-layer comparison is reported, not gated")
        log(f"[bench] table sampling: {tables['steps_per_s']:.3g} steps/s")
        eng.configure(fs_alias=0)

    res["tables"] = tables

    # plain FP64 per-stage path on the same batch and first seed
    plain = None
    if args.plain_steps > 0:
        eng.configure(driver=gv.DRIVER_PLAIN, precision=gv.P64)
        tp = 0.0
        psteps = 0
        edep_plain = None
        for k in range(args.plain_steps):
            torch.cuda.synchronize()
            t = time.perf_counter()
            eng.transport_staged(seed, edep.data_ptr())
            torch.cuda.synchronize()
            dt = time.perf_counter() - t
            st = eng.stats()
            log(f"[bench] plain FP64 {k}: {dt*1e3:.1f} ms, {st['total_steps']} steps")
            if k == 0 and args.plain_steps > 1:
                edep_plain = edep.cpu().numpy()
                continue   # first call allocates the per-stage buffers
            tp += dt
            psteps += st["total_steps"]
            edep_plain = edep.cpu().numpy()
        n_timed = max(args.plain_steps - 1, 1) if args.plain_steps > 1 else 1
        plain = dict(steps_per_s=psteps / tp, primaries_per_s=len(prim) * n_timed / tp,
                     ms_per_transport=tp / n_timed * 1e3, timed_transports=n_timed)
        plain["edep_match"] = paired_layers(edep_first, edep_plain)
    # FP64 batched for context
    b64 = None
    if args.fp64_batched:
        eng.configure(driver=gv.DRIVER_BATCHED, precision=gv.P64)
        eng.transport_staged(seed, edep.data_ptr())
        torch.cuda.synchronize()
        t = time.perf_counter()
        eng.transport_staged(seed, edep.data_ptr())
        torch.cuda.synchronize()
        dt = time.perf_counter() - t
        st = eng.stats()
        b64 = dict(steps_per_s=st["total_steps"] / dt, primaries_per_s=len(prim) / dt, ms_per_transport=dt * 1e3)
        log(f"[bench] batched FP64: {dt*1e3:.1f} ms")
    # one GPU's share of an 8-way event split of the same batch, in one
    # transport: the population, and so the occupancy, is 8x smaller
    share = None
    if args.share_events > 0 and args.share_events < n_events:
        eng.configure(driver=gv.DRIVER_BATCHED, precision=gv.PMIX)
        sub = prim[prim["event"] < args.share_events]
        eng.stage(sub)
        eng.transport_staged(seed, edep.data_ptr())
        ts, ssteps = [], 0
        for k in range(3):
            torch.cuda.synchronize()
            t = time.perf_counter()
            eng.transport_staged(seed + k, edep.data_ptr())
            torch.cuda.synchronize()
            ts.append(time.perf_counter() - t)
            ssteps += eng.stats()["total_steps"]
        share = dict(events=int(args.share_events), steps_per_s=ssteps / sum(ts),
                     median_ms_per_transport=float(np.median(ts)) * 1e3)
        log(f"[bench] one GPU's share ({args.share_events} events): {share['steps_per_s']:.3g} steps/s")
        eng.stage(prim)
    res["share"] = share
    # last: the single-slab and field-map legs set up their own contexts (one per process)
    res["testem5"] = run_testem5(args, gv, torch, eng.config) if args.testem5 else None
    res["field_map"] = run_field_map(args, gv, torch, eng.config) if args.field_map else None
    res["barrel"] = run_barrel_precision(args, gv, torch, eng.config) if args.barrel else None
    return res, plain, b64


def run_testem5(args, gv, torch, cfg):
    """Single-slab transmission / reflection (10 MeV e- on 2 mm Pb, 20000
    primaries): mixed-precision throughput and the fractions of primaries'
    worth of e- leaving forward and backward, beside the oracle's."""
    import numpy as np

    import gv_inputs
    geom, prim, seed = gv_inputs.workload("t5")
    eng = gv.Engine(geom, driver=gv.DRIVER_BATCHED, precision=gv.PMIX, edep_on_device=1,
                    hip_stream=cfg["hip_stream"])
    edep = torch.zeros((len(prim), eng.n_cells), dtype=torch.float64, device="cuda:0")
    eng.stage(prim)
    eng.transport_staged(seed, edep.data_ptr())
    ts, steps = [], 0
    for k in range(3):
        torch.cuda.synchronize()
        t = time.perf_counter()
        eng.transport_staged(seed, edep.data_ptr())
        torch.cuda.synchronize()
        ts.append(time.perf_counter() - t)
        steps += eng.stats()["total_steps"]
    h = eng.escape_hist()
    n = len(prim)
    out = dict(workload="t5: 20000 x 10 MeV e- on 2 mm Pb", steps_per_s=steps / sum(ts),
               ms_per_transport=float(np.median(ts)) * 1e3,
               electrons_forward=float(h[1, :, 10:].sum() / n), electrons_backward=float(h[1, :, :10].sum() / n),
               photons_forward=float(h[0, :, 10:].sum() / n), photons_backward=float(h[0, :, :10].sum() / n))
    if not args.no_cpu:
        import oracle
        r = oracle.Oracle(geom).transport(prim, seed, n_threads=host_cpus()["threads"])["escape_hist"]
        out["oracle"] = dict(electrons_forward=float(r[1, :, 10:].sum() / n),
                             electrons_backward=float(r[1, :, :10].sum() / n),
                             photons_forward=float(r[0, :, 10:].sum() / n), photons_backward=float(r[0, :, :10].sum() / n))
    eng.close()
    log(f"[bench] testem5: {out['steps_per_s']:.3g} steps/s, e- forward {out['electrons_forward']:.4f} "
        f"backward {out['electrons_backward']:.4f}")
    return out


def run_barrel_precision(args, gv, torch, cfg):
    """The barrel in its 3.8 T field (c5: 2000 x 50 GeV e-/gamma): mixed
    precision against all-FP64, both batched on the GPU, on the same seed:
    throughput of each and the paired per-cell deposit comparison."""
    import numpy as np

    import gv_inputs
    geom, prim, seed = gv_inputs.workload("c5")
    eng = gv.Engine(geom, driver=gv.DRIVER_BATCHED, precision=gv.PMIX, edep_on_device=1,
                    hip_stream=cfg["hip_stream"])
    n_ev = int(prim["event"].max()) + 1
    edep = torch.zeros((n_ev, eng.n_cells), dtype=torch.float64, device="cuda:0")
    eng.stage(prim)
    out = dict(workload=f"c5: {len(prim)} x 50 GeV e-/gamma, barrel, 3.8 T along z")
    res = {}
    for name, prec in (("pmix", gv.PMIX), ("p64", gv.P64)):
        eng.configure(precision=prec)
        eng.transport_staged(seed, edep.data_ptr())
        ts, steps = [], 0
        for k in range(2):
            torch.cuda.synchronize()
            t = time.perf_counter()
            eng.transport_staged(seed, edep.data_ptr())
            torch.cuda.synchronize()
            ts.append(time.perf_counter() - t)
            steps += eng.stats()["total_steps"]
        res[name] = edep.cpu().numpy()
        out[name] = dict(steps_per_s=steps / sum(ts), ms_per_transport=float(np.median(ts)) * 1e3)
    out["pmix_vs_p64"] = paired_layers(res["pmix"], res["p64"])
    eng.close()
    log(f"[bench] barrel c5: mixed {out['pmix']['steps_per_s']:.3g} steps/s, FP64 {out['p64']['steps_per_s']:.3g} "
        f"steps/s, per-cell worst {out['pmix_vs_p64']['worst_rel_big_layers']:.2e}")
    return out


def run_field_map(args, gv, torch, cfg):
    """The barrel in the solenoid map (c5m: 2000 x 50 GeV e-/gamma), mixed
    precision: helix in the pre-step field against adaptive RK45 (Sec. 3.6),
    with the RK45 work per charged step and the fraction of idle lanes in the
    integration loop (the quantity of the paper's active-lanes table)."""
    import numpy as np

    import gv_inputs
    geom, prim, seed = gv_inputs.workload("c5m", args.field_events)
    eng = gv.Engine(geom, driver=gv.DRIVER_BATCHED, precision=gv.PMIX, edep_on_device=1,
                    hip_stream=cfg["hip_stream"])
    edep = torch.zeros((int(prim["event"].max()) + 1, eng.n_cells), dtype=torch.float64, device="cuda:0")
    eng.stage(prim)
    out = dict(workload=f"c5m: {len(prim)} x 50 GeV e-/gamma, barrel in a 3.8 T finite solenoid")
    for name, fm, order in (("helix", gv.FIELD_HELIX, gv.ORDER_ARRIVAL), ("rk45", gv.FIELD_RK45, gv.ORDER_ARRIVAL),
                            ("rk45_in_step", gv.FIELD_RK45, gv.ORDER_STABLE)):
        eng.configure(field_method=fm, queue_order=order)
        eng.transport_staged(seed, edep.data_ptr())
        ts, steps, sub, rej, slots, charged, kms, parked = [], 0, 0, 0, 0, 0, 0.0, 0
        reps = 3 if fm == gv.FIELD_HELIX else 2
        for k in range(reps):
            torch.cuda.synchronize()
            t = time.perf_counter()
            eng.transport_staged(seed, edep.data_ptr())
            torch.cuda.synchronize()
            ts.append(time.perf_counter() - t)
            st = eng.stats()
            steps += st["total_steps"]
            charged += st["steps"][1] + st["steps"][2]
            sub += st["rk_substeps"]
            rej += st["rk_rejected"]
            slots += st["rk_lane_slots"]
            parked += st["rk_parked"]
            kms += st["kernel_ms"]
        leg = dict(steps_per_s=steps / sum(ts), ms_per_transport=float(np.median(ts)) * 1e3,
                   kernel_ms_per_transport=kms / reps, e_dep_GeV=float(st["e_dep"]) * 1e-3 / len(prim),
                   tail_kernel_ms=float(st["tail_kernel_ms"]))
        # kernel time outside the low-population tail replays (the shower phase)
        leg["shower_kernel_ms"] = leg["kernel_ms_per_transport"] - leg["tail_kernel_ms"]
        if name != "helix":
            leg["shower_kernel_vs_helix"] = leg["shower_kernel_ms"] / max(out["helix"]["shower_kernel_ms"], 1e-9)
        if name == "rk45":
            leg["integration"] = ("integration queue: charged steps parked at their RK45 move while the population "
                                  "fills the GPU, integrated by one kernel with lanes refilled at every attempt")
        if name == "rk45_in_step":
            leg["integration"] = "each lane integrates its own track inside the step (stable-order queues)"
        if fm == gv.FIELD_RK45:
            leg.update(substeps_per_charged_step=sub / max(charged, 1), rejected_per_charged_step=rej / max(charged, 1),
                       substeps_per_s=sub / sum(ts), idle_lane_fraction=1.0 - (sub + rej) / max(slots, 1),
                       parked_fraction=parked / max(charged, 1))
        out[name] = leg
        log(f"[bench] field map {name}: {leg['steps_per_s']:.3g} steps/s, {leg['ms_per_transport']:.1f} ms"
            + (f", {leg['substeps_per_charged_step']:.2f} substeps + {leg['rejected_per_charged_step']:.2f} "
               f"rejected per charged step, idle lanes {leg['idle_lane_fraction']:.3f}" if fm == gv.FIELD_RK45 else ""))
    eng.close()
    return out


def host_cpus():
    """CPUs this process may run on, the pool size of the CPU legs (at most
    16: the host share of one GPU on a shared box), and the host's core count
    from lscpu."""
    avail = len(os.sched_getaffinity(0)) if hasattr(os, "sched_getaffinity") else (os.cpu_count() or 1)
    lscpu = {}
    try:
        import subprocess
        txt = subprocess.run(["lscpu"], capture_output=True, text=True, timeout=10).stdout
        for line in txt.splitlines():
            if ":" in line:
                k, v = line.split(":", 1)
                lscpu[k.strip()] = v.strip()
    except (OSError, ValueError):
        pass

    def num(k):
        try:
            return int(lscpu.get(k, "").split()[0])
        except (ValueError, IndexError):
            return None
    cores = None
    if num("Core(s) per socket") and num("Socket(s)"):
        cores = num("Core(s) per socket") * num("Socket(s)")
    return dict(available=avail, threads=max(1, min(avail, 16)), lscpu_cpus=num("CPU(s)"), lscpu_cores=cores,
                model=lscpu.get("Model name") or cpu_model())


def run_cpu_baseline(args):
    """The FP64 oracle on the host: the whole batch of the timed workload when
    it fits the time budget (then its deposits also serve as the reference of
    the paired per-layer test of the headline), else the first events; plus a
    single-thread rate on a small sample."""
    import numpy as np

    import gv_inputs
    import oracle
    geom, prim, seed = gv_inputs.workload(args.workload, args.events)
    cpus = host_cpus()
    threads = cpus["threads"]
    o = oracle.Oracle(geom)
    # single thread on the first events, for the per-core rate and the budget
    small = prim[prim["event"] < max(1, args.cpu_events // 10)]
    t = time.perf_counter()
    r1 = o.transport(small, seed, n_threads=1)
    dt1 = time.perf_counter() - t
    c1 = r1["counters"]
    steps1 = c1["steps_gamma"] + c1["steps_electron"] + c1["steps_positron"]
    rate1 = steps1 / dt1
    n_events = int(prim["event"].max()) + 1
    est_steps = steps1 / len(small) * len(prim)
    est_s = est_steps / (rate1 * threads * 0.6)
    full = args.cpu_full and est_s <= args.cpu_budget_s
    sample = prim if full else prim[prim["event"] < args.cpu_events]
    log(f"[bench] CPU oracle: {'whole batch' if full else f'first {args.cpu_events} events'} on {threads} threads "
        f"(estimate for the whole batch {est_s:.0f} s)")
    t = time.perf_counter()
    r = o.transport(sample, seed, n_threads=threads)
    dt = time.perf_counter() - t
    c = r["counters"]
    steps = c["steps_gamma"] + c["steps_electron"] + c["steps_positron"]
    what = f"the whole batch ({n_events} events" if full else f"first {args.cpu_events} events of the same batch ("
    out = dict(value=steps / dt, unit="steps/s", cores=threads, kind="oracle",
               sample=f"{what}, {len(sample)} primaries, {steps} steps, {dt:.1f} s, FP64 history-based, "
                      f"{threads} threads)",
               primaries_per_s=len(sample) / dt, cpu_model=cpus["model"], host_cpus_lscpu=cpus["lscpu_cpus"],
               host_cores_lscpu=cpus["lscpu_cores"], cpus_available=cpus["available"],
               single_thread_steps_per_s=rate1,
               single_thread_sample=f"first {len(small)} events, {steps1} steps, {dt1:.1f} s")
    return out, (r["edep"] if full else None)


def cpu_model():
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return None


def copy_probe(nbytes, reps):
    """Device-to-device copy of a known size: the calibration run for the HBM
    byte counters (their reading for this copy against 2 x nbytes moved)."""
    import torch
    torch.cuda.set_device(0)
    n = nbytes // 4
    x = torch.ones(n, dtype=torch.float32, device="cuda:0")
    y = torch.empty_like(x)
    for _ in range(reps):
        y.copy_(x)
    torch.cuda.synchronize()
    log(f"[bench] copy probe: {reps} x {n * 4} bytes read and written")


def main():
    ap = argparse.ArgumentParser(description=__doc__.split("\n")[0])
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--workload", default="c4")
    ap.add_argument("--events", type=int, default=None)
    ap.add_argument("--basket", type=int, default=0)
    ap.add_argument("--occupancy", type=int, default=0)
    ap.add_argument("--inner", type=int, default=0)
    ap.add_argument("--graph-steps", type=int, default=0,
                    help="step launches per bulk graph replay (0: the library's default)")
    ap.add_argument("--plain-steps", type=int, default=2)
    ap.add_argument("--testem5", type=int, default=1, help="run the single-slab leg")
    ap.add_argument("--field-map", type=int, default=1, help="run the solenoid-map (helix vs RK45) leg")
    ap.add_argument("--share-events", type=int, default=1250,
                    help="events of the one-GPU-share leg (an 8-way split of the batch); 0 = skip")
    ap.add_argument("--field-events", type=int, default=None, help="events of the solenoid-map leg")
    ap.add_argument("--barrel", type=int, default=1, help="run the barrel mixed-vs-FP64 leg")
    ap.add_argument("--table-steps", type=int, default=3,
                    help="timed transports with table (alias) final-state sampling")
    ap.add_argument("--fp64-batched", type=int, default=1)
    ap.add_argument("--cpu-events", type=int, default=600,
                    help="events of the CPU oracle sample when the whole batch does not fit the budget")
    ap.add_argument("--cpu-full", type=int, default=1, help="run the CPU oracle on the whole batch if it fits")
    ap.add_argument("--cpu-budget-s", type=float, default=60.0,
                    help="estimated wall time up to which the CPU oracle runs the whole batch")
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--no-pcie", action="store_true", help="skip the host-buffer (PCIe-inclusive) transport")
    ap.add_argument("--out", default=None)
    ap.add_argument("--copy-probe", type=int, default=0, metavar="BYTES",
                    help="only run a device copy of BYTES (counter calibration) and exit")
    args = ap.parse_args()
    if args.copy_probe:
        copy_probe(args.copy_probe, 3)
        return
    if args.gpus != 1:
        print(f"bench.py measures one GPU (asked for --gpus {args.gpus}): the transport shards by event across "
              f"GPUs with no communication inside the step loop, so N GPUs run N independent event ranges",
              file=sys.stderr)
        sys.exit(2)

    res, plain, b64 = run_gpu(args)
    cpu, edep_oracle = (None, None) if args.no_cpu else run_cpu_baseline(args)
    # the headline's matched-edep check against the FP64 oracle itself: the
    # first timed transport (same primaries and seed) against the oracle's
    # deposits, paired per layer
    vs_oracle = paired_layers(res["edep_first"], edep_oracle) if edep_oracle is not None else None

    value = res["steps"] / res["elapsed"]
    ms = res["elapsed"] / args.steps * 1e3
    avg_launch_s = res["kernel_ms"] * 1e-3 / max(res["launches"], 1)
    bytes_per_launch = res["alg_bytes"] / max(res["launches"], 1)
    achieved = bytes_per_launch / avg_launch_s if avg_launch_s > 0 else 0.0
    st0 = res["stats0"]
    steps_per_launch = res["steps"] / max(res["launches"], 1)
    workload_id = f"{args.workload}x{res['primaries'] // args.steps}"
    traffic = measured_traffic(steps_per_launch, workload_id,
                               (st0["basket"], st0["occupancy"], st0["inner_steps"]))
    out = {
        "metric": METRIC,
        "value": value,
        "unit": "steps/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32/f64",
        "data": "synthetic",
        "config": {
            "workload": ("c4: 50 x (2.3 mm Pb + 5.7 mm lAr) 40x40 cm, 4 T along y, 10000 events, one primary "
                         "each (e-/e+/gamma by event mod 3), T log-uniform 100 MeV-100 GeV, 1 mrad spread"
                         if args.workload == "c4" and args.events is None else f"{args.workload} x {args.events}"),
            "events": res["n_events"], "primaries_per_step": res["primaries"] // args.steps,
            "driver": "batched persistent kernel, graph-captured step loop",
            "precision": "mixed: FP32 physics/tables/direction/energy, FP64 position/boundary/deposit",
            "basket": st0["basket"], "occupancy": st0["occupancy"], "inner_steps": st0["inner_steps"],
            "graph_steps": st0["graph_steps"], "autotuned": bool(st0["tuned"]),
            "queue_order": "stable" if st0["queue_order"] else "arrival"},
        "primaries_per_s": res["primaries"] / res["elapsed"],
        "median_ms_per_transport": res["median_ms"],
        "ms_per_transport": [round(x, 2) for x in res["per_ms"]],
        "tail_ms_per_transport": [round(x, 2) for x in res["tail_ms"]],
        "autotune_ms": res["autotune_ms"],
        # set-up outside the timed steps: gv_init (tables built on the device)
        # and the warm-up transports (autotuning and graph capture included)
        "init_ms": st0["init_ms"],
        "warmup_ms": res["warm_ms"],
        # share of the stepping loop's lane slots that took a step (steps over
        # 64 x loop iterations of every wavefront, timed transports)
        "lane_use": res["steps"] / res["lane_slots"] if res["lane_slots"] else None,
        "pcie_inclusive": {"ms_per_transport": res["pcie_inclusive_ms"],
                           "steps_per_s": res["pcie_inclusive_steps_per_s"]},
        "track_steps_per_transport": res["steps"] / args.steps,
        # the two phases of a transport: the shower (population above the
        # tail threshold) and the low-population tail of looping tracks
        "shower_steps_per_s": ((res["steps"] - res["tail_steps"]) /
                               max((sum(res["kern_ms"]) - sum(res["tail_ms"])) * 1e-3, 1e-12)),
        "tail_fraction": sum(res["tail_ms"]) / max(sum(res["per_ms"]), 1e-12),
        "tail_steps_per_transport": res["tail_steps"] / args.steps,
        "helper_steps_per_transport": res["helper_steps"] / args.steps,
        "edep_vs_oracle": vs_oracle,
        "plain_fp64": plain,
        "speedup_vs_plain_fp64": (value / plain["steps_per_s"]) if plain else None,
        "batched_fp64": b64,
        "table_sampling": res["tables"],
        "testem5": res["testem5"],
        "field_map": res["field_map"],
        "barrel_precision": res["barrel"],
        "one_gpu_share": res["share"],
        "roofline": {"bound": "hbm", "achieved": achieved / 1e9, "peak": HBM_PEAK / 1e9, "unit": "GB/s",
                     "frac": achieved / HBM_PEAK, "traffic": traffic,
                     "kernel": "k_step_batched<PMix,%d> and k_pool<PMix>" % min(st0["basket"], 256),
                     "launch": "one launch of the step kernel (populations that fill the GPU) or of the pool "
                               "kernel (the others), with the k_vacuum_helper before it where loopers alone are left",
                     "avg_launch_us": avg_launch_s * 1e6, "alg_bytes_per_launch": bytes_per_launch,
                     "steps_per_launch": steps_per_launch, "launches": res["launches"],
                     "kernel_source_sha1": kernel_source_hash(),
                     # the same bytes over the launches of the shower phase only
                     # (the tail's looper steps, 108 B each, taken out)
                     "shower_phase": shower_roofline(res)},
        "cpu_baseline": cpu,
    }
    line = json.dumps(out)
    if args.out:
        with open(args.out, "w") as f:
            f.write(line + "\n")
    print(line, flush=True)


if __name__ == "__main__":
    main()
