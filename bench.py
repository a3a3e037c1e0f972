#!/usr/bin/env python3
"""Benchmark of the Spring-Ising hot path on one MI355X.

Workload: the plain FP32 method on a K2000-shaped instance -- a complete
graph of N = 2000 spins with iid +-1 couplings (seeded synthetic stand-in
for the K2000 benchmark), R = 1024 replicas started at x0 ~ U(-0.1, 0.1) with
zero momenta, 10000 iterations of Eq. (8) with the paper's linear zeta
schedule (k = 0.5, Delta = 0.2, m = 1, zeta 0.04 -> 0.5, walls sqrt 2 / 2),
then the int32 Ising energy of sign(q) for every replica.

One benchmark step = one such full run (reset to x0, 10000 iterations,
energy readout).  Reported value: spin-updates/s = N * R * iterations / s.

Beside the headline line the same run is timed in the BF16 precision forms,
and time-to-target-energy is measured: the target is the 1% quantile of the
final energies of an FP32 run from other initial states; each form runs the
same schedule from five initial states with the exact energy of every
replica checked every 50 steps on the device (check cost included, timed
with HIP events on the stream the kernels run on); its time-to-target for
an initial state is the event time of the first check with a replica at or
below the target, and the form's figure is the median over the five.
The precision form's full configurations (R = 2048: FP8 J at N = 2000, hi +
lo BF16 J at N = 8000) are timed per step against FP32 on the same shapes,
and their time to target is measured with the same protocol over their
5000-step schedule.
The batched configuration (256 uneven instances, R = 64) is timed per step
in FP32 and in the BF16 form (also as a graph replay), with a time to a
per-instance target energy, and against the same instances stepped one
after another; the differentiation configuration (schedule gradient at
N = 2000, R = 64, 2000 steps) is timed beside its plain forward run.

    python bench.py [--steps K] [--warmup W] [--gpus 1]
"""
from __future__ import annotations

import argparse
import json
import os
import re
import sys
import time

# The CPU baseline's BLAS uses every core of this process's share; set before
# NumPy is first imported (an OMP_NUM_THREADS already set by the host wins).
os.environ.setdefault("OMP_NUM_THREADS", str(len(os.sched_getaffinity(0))))
os.environ.setdefault("OPENBLAS_NUM_THREADS", os.environ["OMP_NUM_THREADS"])

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

N, R, ITERS = 2000, 1024, 10000
CHECK_EVERY = 50
# MI355X published peaks
PEAK_FP32_MFMA_TFLOPS = 157.3
PEAK_BF16_MFMA_TFLOPS = 2500.0
PEAK_HBM_GBS = 8000.0
PEAK_INT8_MFMA_TOPS = 5000.0
FORMS = ["bf16x_fp8j", "bf16x_bf16j", "bf16x3_exactj"]
# HBM/MALL bytes per launch of a step kernel, from two rocprofv3 counter
# passes (FETCH_SIZE x 2.000 + WRITE_SIZE x 1.000; the factors come from an
# elementwise kernel of known size in the same runs).  Keyed by (kernel,
# precision, N, R); an entry is removed whenever that kernel's code changes.
MEASURED_TRAFFIC_BYTES = {
    ("step_f32_64x128_w2x4_mfma32_k32_s4_a1", "fp32", 2000, 1024): 113.20e6,
    ("step_bf16_128x64_w4x2_k128_s3_p2", "bf16x_fp8j", 2000, 1024): 75.63e6,
    ("step_bf16_128x64_w4x2_k128_s3_p2", "bf16x_bf16j", 2000, 1024): 79.83e6,
    ("step_bf16_128x64_w4x2_k64_s3_p1", "bf16x3_exactj", 2000, 1024): 155.29e6,
    ("step_bf16_128x128_w4x2_k128_s3", "bf16x_fp8j", 2000, 2048): 146.93e6,
    ("step_bf16_128x256_w2x4_k64_s2_p1", "bf16x_hiloj", 8000, 2048): 1143.93e6,
}
# The same of the fixed-point form, which has no tile table to check names against.
FIXED_POINT_TRAFFIC_BYTES = {
    ("step_i8x4_256x32_w4_k256_s3", "fp32", 2000, 1024): 80.12e6,
    ("step_i8x4_256x32_w4_k256_s3", "bf16x3_exactj", 2000, 1024): 80.12e6,
    ("step_i8x10_128x64_w4_k128_s3", "fp32", 8000, 2048): 2463.0e6,
}


def _cpu_model():
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def _oracle_steps(J, Q, P, iters, budget_s):
    """FP64 oracle steps of the paper schedule until `iters` or the budget."""
    import numpy as np

    import oracle
    dt = oracle.dt_schedule(iters)
    zeta = oracle.zeta_schedule(iters, float(np.float32(0.04)), float(np.float32(0.5)))
    qmax = float(np.float32(np.sqrt(2.0)))
    t0 = time.perf_counter()
    done = 0
    while done < iters and time.perf_counter() - t0 < budget_s:
        Q, P = oracle.step(J, Q, P, float(dt[done]), float(zeta[done]), qmax=qmax)
        done += 1
    return done, time.perf_counter() - t0


def cpu_baseline(budget_s: float = 15.0, subset_budget_s: float = 6.0):
    """Time the FP64 oracle (as it stands, J @ Q on the host BLAS) on a
    bounded sample of the headline workload on the host cores and
    extrapolate per iteration; also on the precision form's N = 8000
    Gaussian configuration at R = 64 and on 16 sampled instances of the
    batched configuration (R = 64)."""
    import numpy as np

    from paper_2305_07187_amd import instances
    try:
        from threadpoolctl import threadpool_info
        cores = max((i.get("num_threads", 1) for i in threadpool_info()), default=os.cpu_count())
    except Exception:
        cores = os.cpu_count()
    J = instances.make_pm1(N, 0).astype(np.float64)
    Q = instances.make_x0(N, R, 0).T.astype(np.float64)
    done, el = _oracle_steps(J, Q, np.zeros_like(Q), ITERS, budget_s)
    out = {"value": N * R * done / el, "unit": "spin-updates/s", "cores": int(cores),
           "kind": "oracle",
           "sample": f"first {done} of {ITERS} iterations at N={N}, R={R} (FP64 NumPy, "
                     f"{el:.1f} s), extrapolated per iteration",
           "cpu_model": _cpu_model(), "affinity_cpus": len(os.sched_getaffinity(0)),
           "blas_threads_env": os.environ.get("OPENBLAS_NUM_THREADS")}
    # precision form, Gaussian N = 8000, on an R = 64 subset of its R = 2048
    n8, r8 = 8000, 64
    # the same values as instances.make_gauss, drawn by the torch form of the
    # generator on the device (the NumPy form takes about 15 s at this size)
    import torch
    gen_dev = torch.device("cuda:0") if torch.cuda.is_available() else torch.device("cpu")
    J8 = instances.make_J_torch(n8, "gauss", 0, gen_dev).cpu().numpy().astype(np.float64)
    Q8 = instances.make_x0(n8, r8, 0).T.astype(np.float64)
    d8, e8 = _oracle_steps(J8, Q8, np.zeros_like(Q8), 5000, subset_budget_s)
    del J8, Q8
    # batched form: 16 of the 256 instances (every 16th of the recipe), R = 64
    recipe = instances.make_batch(256, 0)[::16]
    spins_done, el3, steps3 = 0, 0.0, 0
    per = subset_budget_s / len(recipe)
    for n_i, kind, seed in recipe:
        Ji = instances.make_J(n_i, kind, seed).astype(np.float64)
        Qi = instances.make_x0(n_i, 64, seed).T.astype(np.float64)
        d, e = _oracle_steps(Ji, Qi, np.zeros_like(Qi), 3000, per)
        spins_done += n_i * 64 * d
        el3 += e
        steps3 += d
    out["subsets"] = {
        "precision_gauss_n8000": {"value": n8 * r8 * d8 / e8, "unit": "spin-updates/s",
                                  "sample": f"{d8} iterations at N={n8}, R={r8} of R=2048 "
                                            f"(FP64 NumPy, {e8:.1f} s)"},
        "batched_16_instances": {"value": spins_done / el3, "unit": "spin-updates/s",
                                 "sample": f"{steps3} iterations over 16 of the 256 instances "
                                           f"(N {min(r[0] for r in recipe)}..{max(r[0] for r in recipe)}), "
                                           f"R=64 ({el3:.1f} s)"}}
    return out


def batched_form(si, steps=300, n_inst=256, r=64, sequential=True, time_to_target=True):
    """The batched configuration (256 uneven instances, N in [64, 4096], half
    +-1 and half Gaussian, R = 64): ms per step of all instances together,
    batched in FP32 and in the BF16 form (FP8 / hi + lo J), and (unless
    sequential is off) the same instances stepped one after another as
    single FP32 contexts; unless time_to_target is off, the time to a target
    energy of both batched forms."""
    import torch

    from paper_2305_07187_amd import instances
    dev = torch.device("cuda:0")
    recipe = instances.make_batch(n_inst, 0)
    Js = [instances.make_J_torch(n, kind, seed, dev) for n, kind, seed in recipe]
    xs = [instances.make_x0_torch(n, r, seed, device=dev) for n, kind, seed in recipe]
    torch.cuda.synchronize()
    out = {"workload": f"{n_inst} instances, N uniform in [64, 4096] (sum {sum(n for n, _, _ in recipe)}), "
                       f"half +-1 half Gaussian, R={r}", "steps_timed": steps}
    for form in ("fp32", "bf16x_mixedj"):
        # the autotuner picks the batch tile on a context of its own; the
        # timed context (and the time-to-target runs) read it from the cache
        tb = si.SpringIsingBatch(Js, xs, total_steps=20, precision=form)
        tile, us = tb.autotune(6)
        tb.close()
        b = si.SpringIsingBatch(Js, xs, total_steps=steps + 10, precision=form)
        info = b.info()
        out[f"{form}_tile"] = {"autotuned": tile, "autotune_us": round(us, 1),
                               "used": info["tile"],
                               "source": si.TILE_SOURCES[info["tile_source"]]}
        b.run(10)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        b.run(steps)
        torch.cuda.synchronize()
        out[f"{form}_batched_ms_per_step"] = 1000.0 * (time.perf_counter() - t0) / steps
        out[f"{form}_kernel"] = b.info()["kernel_name"]
        # a restart of the schedule replays the HIP graph its first run captured
        b.set_graph(steps)
        b.set_state(xs, None, 0)
        b.run(steps)
        b.set_state(xs, None, 0)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        b.run(steps)
        torch.cuda.synchronize()
        out[f"{form}_batched_graph_ms_per_step"] = 1000.0 * (time.perf_counter() - t0) / steps
        # where the step's time goes: two traced steps (CU busy share of the
        # step, the tail after the first CU runs out of work, the gap between
        # the two launches)
        rec, mhz = b.timeline(2)
        st = si.batch_timeline_stats(rec, mhz)
        out[f"{form}_timeline"] = {
            "span_us": round(st[0]["span_us"], 1), "cu_busy_mean": round(st[0]["cu_busy_mean"], 4),
            "cu_busy_min": round(st[0]["cu_busy_min"], 4), "tail_us": round(st[0]["tail_us"], 1),
            "launch_gap_us": round(st[0]["gap_to_next_us"], 2)}
        b.close()
    if time_to_target:
        ref_xs = [instances.make_x0_torch(n, r, seed ^ 0x5A5A5A5A, device=dev)
                  for n, kind, seed in recipe]
        out["time_to_target"] = batched_time_to_target(si, Js, xs, ref_xs,
                                                       sequential=sequential)
    if not sequential:
        return out
    seq = 0.0
    for J, x in zip(Js, xs):
        m = si.SpringIsing(J, x, total_steps=30)
        m.run(5)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        m.run(25)
        torch.cuda.synchronize()
        seq += (time.perf_counter() - t0) / 25
        m.close()
    out["fp32_sequential_ms_per_step"] = 1000.0 * seq
    out["batched_vs_sequential_fp32"] = seq * 1000.0 / out["fp32_batched_ms_per_step"]
    out["bf16_vs_fp32_batched"] = (out["fp32_batched_ms_per_step"] /
                                   out["bf16x_mixedj_batched_ms_per_step"])
    return out


def _chunked_run(model, every, checks, stream):
    """model.run(every) `checks` times with a HIP event after each chunk (the
    in-run energy check closes every chunk); returns the event times in s
    from the start."""
    import torch
    evs = [torch.cuda.Event(enable_timing=True) for _ in range(checks + 1)]
    evs[0].record(stream)
    for c in range(checks):
        model.run(every)
        evs[c + 1].record(stream)
    torch.cuda.synchronize()
    return [evs[0].elapsed_time(e) / 1000.0 for e in evs[1:]]


def batched_time_to_target(si, Js, xs, ref_xs, steps=3000, every=100, rank=13,
                           sequential=True):
    """Time to target energy of the batched forms over the batched workload's
    3000 steps.  Each instance's target is the `rank`-th best of its R final
    energies in a separate FP32 batch run from other initial states (ref_xs),
    so that no timed form is measured against its own final energies.  The
    energies of all instances are checked on the device every `every` steps
    (si_params.energy_every, the check cost included); a batched form's time
    to target is the HIP-event time of the first check at which every
    instance has a replica at or below its target.  The sequential FP32
    reference steps each instance alone as a single FP32 context with the
    same checks until it reaches its target; its time to target is the sum of
    those per-instance times (the instances solved one after another)."""
    import numpy as np
    import torch

    stream = torch.cuda.current_stream()
    checks = steps // every
    out = {"steps": steps, "check_every": every,
           "target": f"per instance, the {rank}th best of R final energies of an FP32 run "
                     f"from other initial states"}
    ref = si.SpringIsingBatch(Js, ref_xs, total_steps=steps, precision="fp32")
    ref.run(steps)
    targets = np.sort(torch.stack(ref.energy(exact=False)).cpu().numpy(), axis=1)[:, rank - 1]
    ref.close()
    for form in ("fp32", "bf16x_mixedj"):
        b = si.SpringIsingBatch(Js, xs, total_steps=steps, precision=form, energy_every=every)
        b.run(every)  # warm-up
        b.set_state(xs, None, 0)
        torch.cuda.synchronize()
        times = _chunked_run(b, every, checks, stream)
        mins = b.energy_trace().min(dim=2).values.cpu().numpy()  # [checks, n_inst]
        b.close()
        hit = np.nonzero((mins <= targets[None, :]).all(axis=1))[0]
        out[form] = {"ttt_s": float(times[hit[0]]) if len(hit) else None,
                     "ttt_step": int((hit[0] + 1) * every) if len(hit) else None,
                     "instances_at_target_at_end": int((mins[-1] <= targets).sum())}
    t32, t16 = out["fp32"]["ttt_s"], out["bf16x_mixedj"]["ttt_s"]
    out["bf16_speedup_vs_fp32"] = (t32 / t16) if (t32 and t16) else None
    if sequential:
        total, reached, block = 0.0, 0, 5
        for i, (J, x) in enumerate(zip(Js, xs)):
            m = si.SpringIsing(J, x, total_steps=steps, energy_every=every)
            m.run(every)  # warm-up (code objects of this instance's tile)
            m.set_state(x, None, 0)
            torch.cuda.synchronize()
            t_i, done = None, 0
            while done < checks and t_i is None:
                k = min(block, checks - done)
                times = _chunked_run(m, every, k, stream)
                mins = m.energy_trace()[done:done + k].min(dim=1).values.cpu().numpy()
                h = np.nonzero(mins <= targets[i])[0]
                if len(h):
                    t_i = float(times[h[0]])
                else:
                    total += times[-1]
                done += k
            if t_i is not None:
                total += t_i
                reached += 1
            m.close()
        out["fp32_sequential"] = {"ttt_s": total, "instances_reaching_target": reached,
                                  "note": "each instance alone (single FP32 context, its own "
                                          "automatic tile), stopped at its first check at or "
                                          "below its target; times summed"}
        t_seq = total if reached == len(Js) else None
        out["batched_fp32_speedup_vs_sequential"] = (t_seq / t32) if (t_seq and t32) else None
        out["batched_bf16_speedup_vs_sequential"] = (t_seq / t16) if (t_seq and t16) else None
    return out


def precision_full_configurations(si, r=2048, total=5000, steps=200, warm=20):
    """The precision form at its full configurations (R = 2048, the 5000-step
    schedule): FP8 J at N = 2000 (+-1 couplings) and hi + lo BF16 J at
    N = 8000 (Gaussian couplings), each against the plain FP32 step on the
    same shape.  HIP-event time of `steps` steps after `warm` warm-up steps."""
    import torch

    from paper_2305_07187_amd import instances
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream()
    out = {"replicas": r, "schedule_steps": total, "steps_timed": steps}
    for key, n, kind, form in (("fp8j_n2000", 2000, "pm1", "bf16x_fp8j"),
                               ("hiloj_n8000", 8000, "gauss", "bf16x_hiloj")):
        J = instances.make_J_torch(n, kind, 0, dev)
        x0 = instances.make_x0_torch(n, r, 0, device=dev)
        rec = {"n": n, "couplings": kind}
        for prec in (form, "fp32"):
            m = si.SpringIsing(J, x0, total_steps=total, precision=prec)
            m.run(warm)
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record(stream)
            m.run(steps)
            b.record(stream)
            torch.cuda.synchronize()
            ms = a.elapsed_time(b) / steps
            rec[prec] = {"ms_per_step": ms, "spin_updates_per_s": n * r / (ms / 1000.0),
                         "kernel": m.info()["kernel_name"]}
            m.close()
        rec["speedup_vs_fp32"] = rec["fp32"]["ms_per_step"] / rec[form]["ms_per_step"]
        out[key] = rec
        del J, x0
    return out


def precision_time_to_target(si, r=2048, total=5000):
    """Time to target energy at the precision form's own configurations
    (R = 2048, the 5000-step schedule): FP8 J against FP32 at N = 2000 (+-1
    couplings, initial seeds 0-4, checks every 50 steps) and hi + lo BF16 J
    against FP32 at N = 8000 (Gaussian couplings, seeds 0-2, checks every 100
    steps, real-valued energies), with the protocol of time_to_target."""
    import torch

    from paper_2305_07187_amd import instances
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream()
    out = {"replicas": r, "schedule_steps": total}
    for key, n, kind, form, every, seeds in (("fp8j_n2000", 2000, "pm1", "bf16x_fp8j", 50, TTT_SEEDS),
                                            ("hiloj_n8000", 8000, "gauss", "bf16x_hiloj", 100,
                                             TTT_SEEDS[:3])):
        J = instances.make_J_torch(n, kind, 0, dev)
        rec = time_to_target(si, J, n, r, total, every, stream, 0, forms_timed=[form],
                             seeds=seeds)
        rec["n"] = n
        rec["couplings"] = kind
        out[key] = rec
        del J
        torch.cuda.synchronize()
    return out


def differentiation_form(si, n=2000, r=64, steps=2000, ckpt=100, repeats=3):
    """The differentiation configuration: gradient of the mean relaxed
    end-energy with respect to the 2000-entry Delta and zeta schedules at
    N = 2000, R = 64 (checkpoints every 100 steps), timed end to end on the
    stream (forward with checkpoints, per-segment recomputation, backward),
    beside the plain forward run of the same length."""
    import torch

    from paper_2305_07187_amd import instances
    dev = torch.device("cuda:0")
    J = instances.make_J_torch(n, "pm1", 0, device=dev)
    x0 = instances.make_x0_torch(n, r, 0, device=dev)
    stream = torch.cuda.current_stream()
    m = si.SpringIsing(J, x0, total_steps=steps)
    m.relaxed_energy_grad(ckpt)  # warm-up
    grad_ms, fwd_ms = [], []
    for _ in range(repeats):
        a, b, c = (torch.cuda.Event(enable_timing=True) for _ in range(3))
        m.set_state(x0, None, 0)
        a.record(stream)
        m.run(steps)
        b.record(stream)
        m.set_state(x0, None, 0)
        torch.cuda.synchronize()
        c0 = torch.cuda.Event(enable_timing=True)
        c0.record(stream)
        loss, gd, gz = m.relaxed_energy_grad(ckpt)
        c.record(stream)
        torch.cuda.synchronize()
        fwd_ms.append(a.elapsed_time(b))
        grad_ms.append(c0.elapsed_time(c))
    out = {"workload": f"N={n} +-1, R={r}, {steps}-step schedule, checkpoint every {ckpt}",
           "kernel": m.info()["kernel_name"], "gradient_ms": min(grad_ms),
           "forward_ms": min(fwd_ms), "gradient_over_forward": min(grad_ms) / min(fwd_ms),
           "loss": float(loss.cpu()[0]), "finite": bool(torch.isfinite(gd).all() and
                                                      torch.isfinite(gz).all())}
    m.close()
    return out


def timed_runs(model, x0, iters, steps, warmup, stream):
    """Full runs (reset, iters steps, energy); per-run HIP events bracket the
    step launches.  Returns (elapsed_s, per-launch us, last energies)."""
    import torch
    exact = bool(model.info()["j_integer"])

    def one_run(ev=None):
        model.set_state(x0, None, 0)
        if ev is not None:
            ev[0].record(stream)
        model.run(iters)
        if ev is not None:
            ev[1].record(stream)
        return model.energy(exact=exact)

    for _ in range(warmup):
        one_run()
    torch.cuda.synchronize()
    evs = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
           for _ in range(steps)]
    t0 = time.perf_counter()
    energies = None
    for k in range(steps):
        energies = one_run(evs[k])
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    run_ms = [a.elapsed_time(b) for a, b in evs]
    kernel_us = 1000.0 * sum(run_ms) / (len(run_ms) * iters)
    return elapsed, kernel_us, energies


TTT_SEEDS = (0, 1, 2, 3, 4)
TTT_TARGET_SEED = 5


def time_to_target(si, J, n, r, iters, every, stream, runs_per_form, forms_timed=None,
                   seeds=TTT_SEEDS):
    """Time to target energy, BF16 forms against FP32, on the headline
    instance.  Target: the 1 % quantile (10th best of 1024) of the final
    energies of an FP32 run from initial positions of seed 5, so that no
    timed run is measured against its own final energies.  Every form runs
    the whole schedule from the initial positions of seeds 0-4 with the
    energies of all replicas checked on the device every `every` steps
    (si_params.energy_every; check cost included); its time to target for a
    seed is the HIP-event time of the first check with a replica at or below
    the target, and the form's figure is the median over the seeds.  Equal
    final-energy distribution: a two-sample KS test of the pooled final
    energies (R x 5 seeds) against FP32's, and the difference of the means in
    standard errors.  TTS99 takes one replica as a trial: P_s is the pooled
    fraction of replicas ending at or below the target, a trial costs its
    share t_run / R of a run of all R replicas together, and
    TTS99 = (t_run / R) ln(0.01) / ln(1 - P_s).  P_run = 1 - (1 - P_s)^R is
    the chance that a whole run reaches the target.  forms_timed: the BF16
    forms to compare (default all three); runs_per_form = 0 skips the
    separate throughput runs without checks."""
    import math

    import numpy as np
    from scipy.stats import ks_2samp

    from paper_2305_07187_amd import instances
    dev = J.device
    checks = iters // every
    mref = si.SpringIsing(J, instances.make_x0_torch(n, r, TTT_TARGET_SEED, device=dev),
                          total_steps=iters, precision="fp32")
    mref.run(iters)
    e_ref = mref.energy(exact=bool(mref.info()["j_integer"])).cpu().numpy().astype(np.float64)
    mref.close()
    target = float(np.sort(e_ref)[max(0, int(0.01 * r) - 1)])
    forms_timed = list(FORMS if forms_timed is None else forms_timed)
    x0s = {sd: instances.make_x0_torch(n, r, sd, device=dev) for sd in seeds}
    forms, finals = {}, {}
    for name in ["fp32"] + forms_timed:
        # throughput of the form on full runs without in-run checks
        el_tot, us = None, None
        if runs_per_form > 0:
            plain = si.SpringIsing(J, x0s[seeds[0]], total_steps=iters, precision=name)
            el_tot, us, _ = timed_runs(plain, x0s[seeds[0]], iters, runs_per_form, 1, stream)
            plain.close()
        m = si.SpringIsing(J, x0s[seeds[0]], total_steps=iters, precision=name, energy_every=every)
        m.run(every)  # warm-up
        per_seed, pooled = [], []
        for sd in seeds:
            m.set_state(x0s[sd], None, 0)
            times = _chunked_run(m, every, checks, stream)
            tr = m.energy_trace().cpu().numpy()
            hit = np.nonzero(tr.min(axis=1) <= target)[0]
            per_seed.append({"seed": sd, "ttt_s": float(times[hit[0]]) if len(hit) else None,
                             "ttt_step": int((hit[0] + 1) * every) if len(hit) else None,
                             "run_s": float(times[-1])})
            pooled.append(tr[-1])  # the last check is at the final step
        kernel = m.info()["kernel_name"]
        m.close()
        fin = np.concatenate(pooled)
        finals[name] = fin
        ttts = sorted((p["ttt_s"] if p["ttt_s"] is not None else math.inf) for p in per_seed)
        med = ttts[len(ttts) // 2]
        p_s = float((fin <= target).mean())
        t_run = float(np.median([p["run_s"] for p in per_seed]))
        t_trial = t_run / r
        if p_s >= 0.99:
            tts99 = t_trial
        elif p_s > 0:
            tts99 = t_trial * math.log(0.01) / math.log(1.0 - p_s)
        else:
            tts99 = None
        forms[name] = {"kernel": kernel,
                       "spin_updates_per_s": (n * r * iters * runs_per_form / el_tot
                                              if el_tot else None),
                       "avg_launch_us": us,
                       "ttt_median_s": med if math.isfinite(med) else None,
                       "per_seed": per_seed, "run_with_checks_s": t_run,
                       "p_success": p_s, "p_run": 1.0 - (1.0 - p_s) ** r, "tts99_s": tts99,
                       "mean_energy": float(fin.mean()), "best_energy": float(fin.min())}
    t32 = forms["fp32"]["ttt_median_s"]
    for name in forms_timed:
        f = forms[name]
        f["ks_pvalue_vs_fp32"] = float(ks_2samp(finals[name], finals["fp32"]).pvalue)
        a, b = finals[name], finals["fp32"]
        f["mean_diff_in_se"] = float((a.mean() - b.mean()) /
                                     math.sqrt(a.var() / len(a) + b.var() / len(b)))
        f["equal_distribution"] = bool(f["ks_pvalue_vs_fp32"] >= 0.01 and
                                       abs(f["mean_diff_in_se"]) <= 2.0)
        tf = f["ttt_median_s"]
        f["ttt_speedup_vs_fp32"] = (t32 / tf) if (t32 and tf) else None
        f["tts99_speedup_vs_fp32"] = (forms["fp32"]["tts99_s"] / f["tts99_s"]
                                      if (forms["fp32"]["tts99_s"] and f["tts99_s"]) else None)
    return {"target_energy": target, "check_every": every, "seeds": list(seeds),
            "target": f"1% quantile of the final energies of an FP32 run from initial "
                      f"positions of seed {TTT_TARGET_SEED}",
            "forms": forms}


def energy_readout(si, model, n, r, calls, stream):
    """HIP-event time of the exact Eq. (1) readout of all replicas (sign of q,
    int8 product G = J.S on the matrix cores, per-replica reduction and
    finalisation), per call; 2 N^2 R int8 operations of algorithmic work."""
    import torch
    e = torch.empty(r, dtype=torch.int32, device="cuda:0")
    for _ in range(5):
        si.spring_ising_energy(model.ctx, e, None)
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record(stream)
    for _ in range(calls):
        si.spring_ising_energy(model.ctx, e, None)
    b.record(stream)
    torch.cuda.synchronize()
    us = 1000.0 * a.elapsed_time(b) / calls
    tops = 2.0 * n * n * r / (us * 1e-6) / 1e12
    return {"us_per_call": us, "calls": calls, "int8_tops_incl_sign_and_finalize": tops,
            "frac_of_int8_peak": tops / PEAK_INT8_MFMA_TOPS}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=3)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-forms", action="store_true", help="skip the precision-form lines")
    ap.add_argument("--no-batched", action="store_true", help="skip the batched-form timing")
    ap.add_argument("--batched-steps", type=int, default=300, help=argparse.SUPPRESS)
    ap.add_argument("--no-sequential", action="store_true", help=argparse.SUPPRESS)
    ap.add_argument("--no-batched-ttt", action="store_true", help=argparse.SUPPRESS)
    ap.add_argument("--no-differentiation", action="store_true", help=argparse.SUPPRESS)
    ap.add_argument("--iters", type=int, default=ITERS, help=argparse.SUPPRESS)
    # other shapes, for profiling the precision configurations (not bench lines)
    ap.add_argument("--n", type=int, default=N, help=argparse.SUPPRESS)
    ap.add_argument("--replicas", type=int, default=R, help=argparse.SUPPRESS)
    ap.add_argument("--couplings", default="pm1", choices=["pm1", "gauss"], help=argparse.SUPPRESS)
    ap.add_argument("--tile", type=int, default=0, help="step-kernel tile id (0 = automatic)")
    ap.add_argument("--precision", default="fp32", help="fp32 | bf16x_fp8j | bf16x_bf16j | "
                    "bf16x_hiloj | bf16x3_exactj (the headline line is fp32)")
    ap.add_argument("--energy-calls", type=int, default=200, help=argparse.SUPPRESS)
    ap.add_argument("--calib-copy-mb", type=int, default=0,
                    help="first run one elementwise kernel reading and writing this many MiB "
                         "(calibration of the HBM byte counters)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (asked for --gpus {args.gpus}); the replica-"
              "parallel path has no cross-GPU step to measure here.", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch

    from paper_2305_07187_amd import instances
    from paper_2305_07187_amd import spring_ising as si

    if not os.path.exists(si.LIB_PATH):
        from paper_2305_07187_amd import build
        build.build(verbose=False)
    si.load_library()
    dev = torch.device("cuda:0")
    iters = args.iters
    if args.calib_copy_mb:
        # one elementwise kernel that reads and writes calib_copy_mb MiB each
        src = torch.ones(args.calib_copy_mb * 262144, dtype=torch.float32, device=dev)
        dst = torch.empty_like(src)
        torch.mul(src, 2.0, out=dst)
        torch.cuda.synchronize()
        del src, dst
    n, r = args.n, args.replicas
    J = instances.make_J_torch(n, args.couplings, 0, device=dev)
    x0 = instances.make_x0_torch(n, r, 0, device=dev)
    stream = torch.cuda.current_stream()
    W = float(-torch.triu(J.double(), 1).sum())

    model = si.SpringIsing(J, x0, total_steps=iters, tile=args.tile, precision=args.precision)
    info = model.info()
    kind = ("K2000-shaped +-1" if (n, args.couplings) == (2000, "pm1")
            else {"pm1": "+-1", "gauss": "Gaussian N(0,1)"}[args.couplings])
    elapsed, kernel_us, energies = timed_runs(model, x0, iters, args.steps, args.warmup, stream)
    e = energies.cpu().numpy().astype(np.float64)
    cuts = (W - e) / 2
    flops = 2.0 * n * n * r
    achieved = flops / (kernel_us * 1e-6) / 1e12
    value = n * r * iters * args.steps / elapsed
    fp32_line = args.precision == "fp32"
    peak = PEAK_FP32_MFMA_TFLOPS if fp32_line else PEAK_BF16_MFMA_TFLOPS
    # the fixed-point form of the FP32 step runs several int8 products per
    # coupling product (four, with each position in four base-256 digits; ten,
    # with the couplings in digits as well), so that fraction of the int8 rate
    # is what it can reach in terms of the product's flop
    fixed_point = re.match(r"step_i8x(\d+)_", info["kernel_name"])
    if fixed_point:
        peak = PEAK_INT8_MFMA_TOPS / int(fixed_point.group(1))
    out = {
        "metric": f"spin-updates/s (N*R*steps/s) at N={n}",
        "value": value,
        "unit": "spin-updates/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": 1000.0 * elapsed / args.steps,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32" if fp32_line else "bf16",
        "data": "synthetic",
        "config": {"workload": f"{kind} complete graph, N={n}, R={r} replicas, "
                               f"{iters} iterations, paper linear zeta schedule, "
                               f"{args.precision}",
                   "n": n, "replicas": r, "iterations": iters, "precision": args.precision,
                   "product": ({"4": "fixed point: FP32 positions as 32-bit integers in four int8 "
                                     "digits, exact int32 sums, rounded to FP32 in two halves",
                                "10": "fixed point: FP32 positions and couplings as 32-bit "
                                      "integers in four int8 digits, ten of sixteen digit "
                                      "products, int32 sums"}[fixed_point.group(1)] if fixed_point
                               else "floating point"),
                   "kernel": info["kernel_name"]},
        "roofline": {"bound": "mfma", "achieved": achieved, "peak": peak, "unit": "TFLOP/s",
                     "frac": achieved / peak,
                     "traffic": {**MEASURED_TRAFFIC_BYTES, **FIXED_POINT_TRAFFIC_BYTES}.get(
                         (info["kernel_name"], args.precision, n, r)),
                     "traffic_unit": "bytes per launch",
                     "kernel": info["kernel_name"], "avg_launch_us": kernel_us,
                     "algorithmic_flop_per_launch": flops},
        "result": {"best_cut": float(cuts.max()), "mean_cut": float(cuts.mean()),
                   "best_energy": float(e.min()), "mean_energy": float(e.mean())},
    }

    if bool(info["j_integer"]) and args.energy_calls > 0:
        out["energy_readout"] = energy_readout(si, model, n, r, args.energy_calls, stream)

    if fp32_line and not args.no_forms:
        # the same workload with the positions' wall at |q| = 1 instead of sqrt 2
        m1 = si.SpringIsing(J, x0, total_steps=iters, precision="fp32", qmax=1.0)
        m1.run(iters)
        e1 = m1.energy(exact=bool(m1.info()["j_integer"])).cpu().numpy().astype(np.float64)
        m1.close()
        c1 = (W - e1) / 2
        out["result_qmax1"] = {"best_cut": float(c1.max()), "mean_cut": float(c1.mean()),
                               "best_energy": float(e1.min()), "mean_energy": float(e1.mean())}

    if fp32_line and not args.no_forms and iters % CHECK_EVERY == 0 and args.couplings == "pm1":
        out["time_to_target"] = time_to_target(si, J, n, r, iters, CHECK_EVERY, stream,
                                               runs_per_form=max(1, min(args.steps, 5)))
    model.close()
    if fp32_line and not args.no_forms and (n, r, args.couplings) == (N, R, "pm1"):
        out["precision_full_configurations"] = precision_full_configurations(si)
        out["precision_full_configurations"]["time_to_target"] = precision_time_to_target(si)
    if fp32_line and not args.no_batched and (n, r, args.couplings) == (N, R, "pm1"):
        out["batched_form"] = batched_form(si, steps=args.batched_steps,
                                           sequential=not args.no_sequential,
                                           time_to_target=not args.no_batched_ttt)
        if not args.no_differentiation:
            out["differentiation_form"] = differentiation_form(si)
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline()
    print(json.dumps(out))


if __name__ == "__main__":
    main()
