#!/usr/bin/env python3
"""Throughput of simultaneous local upscaling on one MI355X.

One step is one pass of the plain hot path over one batch of synthetic
samples, with the random variables xi already resident in HBM:

  1. coefficient samples a(x, xi) on the fine grid       (stomsfem_coef_bumps)
  2. local upscaling S_K(xi) for every (element, sample)  (stomsfem_upscale)
  3. coarse solve S U = b per sample, Monte Carlo mean   (stomsfem_coarse_solve)

Default workload: 32 x 32 coarse elements, H/h = 32 (1024 x 1024 fine Q1
grid), 4096 samples (4,194,304 element-sample pairs), FP64.  The metric is
upscaled (element x sample) pairs per second for the whole step.

Prints one JSON line with a roofline entry for the dominant kernel (the local
upscaling, timed with HIP events on the stream it runs on) and a CPU baseline
(the FP64 oracle on the host cores, on a bounded sample of the same workload).
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

FP64_VALU_PEAK_TFLOPS = 78.6   # MI355X: 256 CUs x 2.4 GHz x 128 FP64 flop/clk
HBM_PEAK_GBS = 8000.0


def plain_flops_per_pair(m: int) -> float:
    """FP64 operations of the sliding-window LDL^T Schur-complement algorithm
    for one (element, sample) pair (an FMA counts 2): per pivot j with c
    active rows below it, the rank-1 window update c(c+1)/2 FMA, the column
    scaling c mul + 1 div, the 3-rhs forward step 3c FMA and the y y^T/d
    accumulation 9 ops; plus 20 ops per interior row for assembling the
    9-point stencil row and its Dirichlet lifts, and 12 per boundary element
    for g.K_BB g'."""
    n = m - 1
    NI = n * n
    f = 0.0
    for j in range(NI):
        c = min(m, NI - 1 - j)
        f += c * (c + 1) + c + 1 + 6 * c + 9
    f += 20 * NI + 12 * max(4 * (m - 1), 1)
    return f


def survey_flops_per_pair(m: int) -> float:
    """The coarser count of the plain direct path per pair used for the
    scope table's roofline estimate: banded factor n_I (b^2 + 2b), 3-rhs
    solves 12 n_I b, band assembly 32 m^2, S 250 m (n_I = (m-1)^2, b = m)."""
    nI, b = (m - 1) ** 2, m
    return nI * (b * b + 2 * b) + 12 * nI * b + 32 * m * m + 250 * m


def kernel_source_sha1(name: str) -> str:
    """sha1 of a kernel's source file and of the headers beside it that it
    includes, directly or not, in the order in which they are first met."""
    import hashlib
    import re

    csrc = os.path.join(ROOT, "paper_1607_00693_amd", "csrc")
    digest, todo, seen = hashlib.sha1(), [name], {name}
    while todo:
        text = open(os.path.join(csrc, todo.pop(0)), "rb").read()
        digest.update(text)
        for inc in re.findall(rb'^#include "([^"]+)"', text, re.M):
            inc = inc.decode()
            if inc not in seen and os.path.exists(os.path.join(csrc, inc)):
                seen.add(inc)
                todo.append(inc)
    return digest.hexdigest()


def profiled_traffic_per_pair():
    """Calibrated HBM bytes per pair of the m = 32 upscaling kernel from the
    committed counter summary, or None when the kernel's source or a header of
    it has changed since the counters were taken."""
    prof = os.path.join(ROOT, "profiles", "upscale_mesh32_hbm_traffic.md")
    try:
        vals = dict(line.split(": ", 1) for line in open(prof).read().splitlines() if ": " in line
                    and line.split(": ", 1)[0] in ("traffic_bytes_per_pair", "kernel_source_sha1"))
        if kernel_source_sha1("upscale_rows.hip") != vals["kernel_source_sha1"].strip():
            return None
        return float(vals["traffic_bytes_per_pair"])
    except (OSError, KeyError, ValueError):
        return None


def _cpu_model() -> str:
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def cpu_baseline(wl, budget_s: float = 25.0):
    import numpy as np

    import oracle
    from paper_1607_00693_amd import workloads as W

    threads = os.cpu_count() or 1
    if os.environ.get("OMP_NUM_THREADS", "").isdigit():
        threads = min(threads, int(os.environ["OMP_NUM_THREADS"]))
    nprobe = 2
    xi = W.uniform_xi(wl.nsamples, wl.nxi, wl.seed)

    def run(ns):
        t0 = time.perf_counter()
        a = oracle.coef_bumps(xi[:ns], wl.nfine, **wl.coef_params(), nthreads=threads)
        S, _, _ = oracle.upscale(a, wl.nc, wl.nc, wl.m, nthreads=threads)
        oracle.coarse_solve(S, wl.nc, wl.nc, nthreads=threads)
        return time.perf_counter() - t0

    t = run(nprobe)
    ns = int(max(nprobe, min(wl.nsamples, nprobe * budget_s / max(t, 1e-6))))
    t = run(ns)
    pairs = ns * wl.M
    return {
        "value": pairs / t,
        "unit": "pairs/s",
        "cores": threads,
        "kind": "oracle",
        "sample": f"first {ns} of {wl.nsamples} samples ({pairs} element-sample pairs): coefficient "
                  f"generation + upscaling + coarse solve, OpenMP over pairs, {t:.1f} s",
        "cpu_model": _cpu_model(),
        "build": "gcc -O3 -march=x86-64-v3 -fopenmp",
    }


def _timed(fn, reps=5):
    import torch

    fn()
    torch.cuda.synchronize()
    t = time.perf_counter()
    for _ in range(reps):
        fn()
    torch.cuda.synchronize()
    return (time.perf_counter() - t) / reps


def measure_interpolation(wl, xi, S_plain, t_plain_ms, nn_list, log, sg_levels=()):
    """Random interpolation (Sec. 3.1) on the benchmark mesh: offline node
    solves, then the online evaluation from xi, against the plain path from xi
    (coefficient generation + upscaling, t_plain_ms).  Reports throughput,
    ratio, the largest error of S relative to max|S| per pair, and the worst
    per-sample relative error of the coarse solution; tensor grids of nn
    nodes per variable, and Smolyak sparse grids of the given levels."""
    import numpy as np
    import torch

    from paper_1607_00693_amd import stomsfem as sm

    fam = sm.bump_family(wl)
    lv, nl = sm.local_vars_bumps(wl.nc, wl.nc, wl.m, fam)
    N = xi.shape[0]
    pairs = N * wl.M
    U_pl, _, _ = sm.coarse_solve(S_plain, wl.nc, wl.nc)
    out = {}
    for nn in nn_list:
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        model = sm.interp_build(wl.nc, wl.nc, wl.m, lv, fam, nn)
        t_off = time.perf_counter() - t0
        S_ri = torch.empty_like(S_plain)
        t_on = _timed(lambda: sm.interp_apply(model, xi, S=S_ri))
        scale = S_plain.abs().amax(dim=2, keepdim=True)
        s_err = float(((S_ri - S_plain).abs() / scale).max())
        U_ri, _, _ = sm.coarse_solve(S_ri, wl.nc, wl.nc)
        u_err = float((torch.linalg.norm(U_ri - U_pl, dim=1) / torch.linalg.norm(U_pl, dim=1)).max())
        rows = int(model.export("offsets")[-1])
        out[f"nodes_{nn}"] = {
            "offline_s": t_off, "node_solves": rows, "table_MB": rows * 80 / 1e6,
            "pairs_per_s": pairs / t_on, "plain_pairs_per_s": pairs / (t_plain_ms * 1e-3),
            "ratio": t_plain_ms * 1e-3 / t_on,
            "flops_per_pair": float(np.mean(20.0 * nn ** nl.astype(np.float64))),
            "max_S_rel_err": s_err, "max_coarse_rel_err": u_err}
        log(f"interpolation nn={nn}: {out[f'nodes_{nn}']}")
        model.free()
        del S_ri
    for level in sg_levels:
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        model = sm.sgi_build(wl.nc, wl.nc, wl.m, lv, fam, level)
        t_off = time.perf_counter() - t0
        S_sg = torch.empty_like(S_plain)
        t_on = _timed(lambda: sm.sgi_apply(model, xi, S=S_sg), reps=3)
        scale = S_plain.abs().amax(dim=2, keepdim=True)
        s_err = float(((S_sg - S_plain).abs() / scale).max())
        U_sg, _, _ = sm.coarse_solve(S_sg, wl.nc, wl.nc)
        u_err = float((torch.linalg.norm(U_sg - U_pl, dim=1) / torch.linalg.norm(U_pl, dim=1)).max())
        nodes = {k: (1 if k == 0 else len(sm.sparse_grid(k, level)[1])) for k in set(nl.tolist())}
        out[f"sparse_level_{level}"] = {
            "offline_s": t_off, "node_solves": int(sum(nodes[int(k)] for k in nl)),
            "nodes_per_patch_4_vars": nodes.get(4), "pairs_per_s": pairs / t_on,
            "plain_pairs_per_s": pairs / (t_plain_ms * 1e-3), "ratio": t_plain_ms * 1e-3 / t_on,
            "max_S_rel_err": s_err, "max_coarse_rel_err": u_err}
        log(f"sparse-grid interpolation level={level}: {out[f'sparse_level_{level}']}")
        model.free()
        del S_sg
    return out


def measure_coarse(log, meshes=(64, 48, 33), nsamples=256, reps=10):
    """Batched FP64 coarse solve + QoI (eq. upscaleSUF, Sec. 4.1.1) alone on
    the coarse meshes the blocked kernel serves, at the channels workload's
    batch size: upscaled stiffness of a seeded log-normal medium at H/h = 4
    (the solve does not depend on H/h), HIP-event time per batch on the
    launching stream, algorithmic FP64 flops per sample nU (B^2 + 4B) for the
    banded LDL^T with forward substitution plus 2 nU B for the backward pass."""
    import torch

    from paper_1607_00693_amd import stomsfem as sm
    from paper_1607_00693_amd import workloads as W

    out = {}
    stream = torch.cuda.current_stream()
    for nc in meshes:
        a = torch.from_numpy(W.lognormal_field((nsamples, nc * 4, nc * 4), 1.0, 5)).cuda()
        S = sm.upscale(a, nc, nc, 4)
        del a
        U, qm, qv = sm.coarse_solve(S, nc, nc)
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        ev[0].record(stream)
        for _ in range(reps):
            sm.coarse_solve(S, nc, nc, U=U, qoi_mean=qm, qoi_var=qv)
        ev[1].record(stream)
        ev[1].synchronize()
        ms = ev[0].elapsed_time(ev[1]) / reps
        nU, B = (nc - 1) ** 2, nc
        flops = nU * (B * B + 4 * B) + 2 * nU * B
        out[f"{nc}x{nc}"] = {"samples": nsamples, "ms_per_batch": ms, "samples_per_s": nsamples / (ms * 1e-3),
                             "flops_per_sample": flops,
                             "fp64_frac": flops * nsamples / (ms * 1e-3) / 1e12 / FP64_VALU_PEAK_TFLOPS}
        del S, U
    log(f"coarse solve: {out}")
    return out


def measure_queue(log, reps=3):
    """One round of the channels workload's upscaling: a batch of 256 samples
    at each H/h in {8, 16, 32} on the 64 x 64 coarse mesh (FP32 coefficients,
    generated beforehand, FP64 solves), upscaled (a) by the per-m kernels one
    after the other on one stream, (b) by the per-m kernels on three streams at
    once (as the plan's graph branches run them), (c) by the one persistent
    launch over all three batches (stomsfem_upscale_queue); each batch also
    alone through its per-m kernel and through the persistent kernel.  S of
    (c) is compared bit for bit with (a)."""
    import numpy as np
    import torch

    from paper_1607_00693_amd import stomsfem as sm
    from paper_1607_00693_amd import workloads as W

    wl = W.CHANNELS64
    dev = "cuda"
    kind, x0, y0, size = W.channel_geometry(wl)
    g = [torch.from_numpy(np.ascontiguousarray(v)).to(dev) for v in (kind, x0, y0, size)]
    N = wl.batch
    xi = torch.from_numpy(W.normal_xi(3 * N, wl.nxi, wl.xi_seed)).to(dev)
    bt = {}
    for i, m in enumerate((8, 16, 32)):
        fm = sm.feature_map(wl.nc * m, *g)
        a = sm.coef_features(fm, wl.nxi, xi[i * N:(i + 1) * N].contiguous(), wl.decades, dtype=torch.float32)
        S = torch.empty((N, wl.M, 10), dtype=torch.float64, device=dev)
        st = torch.empty((N, wl.M), dtype=torch.int32, device=dev)
        bt[m] = (a, S, st, sm.make_batch(a, wl.nc, wl.nc, m, S, st))
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)

    def ev(f):
        f()
        torch.cuda.synchronize()
        e0.record()
        for _ in range(reps):
            f()
        e1.record()
        e1.synchronize()
        return e0.elapsed_time(e1) / reps

    allb = [bt[m][3] for m in (8, 16, 32)]
    alone = {}
    for m in (8, 16, 32):
        alone[str(m)] = {"per_m_kernel_ms": ev(lambda: sm.upscale_batches([bt[m][3]])),
                         "persistent_kernel_ms": ev(lambda: sm.upscale_queue([bt[m][3]]))}
    streams = [torch.cuda.Stream() for _ in range(3)]

    def concurrent():
        cur = torch.cuda.current_stream()
        start = torch.cuda.Event()
        start.record(cur)
        for s_, b in zip(streams, allb):
            s_.wait_event(start)
            sm.upscale_batches([b], stream=s_)
        for s_ in streams:
            cur.wait_stream(s_)

    t_seq = ev(lambda: sm.upscale_batches(allb))
    t_conc = ev(concurrent)
    t_q = ev(lambda: sm.upscale_queue(allb))
    sm.upscale_batches(allb)
    torch.cuda.synchronize()
    ref = {m: bt[m][1].clone() for m in (8, 16, 32)}
    sm.upscale_queue(allb)
    torch.cuda.synchronize()
    same = all(torch.equal(ref[m], bt[m][1]) for m in (8, 16, 32))
    pairs = 3 * N * wl.M
    out = {"workload": f"one round of the channels workload: 64x64 coarse, {N} samples at each H/h in {{8, 16, 32}}, "
                       "FP32 coefficients generated beforehand, FP64 solves; upscaling only",
           "sequential_ms": t_seq, "concurrent_streams_ms": t_conc, "persistent_queue_ms": t_q,
           "persistent_over_concurrent": t_q / t_conc, "pairs_per_s_concurrent": pairs / (t_conc * 1e-3),
           "pairs_per_s_persistent": pairs / (t_q * 1e-3), "each_batch_alone": alone,
           "persistent_bitwise_equal": bool(same)}
    log(f"mixed-H/h launches: {out}")
    return out


def measure_channels(log, reps=3):
    """High-contrast channels-and-inclusions workload: 64 x 64 coarse mesh,
    32 batches of 256 samples with H/h drawn per batch from {8, 16, 32}, FP32
    coefficient storage, FP64 solves.  All batches are captured into one
    execution plan (HIP graphs; batches of different H/h run as concurrent
    branches).  Reports the latency of each batch replayed alone (submit to
    QoI ready: p50/p99 over reps x 32 batches, also per H/h) and the
    throughput of whole-plan replays."""
    import numpy as np
    import torch

    from paper_1607_00693_amd import stomsfem as sm
    from paper_1607_00693_amd import workloads as W

    wl = W.CHANNELS64
    dev = "cuda"
    kind, x0, y0, size = W.channel_geometry(wl)
    g = [torch.from_numpy(np.ascontiguousarray(v)).to(dev) for v in (kind, x0, y0, size)]
    ms = W.batch_m(wl)
    fmaps = {int(m): sm.feature_map(wl.nc * int(m), *g) for m in sorted(set(ms.tolist()))}
    xi_all = torch.from_numpy(W.normal_xi(wl.nbatch * wl.batch, wl.nxi, wl.xi_seed)).to(dev)
    nU = (wl.nc - 1) ** 2
    keep, stages = [], []
    for b in range(wl.nbatch):
        xi = xi_all[b * wl.batch:(b + 1) * wl.batch]
        qm = torch.empty(nU, dtype=torch.float64, device=dev)
        qv = torch.empty(nU, dtype=torch.float64, device=dev)
        st = torch.empty((wl.batch, wl.M), dtype=torch.int32, device=dev)
        keep.append((xi, qm, qv, st))
        stages.append(sm.make_stage(wl.nc, int(ms[b]), xi, feature_map=fmaps[int(ms[b])], nfeat=wl.nxi,
                                    decades=wl.decades, a_dtype=torch.float32, qoi_mean=qm, qoi_var=qv, status=st))
    plan = sm.plan_create(stages)
    stream = torch.cuda.current_stream()
    plan.launch(-1, stream)
    torch.cuda.synchronize()
    lat = {int(m): [] for m in fmaps}
    ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    for r in range(reps):
        for b in range(wl.nbatch):
            ev0.record(stream)
            plan.launch(b, stream)
            ev1.record(stream)
            ev1.synchronize()
            lat[int(ms[b])].append(ev0.elapsed_time(ev1))
        log(f"channels: latency rep {r} done")
    bad = sum(int((st != 0).sum().item()) for (_, _, _, st) in keep)
    t_all = []
    for r in range(reps):
        ev0.record(stream)
        plan.launch(-1, stream)
        ev1.record(stream)
        ev1.synchronize()
        t_all.append(ev0.elapsed_time(ev1))
    plan.free()
    allv = np.concatenate([np.asarray(v) for v in lat.values()])
    pairs = wl.nbatch * wl.batch * wl.M
    out = {
        "workload": f"64x64 coarse, {wl.nbatch} batches x {wl.batch} samples, H/h per batch from {{8,16,32}} "
                    f"(counts {({int(k): int(v) for k, v in zip(*np.unique(ms, return_counts=True))})}), 40 channels + 40 squares, "
                    f"xi~N(0,1)^80, contrast up to 1e4, FP32 a, FP64 solves",
        "batch_latency_ms": {"p50": float(np.percentile(allv, 50)), "p99": float(np.percentile(allv, 99)),
                             "samples": int(allv.size)},
        "batch_latency_ms_by_m": {str(m): {"p50": float(np.percentile(v, 50)), "p99": float(np.percentile(v, 99))}
                                  for m, v in lat.items()},
        "whole_plan_ms": float(np.median(t_all)),
        "pairs_per_s": pairs / (np.median(t_all) * 1e-3),
        "serial_sum_ms": float(sum(np.median(v) * len(v) / reps for v in lat.values())),
        "non_ok_pairs": bad,
    }
    out["batch_latency_ms_by_m"] = {k: v for k, v in sorted(out["batch_latency_ms_by_m"].items(), key=lambda kv: int(kv[0]))}
    log(f"channels: {out}")
    out["_latencies_by_m"] = {str(m): v for m, v in lat.items()}
    return out


def measure_channels_surrogate(log, plain=None, ntrain=2048, schedule=((8000, 2e-3), (8000, 5e-4), (8000, 1e-4)),
                               reps=3, tau=3e-4):
    """Learned surrogate on the channels-and-inclusions workload (64 x 64
    coarse mesh, 32 batches of 256 samples, H/h per batch from {8, 16, 32}):
    one network per patch and per H/h, trained on ntrain plain solves of that
    medium (FP64 coefficients); then, per batch, the gated BF16 surrogate with
    the plain fallback (coefficient blocks of the listed pairs regenerated from
    the feature map) followed by the FP64 coarse solve and the QoI.  Reports
    the per-batch latency (submit to QoI ready, p50/p99 over reps x 32
    batches, also per H/h), acceptance, and the coarse-solution error of every
    sample against the plain FP64 path; plain = the per-H/h latencies of the
    plain plan when given, from which a per-H/h policy (the surrogate only
    where its p50 beats the plain batch) is also reported.  Gate tolerance
    tau = 3e-4 here: at 1e-3 the largest coarse error over the 8192 samples
    reaches about 1.5e-3 (the two heads share their hidden layers, so their
    disagreement understates the error of the high-contrast patches)."""
    import numpy as np
    import torch

    from paper_1607_00693_amd import stomsfem as sm
    from paper_1607_00693_amd import workloads as W

    wl = W.CHANNELS64
    dev = "cuda"
    nc = wl.nc
    kind, x0, y0, size = W.channel_geometry(wl)
    g = [torch.from_numpy(np.ascontiguousarray(v)).to(dev) for v in (kind, x0, y0, size)]
    ms = W.batch_m(wl)
    xi_all = torch.from_numpy(W.normal_xi(wl.nbatch * wl.batch, wl.nxi, wl.xi_seed)).to(dev)
    models, fmaps, train = {}, {}, {}
    for m in sorted(set(int(v) for v in ms)):
        fmap = sm.feature_map(nc * m, *g)
        fmaps[m] = fmap
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        xi_tr = torch.from_numpy(W.normal_xi(ntrain, wl.nxi, 2005 + m)).to(dev)
        S_tr = torch.empty((ntrain, wl.M, 10), dtype=torch.float64, device=dev)
        for c0 in range(0, ntrain, 256):
            a = sm.coef_features(fmap, wl.nxi, xi_tr[c0:c0 + 256], wl.decades)
            sm.upscale(a, nc, nc, m, S=S_tr[c0:c0 + 256])
            del a
        torch.cuda.synchronize()
        t_data = time.perf_counter() - t0
        mdl = sm.mlp_create_features(nc, m, fmap, wl.nxi, wl.decades, W.mlp_init(wl.M, 4005 + m), 3.0)
        sm.mlp_set_data(mdl, xi_tr, S_tr)
        perm = torch.from_numpy(W.permutation(ntrain, 5005 + m)).to(dev)
        t0 = time.perf_counter()
        for steps, lr in schedule:
            sm.mlp_train(mdl, steps, lr, perm)
        torch.cuda.synchronize()
        train[m] = {"training_data_s": t_data, "train_s": time.perf_counter() - t0}
        models[m] = mdl
        del S_tr, xi_tr
        log(f"channels surrogate: H/h={m} model trained ({train[m]})")
    nU = (nc - 1) ** 2
    stream = torch.cuda.current_stream()
    bufs = []
    for b in range(wl.nbatch):
        bufs.append(dict(S=torch.empty((wl.batch, wl.M, 10), dtype=torch.float64, device=dev),
                         st=torch.empty((wl.batch, wl.M), dtype=torch.int32, device=dev),
                         U=torch.empty((wl.batch, nU), dtype=torch.float64, device=dev),
                         qm=torch.empty(nU, dtype=torch.float64, device=dev),
                         qv=torch.empty(nU, dtype=torch.float64, device=dev)))

    def run(b):
        xi = xi_all[b * wl.batch:(b + 1) * wl.batch]
        o = bufs[b]
        sm.upscale_surrogate(models[int(ms[b])], xi, tau, sm.PREC_BF16, S=o["S"], status=o["st"])
        sm.coarse_solve(o["S"], nc, nc, U=o["U"], qoi_mean=o["qm"], qoi_var=o["qv"])

    for b in range(wl.nbatch):
        run(b)
    torch.cuda.synchronize()
    lat = {int(m): [] for m in models}
    ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    for r in range(reps):
        for b in range(wl.nbatch):
            ev0.record(stream)
            run(b)
            ev1.record(stream)
            ev1.synchronize()
            lat[int(ms[b])].append(ev0.elapsed_time(ev1))
        log(f"channels surrogate: latency rep {r} done")
    # accuracy of every sample against the plain FP64 path (not timed)
    acc_n = fb_n = au_n = 0
    u_err = 0.0
    u_err_m = {int(m): 0.0 for m in models}
    for b in range(wl.nbatch):
        m = int(ms[b])
        xi = xi_all[b * wl.batch:(b + 1) * wl.batch]
        a = sm.coef_features(fmaps[m], wl.nxi, xi, wl.decades)
        S_p = sm.upscale(a, nc, nc, m)
        del a
        U_p, _, _ = sm.coarse_solve(S_p, nc, nc)
        o = bufs[b]
        e = float((torch.linalg.norm(o["U"] - U_p, dim=1) / torch.linalg.norm(U_p, dim=1)).max())
        u_err = max(u_err, e)
        u_err_m[m] = max(u_err_m[m], e)
        st = o["st"]
        acc_n += int((st == 0).sum())
        fb_n += int((st == 1).sum())
        au_n += int((st == 2).sum())
        del S_p, U_p
    for mdl in models.values():
        mdl.free()
    allv = np.concatenate([np.asarray(v) for v in lat.values()])
    pairs = wl.nbatch * wl.batch * wl.M
    tot = acc_n + fb_n + au_n
    serial_ms = float(sum(np.median(v) * len(v) / reps for v in lat.values()))
    out = {
        "workload": f"64x64 coarse, {wl.nbatch} batches x {wl.batch} samples, H/h per batch from {{8,16,32}}, "
                    f"40 channels + 40 squares, xi~N(0,1)^80; one network per patch and H/h (k<=4 -> 64x3 -> 2x10, "
                    f"GELU), {ntrain} training samples, {sum(s for s, _ in schedule)} Adam steps; per batch: gated "
                    f"BF16 surrogate (tau={tau:g}, box [-3,3]) + plain fallback + FP64 coarse solve + QoI",
        "training": {str(m): v for m, v in train.items()},
        "batch_latency_ms": {"p50": float(np.percentile(allv, 50)), "p99": float(np.percentile(allv, 99)),
                             "samples": int(allv.size)},
        "batch_latency_ms_by_m": {str(m): {"p50": float(np.percentile(v, 50)), "p99": float(np.percentile(v, 99))}
                                  for m, v in sorted(lat.items())},
        "serial_sum_ms": serial_ms,
        "pairs_per_s": pairs / (serial_ms * 1e-3),
        "accepted": acc_n / tot, "fallback": fb_n / tot, "audited": au_n / tot,
        "max_coarse_rel_err": u_err,
        "max_coarse_rel_err_by_m": {str(m): v for m, v in sorted(u_err_m.items())},
    }
    if plain:
        pm = plain["batch_latency_ms_by_m"]
        out["p50_ratio_plain_over_surrogate_by_m"] = {
            k: pm[k]["p50"] / v["p50"] for k, v in out["batch_latency_ms_by_m"].items() if k in pm}
        out["serial_ratio_plain_over_surrogate"] = plain["serial_sum_ms"] / serial_ms
        # policy: per H/h the faster of the two paths (by p50)
        use = {m: out["batch_latency_ms_by_m"][str(m)]["p50"] < pm[str(m)]["p50"] for m in lat if str(m) in pm}
        plat = plain.get("_latencies_by_m", {})
        if plat and all(str(m) in plat for m in lat):
            pol = np.concatenate([np.asarray(lat[m]) if use[m] else np.asarray(plat[str(m)]) for m in lat])
            pol_serial = sum(np.median(lat[m] if use[m] else plat[str(m)]) * len(lat[m]) / reps for m in lat)
            out["policy"] = {"surrogate_at": sorted(int(m) for m in use if use[m]),
                             "batch_latency_ms": {"p50": float(np.percentile(pol, 50)),
                                                  "p99": float(np.percentile(pol, 99))},
                             "serial_sum_ms": float(pol_serial),
                             "serial_ratio_plain_over_policy": plain["serial_sum_ms"] / pol_serial}
    log(f"channels surrogate: {out}")
    return out


def measure_surrogate(wl, xi, S_plain, t_plain_ms, log, ntrain=2048, schedule=((8000, 2e-3), (8000, 5e-4),
                                                                           (8000, 1e-4))):
    """Learned surrogate on the benchmark mesh: one MLP per patch trained on
    ntrain plain solves (seed 2000 + workload), then gated BF16 inference with
    the plain fallback on the benchmark's own xi, against the plain path from
    xi (coefficient generation + upscaling, t_plain_ms)."""
    import torch

    from paper_1607_00693_amd import stomsfem as sm
    from paper_1607_00693_amd import workloads as W

    fam = sm.bump_family(wl)
    lv, nl = sm.local_vars_bumps(wl.nc, wl.nc, wl.m, fam)
    mdl = sm.mlp_create(wl.nc, wl.nc, wl.m, lv, W.mlp_init(wl.M, 4000 + wl.seed % 1000), fam, 1.0)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    xi_tr = torch.from_numpy(W.uniform_xi(ntrain, wl.nxi, 2000 + wl.seed % 1000)).cuda()
    S_tr = torch.empty((ntrain, wl.M, 10), dtype=torch.float64, device="cuda")
    chunk = 256
    for c0 in range(0, ntrain, chunk):  # training data from the plain path, in chunks
        a_tr = sm.coef_bumps(xi_tr[c0:c0 + chunk], wl.nfine, **wl.coef_params())
        sm.upscale(a_tr, wl.nc, wl.nc, wl.m, S=S_tr[c0:c0 + chunk])
        del a_tr
    torch.cuda.synchronize()
    t_data = time.perf_counter() - t0
    sm.mlp_set_data(mdl, xi_tr, S_tr)
    perm = torch.from_numpy(W.permutation(ntrain, 5000 + wl.seed % 1000)).cuda()
    t0 = time.perf_counter()
    for steps, lr in schedule:
        sm.mlp_train(mdl, steps, lr, perm)
    torch.cuda.synchronize()
    t_train = time.perf_counter() - t0
    N = xi.shape[0]
    S_su = torch.empty_like(S_plain)
    status = torch.empty((N, wl.M), dtype=torch.int32, device="cuda")
    t_su = _timed(lambda: sm.upscale_surrogate(mdl, xi, 1e-3, sm.PREC_BF16, S=S_su, status=status), reps=3)
    st = status.cpu()
    U_p, _, _ = sm.coarse_solve(S_plain, wl.nc, wl.nc)
    U_s, _, _ = sm.coarse_solve(S_su, wl.nc, wl.nc)
    u_err = float((torch.linalg.norm(U_s - U_p, dim=1) / torch.linalg.norm(U_p, dim=1)).max())
    # the FP16 single-term kernel on the same networks and samples
    t_h = _timed(lambda: sm.upscale_surrogate(mdl, xi, 1e-3, sm.PREC_F16, S=S_su, status=status), reps=3)
    sth = status.cpu()
    U_h, _, _ = sm.coarse_solve(S_su, wl.nc, wl.nc)
    f16 = {"pairs_per_s": N * wl.M / t_h, "ratio": t_plain_ms * 1e-3 / t_h,
           "accepted": float((sth == 0).float().mean()), "fallback": float((sth == 1).float().mean()),
           "audited": float((sth == 2).float().mean()),
           "max_coarse_rel_err": float((torch.linalg.norm(U_h - U_p, dim=1) / torch.linalg.norm(U_p, dim=1)).max())}
    pairs = N * wl.M
    out = {"workload": f"{wl.nc}x{wl.nc} coarse, H/h={wl.m}, {wl.M} per-patch MLPs (k<=4 -> 64x3 -> 2x10, GELU), "
                       f"{ntrain} training samples/patch, {sum(s for s, _ in schedule)} Adam steps, the benchmark's "
                       f"{N} samples, gate tau=1e-3, BF16 MFMA (3-term split); plain side = generation + upscaling",
           "training_data_s": t_data, "train_s": t_train,
           "pairs_per_s": pairs / t_su, "plain_pairs_per_s": pairs / (t_plain_ms * 1e-3),
           "ratio": t_plain_ms * 1e-3 / t_su,
           "accepted": float((st == 0).float().mean()), "fallback": float((st == 1).float().mean()),
           "audited": float((st == 2).float().mean()), "max_coarse_rel_err": u_err, "fp16_single_term": f16}
    log(f"surrogate on the benchmark mesh: {out}")
    mdl.free()
    return out


FP32_MFMA_PEAK_TFLOPS = 157.3


def measure_reduced_basis(wl, xi, S_plain, t_plain_ms, log, ntrain=40):
    """Reduced basis (Sec. 3.2, Algorithms 3 and 4) on the benchmark mesh:
    offline from ntrain plain training samples per patch (seed 2000 +
    workload; the method of snapshots, with the snapshots from the refined
    FP32/FP64 cell solver), then the FP32 matrix-core online stage on the
    benchmark's own xi with FP32 coefficients, against the plain path from xi
    (FP64 coefficient generation + upscaling, t_plain_ms)."""
    import torch

    from paper_1607_00693_amd import stomsfem as sm
    from paper_1607_00693_amd import workloads as W

    xi_tr = torch.from_numpy(W.uniform_xi(ntrain, wl.nxi, 2000 + wl.seed % 1000)).cuda()
    a_tr = sm.coef_bumps(xi_tr, wl.nfine, **wl.coef_params())
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    model = sm.reduce(a_tr, wl.nc, wl.nc, wl.m, r_max=8, tail_tol=1e-6)
    torch.cuda.synchronize()
    t_off = time.perf_counter() - t0
    del a_tr
    N = xi.shape[0]
    a32 = torch.empty((N, wl.nfine, wl.nfine), dtype=torch.float32, device="cuda")
    t_gen = _timed(lambda: sm.coef_bumps(xi, wl.nfine, **wl.coef_params(), out=a32), reps=3)
    S_rb = torch.empty_like(S_plain)
    status = torch.empty((N, wl.M), dtype=torch.int32, device="cuda")
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    sm.reduce_apply(model, a32, S=S_rb, status=status)
    reps = 5
    ev[0].record()
    for _ in range(reps):
        sm.reduce_apply(model, a32, S=S_rb, status=status)
    ev[1].record()
    ev[1].synchronize()
    t_on = ev[0].elapsed_time(ev[1]) / reps * 1e-3
    bad = int((status != 0).sum().item())
    scale = S_plain.abs().amax(dim=2, keepdim=True)
    s_err = float(((S_rb - S_plain).abs() / scale).max())
    U_p, _, _ = sm.coarse_solve(S_plain, wl.nc, wl.nc)
    U_r, _, _ = sm.coarse_solve(S_rb, wl.nc, wl.nc)
    u_err = float((torch.linalg.norm(U_r - U_p, dim=1) / torch.linalg.norm(U_p, dim=1)).max())
    # control variate (the remark closing Sec. 5.3): E[u_H] from the reduced
    # solution on all samples, corrected by the plain-minus-reduced mean on the
    # first n2 of them (the two-level formula with the coarse nodes as "fine")
    n2 = min(256, N)
    cv_mean, var_r, var_d = sm.two_level_mc(U_r, U_r[:n2].contiguous(), U_p[:n2].contiguous(), wl.nc, 1)
    plain_mean = U_p.mean(dim=0)
    cv = {"n_reduced": N, "n_plain": n2,
          "max_abs_err_vs_plain_mean": float((cv_mean - plain_mean).abs().max()),
          "max_abs_err_uncorrected": float((U_r.mean(dim=0) - plain_mean).abs().max()),
          "var_ratio_d_over_reduced": float(var_d.sum() / var_r.sum())}
    pairs = N * wl.M
    kd = ((wl.m * wl.m + 63) // 64) * 64
    flops = 2.0 * kd * 80  # the GEMM row of one pair (padded table: 80 columns)
    r = model.export("r")
    out = {"workload": f"{wl.nc}x{wl.nc} coarse, H/h={wl.m}, {ntrain} training samples/patch, r<=8 (tail 1e-6), "
                       f"the benchmark's {N} samples with FP32 coefficients, FP32 MFMA GEMM "
                       "[128 samples x m^2] x [m^2 x 80] per workgroup + FP32 8x8 solves",
           "offline_s": t_off, "modes_min": int(r.min()), "modes_max": int(r.max()),
           "online_ms": t_on * 1e3, "pairs_per_s": pairs / t_on,
           "fp32_coef_generation_ms": t_gen * 1e3, "pairs_per_s_with_generation": pairs / (t_on + t_gen),
           "plain_pairs_per_s": pairs / (t_plain_ms * 1e-3), "ratio": t_plain_ms * 1e-3 / t_on,
           "ratio_with_generation": t_plain_ms * 1e-3 / (t_on + t_gen),
           "mfma_flops_per_pair": flops, "achieved_tflops": flops * pairs / t_on / 1e12,
           "fp32_mfma_peak_frac": flops * pairs / t_on / 1e12 / FP32_MFMA_PEAK_TFLOPS,
           "non_ok_pairs": bad, "max_S_rel_err": s_err, "max_coarse_rel_err": u_err,
           "control_variate": cv}
    log(f"reduced basis on the benchmark mesh: {out}")
    model.free()
    del a32, S_rb
    torch.cuda.empty_cache()
    return out


def measure_two_level_bench(wl, S_plain, log, n_h=32):
    """Two-level Monte Carlo (Sec. 4.1.1) on the benchmark mesh: the
    benchmark's coarse solutions (N_H samples) and n_h independent samples
    (seed 1900 + workload) solved both on the coarse mesh and on the full
    fine grid by multigrid-preconditioned CG (relative residual 1e-12)."""
    import torch

    from paper_1607_00693_amd import stomsfem as sm
    from paper_1607_00693_amd import workloads as W

    xh = torch.from_numpy(W.uniform_xi(n_h, wl.nxi, 1900 + wl.seed % 1000)).cuda()
    a_h = sm.coef_bumps(xh, wl.nfine, **wl.coef_params())
    U_Hh, _, _ = sm.coarse_solve(sm.upscale(a_h, wl.nc, wl.nc, wl.m), wl.nc, wl.nc)
    U_H, _, _ = sm.coarse_solve(S_plain, wl.nc, wl.nc)
    nf1 = wl.nfine - 1
    u_f = torch.empty((n_h, nf1 * nf1), dtype=torch.float64, device="cuda")
    iters = torch.empty(n_h, dtype=torch.int32, device="cuda")
    status = torch.empty(n_h, dtype=torch.int32, device="cuda")
    sm.fine_solve_pcg(a_h[:1], u=u_f[:1], iters=iters[:1], status=status[:1])  # warm-up
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    sm.fine_solve_pcg(a_h, u=u_f, iters=iters, status=status)
    torch.cuda.synchronize()
    t_fine = time.perf_counter() - t0
    mean, var_H, var_d = sm.two_level_mc(U_H, U_Hh, u_f, wl.nc, wl.m)
    N_H = U_H.shape[0]
    H2 = 1.0 / wl.nc ** 2
    mse = H2 * float((var_H / N_H + var_d / n_h).sum())
    # fine-only Monte Carlo with the same sampling error needs N with
    # H^2 sum var_fine / N = mse, var_fine ~ var_H
    n_fine_only = H2 * float(var_H.sum()) / mse if mse > 0 else float("nan")
    it = iters.cpu()
    out = {"workload": f"{wl.nc}x{wl.nc} coarse, H/h={wl.m} (fine {wl.nfine}x{wl.nfine}), {N_H} coarse samples "
                       f"(the benchmark's) + {n_h} fine samples, fine solves by multigrid-preconditioned CG",
           "fine_solve_s": t_fine, "fine_solves_per_s": n_h / t_fine,
           "pcg_iterations_min": int(it.min()), "pcg_iterations_max": int(it.max()),
           "non_converged": int((status != 0).sum().item()),
           "sampling_mse": mse, "var_ratio_d_over_H": float(var_d.sum() / var_H.sum()),
           "max_coarse_minus_fine_mean": float((U_Hh.mean(dim=0) - u_f[:, _coarse_node_index(wl)].mean(dim=0))
                                                .abs().max()),
           "fine_only_mc_samples_for_same_error": n_fine_only,
           "fine_only_mc_s_for_same_error": n_fine_only / (n_h / t_fine)}
    log(f"two-level MC on the benchmark mesh: {out}")
    del a_h, u_f
    torch.cuda.empty_cache()
    return out


def _coarse_node_index(wl):
    nf1 = wl.nc * wl.m - 1
    return [(py * wl.m - 1) * nf1 + (px * wl.m - 1) for py in range(1, wl.nc) for px in range(1, wl.nc)]


def os_flops_per_pair(m: int, o: int) -> float:
    """FP64 operations of the oversampled Petrov-Galerkin cell computation for
    one pair (an FMA counts 2), patch of M = m + 2o cells: per pivot with c
    active rows, the rank-1 window update c(c+1)/2 FMA, 1 div, the forward
    step of the ten right-hand sides 10c FMA and the 21 Schur products 42;
    20 ops per interior row for its stencil, lifts and tests; the 4x4
    recombination (about 300)."""
    M = m + 2 * o
    n = M - 1
    NI = n * n
    f = 0.0
    for j in range(NI):
        c = min(M, NI - 1 - j)
        f += c * (c + 1) + 1 + 20 * c + 42
    return f + 20 * NI + 300


def measure_oversampling(log, N=16384, rb_ntrain=64):
    """Oversampling with the Petrov-Galerkin local stiffness (Sec. 2.2 remark,
    eq. stiffness_local_petrov) on the 8x8 coarse mesh, H/h = 8: patches of
    16 and 24 fine cells per side (oversampling ratios 2 and 3), then the
    non-symmetric coarse solve; against the plain path (no oversampling) at
    the same shape.  The change of the coarse solution that oversampling
    makes is reported as information (the resonance effect itself is a test
    of the oracle)."""
    import torch

    from paper_1607_00693_amd import stomsfem as sm
    from paper_1607_00693_amd import workloads as W

    wl = W.MESH8
    xi = torch.from_numpy(W.uniform_xi(N, wl.nxi, wl.seed)).cuda()
    a = sm.coef_bumps(xi, wl.nfine, **wl.coef_params())
    S_pl = torch.empty((N, wl.M, 10), dtype=torch.float64, device="cuda")
    t_pl = _timed(lambda: sm.upscale(a, wl.nc, wl.nc, wl.m, S=S_pl))
    U_pl, _, _ = sm.coarse_solve(S_pl, wl.nc, wl.nc)
    t_cpl = _timed(lambda: sm.coarse_solve(S_pl, wl.nc, wl.nc, U=U_pl))
    out = {"workload": f"8x8 coarse, H/h=8, {N} samples (bump family, the 8x8 mesh's xi seed)",
           "plain": {"upscale_ms": t_pl * 1e3, "coarse_ms": t_cpl * 1e3, "pairs_per_s": N * wl.M / t_pl}}
    for o in (wl.m // 2, wl.m):
        M = wl.m + 2 * o
        S = torch.empty((N, wl.M, 16), dtype=torch.float64, device="cuda")
        st = torch.empty((N, wl.M), dtype=torch.int32, device="cuda")
        t_os = _timed(lambda: sm.upscale_os(a, wl.nc, wl.nc, wl.m, o, S=S, status=st), reps=3)
        U, _, _ = sm.coarse_solve_pg(S, wl.nc, wl.nc)
        t_cpg = _timed(lambda: sm.coarse_solve_pg(S, wl.nc, wl.nc, U=U), reps=3)
        fl = os_flops_per_pair(wl.m, o)
        d = torch.linalg.norm(U - U_pl, dim=1) / torch.linalg.norm(U_pl, dim=1)
        key = f"ratio_{M // wl.m}"
        out[key] = {"patch_cells": M, "oversample_cells": o,
                    "upscale_ms": t_os * 1e3, "coarse_pg_ms": t_cpg * 1e3,
                    "pairs_per_s": N * wl.M / t_os, "vs_plain_upscale": t_pl / t_os,
                    "flops_per_pair": fl, "achieved_tflops": fl * N * wl.M / t_os / 1e12,
                    "fp64_peak_frac": fl * N * wl.M / t_os / 1e12 / FP64_VALU_PEAK_TFLOPS,
                    "non_ok_pairs": int((st != 0).sum().item()),
                    "max_rel_change_of_U_vs_plain": float(d.max().item())}
        out[key]["reduced_basis"] = measure_rb_os(wl, a, o, S, U, t_os, ntrain=rb_ntrain)
        log(f"oversampling ratio {M // wl.m}: {out[key]}")
    return out


def measure_oversampling_large(log):
    """Oversampled Petrov-Galerkin upscaling with patches of 30 to 64 cells
    (log-normal coefficients, sigma = 1, seed 11), ratio 3 at H/h = 10, 14,
    16, 18 and 20 (30, 42, 48, 54 and 60 cells; 16x16, 16x16, 16x16, 8x8 and
    12x12 coarse meshes, 64 samples; 60 cells is the geometry of the
    high-contrast example of Sec. 5.2) and 64 cells (16x16 coarse, H/h = 32,
    ratio 2, 16 samples)."""
    import torch

    from paper_1607_00693_amd import stomsfem as sm
    from paper_1607_00693_amd import workloads as W

    out = {}
    for nc, m, o, N in ((16, 10, 10, 64), (16, 14, 14, 64), (16, 16, 16, 64), (8, 18, 18, 64), (12, 20, 20, 64),
                        (16, 32, 16, 16)):
        a = torch.from_numpy(W.lognormal_field((N, nc * m, nc * m), 1.0, 11)).cuda()
        S = torch.empty((N, nc * nc, 16), dtype=torch.float64, device="cuda")
        st = torch.empty((N, nc * nc), dtype=torch.int32, device="cuda")
        t = _timed(lambda: sm.upscale_os(a, nc, nc, m, o, S=S, status=st), reps=3)
        fl = os_flops_per_pair(m, o)
        pairs = N * nc * nc
        out[f"patch_{m + 2 * o}"] = {"mesh": f"{nc}x{nc} coarse, H/h={m}, oversample {o}, {N} samples",
                                     "ms": t * 1e3, "pairs_per_s": pairs / t, "flops_per_pair": fl,
                                     "fp64_peak_frac": fl * pairs / t / 1e12 / FP64_VALU_PEAK_TFLOPS,
                                     "non_ok_pairs": int((st != 0).sum().item())}
        log(f"oversampled patches of {m + 2 * o} cells: {out[f'patch_{m + 2 * o}']}")
        del a, S, st
    return out


def measure_rb_os_sec52(log, nc=12, m=20, o=20, ntrain=64, N=1024):
    """Reduced basis on oversampled patches in the geometry of the example of
    Sec. 5.2 (H/h = 20, oversampling ratio 3: 60-cell patches) on the bump
    medium (16 bumps of radius 1/4 on a 4x4 grid, eps = 1/32; xi ~ U[-1,1]^16,
    training seed 2003, samples seed 1003): offline time (band-window
    snapshots, method of snapshots), both online stages against the
    oversampled solve of the same pairs (row-distributed kernel)."""
    import torch

    from paper_1607_00693_amd import stomsfem as sm
    from paper_1607_00693_amd import workloads as W

    wl = W.MESH8
    nf = nc * m
    xi_tr = torch.from_numpy(W.uniform_xi(ntrain, wl.nxi, 2003)).cuda()
    a_tr = sm.coef_bumps(xi_tr, nf, **wl.coef_params())
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    model = sm.reduce_os(a_tr, nc, nc, m, o, r_max=8, tail_tol=1e-6)
    t_off = time.perf_counter() - t0
    del a_tr
    xi = torch.from_numpy(W.uniform_xi(N, wl.nxi, 1003)).cuda()
    a = sm.coef_bumps(xi, nf, **wl.coef_params())
    M = nc * nc
    S_os = torch.empty((N, M, 16), dtype=torch.float64, device="cuda")
    t_os = _timed(lambda: sm.upscale_os(a, nc, nc, m, o, S=S_os), reps=2)
    U_os, _, _ = sm.coarse_solve_pg(S_os, nc, nc)
    r = model.export("r")
    out = {"workload": f"{nc}x{nc} coarse, H/h={m}, oversample {o} (patches of {m + 2 * o} cells, ratio "
                       f"{(m + 2 * o) // m}), bump medium, {ntrain} training samples, {N} samples",
           "offline_s": t_off, "modes_min": int(r.min()), "modes_max": int(r.max()),
           "oversampled_solve_ms": t_os * 1e3, "oversampled_solve_pairs_per_s": N * M / t_os}
    S = torch.empty_like(S_os)
    a32 = a.float()
    scale = S_os.abs().amax(dim=2, keepdim=True)
    for key, prec, aa in (("fp32_matrix_core", sm.PREC_F32, a32), ("fp64", sm.PREC_F64, a)):
        t_on = _timed(lambda: sm.reduce_os_apply(model, aa, S=S, precision=prec), reps=3)
        rel = ((S - S_os).abs() / scale).amax(dim=2)
        U, _, _ = sm.coarse_solve_pg(S, nc, nc)
        d = torch.linalg.norm(U - U_os, dim=1) / torch.linalg.norm(U_os, dim=1)
        out[key] = {"online_ms": t_on * 1e3, "pairs_per_s": N * M / t_on, "vs_oversampled_solve": t_os / t_on,
                    "max_S_rel_err": float(rel.max()), "median_S_rel_err": float(rel.median()),
                    "max_coarse_rel_err": float(d.max())}
    log(f"reduced basis, oversampled, Sec. 5.2 geometry: {out}")
    model.free()
    return out


def measure_rb_os(wl, a, o, S_os, U_os, t_os, ntrain=64, r_max=8, tail_tol=1e-6):
    """Reduced basis on the oversampled patches (Sec. 3.2 on the patches of
    the Petrov-Galerkin MsFEM, as in the high-contrast example of Sec. 5.2):
    offline from ntrain training samples (seed 2003), FP64 online stage on the
    samples a, against the oversampled solve S_os (t_os seconds)."""
    import torch

    from paper_1607_00693_amd import stomsfem as sm
    from paper_1607_00693_amd import workloads as W

    xi_tr = torch.from_numpy(W.uniform_xi(ntrain, wl.nxi, 2003)).cuda()
    a_tr = sm.coef_bumps(xi_tr, wl.nfine, **wl.coef_params())
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    model = sm.reduce_os(a_tr, wl.nc, wl.nc, wl.m, o, r_max=r_max, tail_tol=tail_tol)
    t_off = time.perf_counter() - t0
    del a_tr
    N = a.shape[0]
    S = torch.empty_like(S_os)
    st = torch.empty((N, wl.M), dtype=torch.int32, device="cuda")
    scale = S_os.abs().amax(dim=2, keepdim=True)
    r = model.export("r")
    out = {"workload": f"{ntrain} training samples, r<={r_max} (tail {tail_tol:g}); FP32 matrix-core online "
                       "stage on FP32 coefficients (GEMM [128 samples x Mp^2] x [Mp^2 x 112] per workgroup, "
                       "FP64 8x8 solve and 4x4 recombination per pair) and the FP64 online stage",
           "offline_s": t_off, "modes_min": int(r.min()), "modes_max": int(r.max())}
    a32 = a.float()
    mp = wl.m + 2 * o
    for key, prec, aa in (("fp32_matrix_core", sm.PREC_F32, a32), ("fp64", sm.PREC_F64, a)):
        t_on = _timed(lambda: sm.reduce_os_apply(model, aa, S=S, status=st, precision=prec), reps=3)
        s_err = float(((S - S_os).abs() / scale).max())
        U, _, _ = sm.coarse_solve_pg(S, wl.nc, wl.nc)
        d = torch.linalg.norm(U - U_os, dim=1) / torch.linalg.norm(U_os, dim=1)
        out[key] = {"online_ms": t_on * 1e3, "pairs_per_s": N * wl.M / t_on, "vs_oversampled_solve": t_os / t_on,
                    "non_ok_pairs": int((st != 0).sum().item()), "max_S_rel_err": s_err,
                    "max_coarse_rel_err": float(d.max().item())}
        if prec == sm.PREC_F32:
            kd = ((mp * mp + 63) // 64) * 64
            fl = 2.0 * kd * 112  # the GEMM row of one pair (padded table)
            out[key]["mfma_flops_per_pair"] = fl
            out[key]["achieved_tflops"] = fl * N * wl.M / t_on / 1e12
            out[key]["fp32_mfma_peak_frac"] = fl * N * wl.M / t_on / 1e12 / FP32_MFMA_PEAK_TFLOPS
    del a32
    model.free()
    return out


def measure_rb_os_channels(log, nsub=16, ntrain=64, N=1024, r_max=8, tail_tol=1e-6):
    """Reduced basis on oversampled patches in the high-contrast medium (the
    setting of the example of Sec. 5.2: oversampling, Petrov-Galerkin, a few
    reduced modes per patch): the channels-and-inclusions medium at H/h = 8
    (64 x 64 coarse mesh, 512 x 512 fine), restricted to the nsub x nsub coarse
    elements with the most features, ratios 2 and 3; ntrain training samples
    (seed 6005), N test samples (seed 6006); both online stages against the
    oversampled solve of the same pairs."""
    import numpy as np
    import torch

    from paper_1607_00693_amd import stomsfem as sm
    from paper_1607_00693_amd import workloads as W

    wl = W.CHANNELS64
    m = 8
    kind, x0, y0, size = W.channel_geometry(wl)
    g = [torch.from_numpy(np.ascontiguousarray(v)).cuda() for v in (kind, x0, y0, size)]
    fmap = sm.feature_map(wl.nc * m, *g)
    # the sub-domain of nsub x nsub elements (aligned to nsub) holding the most distinct features
    f = fmap.cpu().numpy()
    w = nsub * m
    best, org = -1, (0, 0)
    for by in range(0, wl.nc * m, w):
        for bx in range(0, wl.nc * m, w):
            nf = len(np.unique(f[by:by + w, bx:bx + w]))
            if nf > best:
                best, org = nf, (by, bx)
    by, bx = org

    def field(n, seed):
        xi = torch.from_numpy(W.normal_xi(n, wl.nxi, seed)).cuda()
        return sm.coef_features(fmap, wl.nxi, xi, wl.decades)[:, by:by + w, bx:bx + w].contiguous()

    a_tr, a = field(ntrain, 6005), field(N, 6006)
    out = {"workload": f"channels medium, H/h = {m}, the {nsub}x{nsub} coarse elements at fine offset ({by}, {bx}) "
                       f"({best - 1} features), {ntrain} training samples, r<={r_max} (tail {tail_tol:g}), {N} samples",
           "contrast": float(a.max() / a.min())}
    for o in (m // 2, m):
        S_os = torch.empty((N, nsub * nsub, 16), dtype=torch.float64, device="cuda")
        t_os = _timed(lambda: sm.upscale_os(a, nsub, nsub, m, o, S=S_os), reps=2)
        U_os, _, _ = sm.coarse_solve_pg(S_os, nsub, nsub)
        t0 = time.perf_counter()
        model = sm.reduce_os(a_tr, nsub, nsub, m, o, r_max=r_max, tail_tol=tail_tol)
        t_off = time.perf_counter() - t0
        r = model.export("r")
        res = {"patch_cells": m + 2 * o, "offline_s": t_off, "modes_min": int(r.min()),
               "modes_mean": float(r.mean()), "modes_max": int(r.max()),
               "oversampled_solve_pairs_per_s": N * nsub * nsub / t_os}
        S = torch.empty_like(S_os)
        st = torch.empty((N, nsub * nsub), dtype=torch.int32, device="cuda")
        a32 = a.float()
        for key, prec, aa in (("fp32_matrix_core", sm.PREC_F32, a32), ("fp64", sm.PREC_F64, a)):
            t_on = _timed(lambda: sm.reduce_os_apply(model, aa, S=S, status=st, precision=prec), reps=3)
            scale = S_os.abs().amax(dim=2, keepdim=True)
            rel = ((S - S_os).abs() / scale).amax(dim=2)
            U, _, _ = sm.coarse_solve_pg(S, nsub, nsub)
            d = torch.linalg.norm(U - U_os, dim=1) / torch.linalg.norm(U_os, dim=1)
            res[key] = {"pairs_per_s": N * nsub * nsub / t_on, "vs_oversampled_solve": t_os / t_on,
                        "non_ok_pairs": int((st != 0).sum().item()), "max_S_rel_err": float(rel.max()),
                        "median_S_rel_err": float(rel.median()),
                        "fraction_of_pairs_above": {f"{t:g}": float((rel > t).float().mean()) for t in (1e-6, 1e-3, 1e-1)},
                        "median_coarse_rel_err": float(d.median()), "max_coarse_rel_err": float(d.max())}
        # the same pairs, coefficients rounded to FP32 for both sides: the matrix-core stage's own error
        S32_os = sm.upscale_os(a32, nsub, nsub, m, o)
        sm.reduce_os_apply(model, a32, S=S, status=st, precision=sm.PREC_F64)
        S64 = S.clone()
        sm.reduce_os_apply(model, a32, S=S, status=st, precision=sm.PREC_F32)
        res["fp32_stage_vs_fp64_stage_max_rel"] = float(((S - S64).abs() / S64.abs().amax(dim=2, keepdim=True)).max())
        res["fp64_stage_on_fp32_a_vs_solve_max_rel"] = float(
            ((S64 - S32_os).abs() / S32_os.abs().amax(dim=2, keepdim=True)).max())
        out[f"ratio_{(m + 2 * o) // m}"] = res
        log(f"reduced basis, oversampled, channels medium, ratio {(m + 2 * o) // m}: {res}")
        model.free()
        del a32, S32_os, S64
    return out


def measure_collocation(log, wl=None, level=4, errors=True, plain_chunk=1024):
    """Sparse-grid stochastic collocation with search-and-plug-in
    dictionaries (Sec. 4.1.2, global SC methods; Sec. 5.2)
    on a bump-family mesh (default 8x8, H/h = 8, 16 uniform variables), the
    level-`level` Smolyak Clenshaw-Curtis grid: offline dictionaries, then
    the online stage for every collocation point (search and plug-in, coarse
    solve, weighted quadrature) against the plain path at the same points
    (coefficients from the node values, upscaling, coarse solve, quadrature;
    timed on the first `plain_chunk` points and scaled to all of them when
    there are more); the ratio is the online saving 1/R of eq. SConlinecost.
    With `errors`: the quadrature error of the lower levels and of Monte
    Carlo with as many samples as the level-(level-1) grid, both against the
    level-`level` estimate."""
    import math

    import torch

    from paper_1607_00693_amd import stomsfem as sm
    from paper_1607_00693_amd import workloads as W

    wl = wl or W.MESH8
    fam = sm.bump_family(wl)
    lv, nl = sm.local_vars_bumps(wl.nc, wl.nc, wl.m, fam)
    nU = (wl.nc - 1) ** 2
    t0 = time.perf_counter()
    dg, w = sm.sparse_grid(wl.nxi, level)
    t_grid = time.perf_counter() - t0
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    model = sm.sc_build(wl.nc, wl.nc, wl.m, lv, fam, level, dg)
    torch.cuda.synchronize()
    t_off = time.perf_counter() - t0
    n = len(w)
    dgd, wd = torch.from_numpy(dg).cuda(), torch.from_numpy(w).cuda()
    S = torch.empty((n, wl.M, 10), dtype=torch.float64, device="cuda")
    U = torch.empty((n, nU), dtype=torch.float64, device="cuda")

    def online():
        sm.sc_apply(model, dgd, S=S)
        sm.coarse_solve(S, wl.nc, wl.nc, U=U)
        return sm.quadrature(U, wd)

    t_on = _timed(online)
    mean, var = online()
    t_apply = _timed(lambda: sm.sc_apply(model, dgd, S=S))
    t_quad = _timed(lambda: sm.quadrature(U, wd))
    npl = min(n, plain_chunk)
    xi = torch.cos(math.pi * dgd[:npl].double() / 2 ** level)  # node values on [-1, 1]
    Sp, Up = S[:npl], U[:npl]

    def plain():
        a = sm.coef_bumps(xi, wl.nfine, **wl.coef_params())
        sm.upscale(a, wl.nc, wl.nc, wl.m, S=Sp)
        sm.coarse_solve(Sp, wl.nc, wl.nc, U=Up)
        return sm.quadrature(Up, wd[:npl])

    t_plain = _timed(plain, reps=3) * n / npl
    diff = float((S[:npl] - sm.sc_apply(model, dgd[:npl])).abs().max().item())  # S holds the plain S here
    dict_rows = 0
    for K in range(wl.M):
        cols = [int(j) for j in lv[K][:nl[K]]]
        dict_rows += len({tuple(r) for r in dg[:, cols].tolist()}) if cols else 1
    out = {"workload": (f"{wl.nc}x{wl.nc} coarse, H/h={wl.m}, {wl.nxi} uniform variables (bump family), "
                        f"Smolyak Clenshaw-Curtis level {level}"),
           "points": n, "dictionary_entries": dict_rows, "grid_s": t_grid, "offline_s": t_off,
           "online_ms": t_on * 1e3, "online_points_per_s": n / t_on, "search_plug_in_ms": t_apply * 1e3,
           "search_plug_in_GB_per_s": n * wl.M * 80 / t_apply / 1e9, "quadrature_ms": t_quad * 1e3,
           "plain_ms": t_plain * 1e3, "plain_timed_points": npl, "online_saving_vs_plain": t_plain / t_on,
           "max_abs_S_diff_plug_in_vs_plain": diff,
           "max_mean": float(mean.abs().max().item()), "max_std": float(var.clamp(min=0).sqrt().max().item())}
    if errors:
        err = {}
        for L in range(1, level):
            dl, wlv = sm.sparse_grid(wl.nxi, L)
            dl = torch.from_numpy(dl * (2 ** level // 2 ** max(L, 1))).cuda()
            SL = sm.sc_apply(model, dl)
            UL, _, _ = sm.coarse_solve(SL, wl.nc, wl.nc)
            mL, _ = sm.quadrature(UL, torch.from_numpy(wlv).cuda())
            err[f"level_{L}"] = {"points": int(len(wlv)), "err": float(torch.linalg.norm(mL - mean).item())}
        nmc = err[f"level_{level - 1}"]["points"]
        xmc = torch.from_numpy(W.uniform_xi(nmc, wl.nxi, wl.seed + 77)).cuda()
        Smc = sm.upscale(sm.coef_bumps(xmc, wl.nfine, **wl.coef_params()), wl.nc, wl.nc, wl.m)
        _, mmc, _ = sm.coarse_solve(Smc, wl.nc, wl.nc)
        err["monte_carlo"] = {"points": nmc, "err": float(torch.linalg.norm(mmc - mean).item())}
        out["quadrature_error_vs_top_level"] = err
    log(f"collocation: {out}")
    return out


def measure_two_level(log, n_H=16384, n_h=512):
    """Two-level Monte Carlo (Sec. 4.1.1, the remark with eqs. MCmean2level
    and mseML) on the 8x8 mesh, H/h = 8: n_H coarse StoMsFEM samples
    (coefficients, upscaling, coarse solve), n_h independent samples with both
    the coarse and the fine-grid (64 x 64) FEM solution, and the estimator.
    Reports the times, the per-sample cost ratio of the coarse and fine
    solves, the estimated sampling part of the MSE, the discretisation bias
    of the coarse-only mean that the correction removes, and the cost of a
    fine-grid-only MC with the same sampling error (from the sample
    variances)."""
    import torch

    from paper_1607_00693_amd import stomsfem as sm
    from paper_1607_00693_amd import workloads as W

    wl = W.MESH8
    xH = torch.from_numpy(W.uniform_xi(n_H, wl.nxi, wl.seed + 11)).cuda()
    xh = torch.from_numpy(W.uniform_xi(n_h, wl.nxi, wl.seed + 12)).cuda()
    nU = (wl.nc - 1) ** 2
    U_H = torch.empty((n_H, nU), dtype=torch.float64, device="cuda")
    U_Hh = torch.empty((n_h, nU), dtype=torch.float64, device="cuda")
    u_f = torch.empty((n_h, (wl.nfine - 1) ** 2), dtype=torch.float64, device="cuda")

    def coarse(x, U):
        a = sm.coef_bumps(x, wl.nfine, **wl.coef_params())
        sm.coarse_solve(sm.upscale(a, wl.nc, wl.nc, wl.m), wl.nc, wl.nc, U=U)
        return a

    def fine():
        a = coarse(xh, U_Hh)
        sm.fine_solve(a, u=u_f)

    t_H = _timed(lambda: coarse(xH, U_H), reps=3)
    t_h = _timed(fine, reps=3)
    t_est = _timed(lambda: sm.two_level_mc(U_H, U_Hh, u_f, wl.nc, wl.m))
    a_h = sm.coef_bumps(xh, wl.nfine, **wl.coef_params())
    t_fine_only = _timed(lambda: sm.fine_solve(a_h, u=u_f), reps=3)
    coarse(xh, U_Hh)
    sm.fine_solve(a_h, u=u_f)
    mean, var_H, var_d = sm.two_level_mc(U_H, U_Hh, u_f, wl.nc, wl.m)
    torch.cuda.synchronize()
    H2 = 1.0 / wl.nc**2
    mse = H2 * float((var_H / n_H + var_d / n_h).sum())
    # fine-grid-only MC with the same sampling error: var[u_h] ~ var[u_H]
    n_fine_equiv = H2 * float(var_H.sum()) / mse
    cost_fine_only = n_fine_equiv * t_h / n_h
    out = {"workload": f"8x8 coarse, H/h=8 (fine 64x64), {n_H} coarse + {n_h} fine samples (bump family)",
           "coarse_ms": t_H * 1e3, "fine_ms": t_h * 1e3, "fine_solve_ms": t_fine_only * 1e3,
           "fine_solves_per_s": n_h / t_fine_only, "estimator_ms": t_est * 1e3,
           "coarse_per_sample_us": t_H / n_H * 1e6, "fine_per_sample_us": t_h / n_h * 1e6,
           "sampling_mse": mse, "rms_sampling_error": mse ** 0.5,
           "coarse_only_bias_max": float((U_H.mean(dim=0) - mean).abs().max().item()),
           "var_ratio_d_over_H": float(var_d.sum().item() / var_H.sum().item()),
           "fine_only_mc_samples_for_same_error": n_fine_equiv,
           "fine_only_mc_ms_for_same_error": cost_fine_only * 1e3,
           "two_level_ms": (t_H + t_h + t_est) * 1e3}
    log(f"two-level MC: {out}")
    return out


def measure_gauss(log, N=1024, n_trunc=64):
    """The short-correlation Gaussian medium (Sec. 5.3) on a 16x16 coarse
    mesh with H/h = 16 and its local KL on the coarse elements: field
    generation (randomized spectral method, 256 terms) and projection to the
    local parameters for N samples; the rate of pairs with a parameter
    outside [-3, 3] among the four kept ones against 1 - P(|Z| <= 3)^4 =
    0.0108; and, on n_trunc samples, the error of S and of the coarse
    solution (source b = 2 + x1 x2 as in Sec. 5.3, through the element loads)
    when kappa is replaced by its truncated local KL with K terms
    (eq. local_KL_truncation); and the local KL in the paper's geometry, on
    the oversampled patches of side 2H with l2 = H (kept spectrum, out-of-box
    rate, projection throughput)."""
    import math

    import numpy as np
    import torch

    from paper_1607_00693_amd import stomsfem as sm
    from paper_1607_00693_amd import workloads as W

    wl = W.GAUSS16
    gl = sm.element_loads(wl.nc, wl.nc)  # Sec. 5.3's source b = 2 + x1 x2
    z, u = W.spectral_draws(N, wl.nterms, wl.seed)
    z, u = torch.from_numpy(z).cuda(), torch.from_numpy(u).cuda()
    t_field = _timed(lambda: sm.coef_gauss(z, u, wl.nfine, wl.l1, wl.l2, with_beta=True), reps=3)
    kap, beta = sm.coef_gauss(z, u, wl.nfine, wl.l1, wl.l2, with_beta=True)
    Kmax = 8
    mu, V, cap = sm.local_kl(wl.m, 1.0 / wl.nfine, wl.l1, wl.l2, Kmax)
    mu_d, V_d = torch.from_numpy(mu).cuda(), torch.from_numpy(V).cuda()
    mu4, V4 = mu_d[:wl.kl_terms].contiguous(), V_d[:wl.kl_terms].contiguous()
    t_proj = _timed(lambda: sm.kl_project(beta, wl.nc, wl.m, mu4, V4, wl.box))
    _, _, count = sm.kl_project(beta, wl.nc, wl.m, mu4, V4, wl.box)
    pairs = N * wl.M
    rate = int(count.item()) / pairs
    p_ref = 1.0 - math.erf(wl.box / math.sqrt(2.0)) ** wl.kl_terms
    n = n_trunc
    xi, _, _ = sm.kl_project(beta[:n].contiguous(), wl.nc, wl.m, mu_d, V_d, wl.box)
    S_full = sm.upscale(kap[:n].contiguous(), wl.nc, wl.nc, wl.m)
    U_full, _, _ = sm.coarse_solve(S_full, wl.nc, wl.nc, load=gl)
    scale = S_full.abs().amax(dim=2)
    trunc = {}
    for K in (1, 2, 3, 4, 6, 8):
        S_t = sm.upscale(sm.kl_blocks(xi, mu_d, V_d, K), 1, 1, wl.m).reshape(n, wl.M, 10)
        U_t, _, _ = sm.coarse_solve(S_t, wl.nc, wl.nc, load=gl)
        trunc[f"K_{K}"] = {
            "captured": float(mu[:K].sum() / (wl.m * wl.m)),
            "max_S_rel_err": float(((S_t - S_full).abs().amax(dim=2) / scale).max().item()),
            "max_coarse_rel_err": float((torch.linalg.norm(U_t - U_full, dim=1) /
                                         torch.linalg.norm(U_full, dim=1)).max().item())}
    # interpolation in the four local parameters (7 and 9 Lobatto nodes each)
    # with the plain path on the sample's own coefficient outside [-3, 3]
    xi4, out4, _ = sm.kl_project(beta, wl.nc, wl.m, mu4, V4, wl.box)
    S_all = sm.upscale(kap, wl.nc, wl.nc, wl.m)
    torch.cuda.synchronize()
    t_plain = _timed(lambda: sm.upscale(kap, wl.nc, wl.nc, wl.m, S=S_all), reps=3)
    sc_all = S_all.abs().amax(dim=2)
    # reference for the interpolation error alone: the truncated-coefficient
    # S, with the out-of-box pairs taken from the sample as the online stage does
    S_t4 = sm.upscale(sm.kl_blocks(xi4[:n].contiguous(), mu4, V4, wl.kl_terms), 1, 1, wl.m).reshape(n, wl.M, 10)
    fb4 = out4[:n].bool()
    S_t4[fb4] = S_all[:n][fb4]
    U_t4, _, _ = sm.coarse_solve(S_t4, wl.nc, wl.nc, load=gl)
    interp = {}
    for nn in (7, 9):
        t0 = time.perf_counter()
        model = sm.kl_interp_build(wl.nc, wl.nc, wl.m, mu4, V4, nn, wl.box)
        torch.cuda.synchronize()
        t_build = time.perf_counter() - t0
        S_int = torch.empty((N, wl.M, 10), dtype=torch.float64, device="cuda")
        t_int = _timed(lambda: sm.kl_interp_apply(model, xi4, kap, S=S_int), reps=3)
        _, nfb = sm.kl_interp_apply(model, xi4, kap, S=S_int)
        U_int, _, _ = sm.coarse_solve(S_int[:n].contiguous(), wl.nc, wl.nc, load=gl)
        interp[f"nodes_{nn}"] = {
            "table_rows": nn ** 4, "build_s": t_build, "apply_ms": t_int * 1e3,
            "pairs_per_s": pairs / t_int, "plain_pairs_per_s": pairs / t_plain, "ratio_vs_plain": t_plain / t_int,
            # per sample as in the paper's comparison: field generation and
            # projection included on the interpolation side
            "ratio_vs_plain_with_field": (t_field + t_plain) / (t_field + t_proj + t_int),
            "plain_fallback_pairs": nfb, "fallback_rate": nfb / pairs,
            "max_S_rel_err_vs_sample": float(((S_int - S_all).abs().amax(dim=2) / sc_all).max().item()),
            "max_S_rel_err_vs_truncated_interpolated_pairs": float(
                ((S_int[:n] - S_t4).abs().amax(dim=2) / sc_all[:n])[~fb4].max().item()),
            "max_coarse_rel_err_vs_sample": float((torch.linalg.norm(U_int - U_full, dim=1) /
                                                   torch.linalg.norm(U_full, dim=1)).max().item()),
            "max_coarse_rel_err_vs_truncated": float((torch.linalg.norm(U_int - U_t4, dim=1) /
                                                      torch.linalg.norm(U_t4, dim=1)).max().item())}
        model.free()
    # the paper's geometry: local KL on the oversampled patches of side 2H
    # (ratio 2: H/2 on each side, moved inside at the boundary) with l2 = H,
    # four terms; kept spectrum and out-of-box rate against 0.0108
    o = wl.m // 2
    l2_os = 1.0 / wl.nc
    _, beta_os = sm.coef_gauss(z, u, wl.nfine, wl.l1, l2_os, with_beta=True)
    mu_os, V_os, _ = sm.local_kl(wl.m + 2 * o, 1.0 / wl.nfine, wl.l1, l2_os, wl.kl_terms)
    mu_os_d, V_os_d = torch.from_numpy(mu_os).cuda(), torch.from_numpy(V_os).cuda()
    t_proj_os = _timed(lambda: sm.kl_project(beta_os, wl.nc, wl.m, mu_os_d, V_os_d, wl.box, oversample=o))
    _, _, count_os = sm.kl_project(beta_os, wl.nc, wl.m, mu_os_d, V_os_d, wl.box, oversample=o)
    patch_kl = {"patch_side_cells": wl.m + 2 * o, "l2": l2_os, "terms": wl.kl_terms,
                "kept_fraction": float(mu_os.sum() / (wl.m + 2 * o) ** 2),
                "outside_rate": int(count_os.item()) / pairs, "outside_rate_gaussian": p_ref,
                "projection_ms": t_proj_os * 1e3, "pairs_per_s_projection": pairs / t_proj_os}
    # interpolation of the oversampled Petrov-Galerkin stiffness in the patch
    # parameters (the paper's combination), against the oversampled solve of
    # every pair of the same samples
    kap_os = 0.1 + torch.exp(beta_os)
    xi_os, out_os, _ = sm.kl_project(beta_os, wl.nc, wl.m, mu_os_d, V_os_d, wl.box, oversample=o)
    S_pl = sm.upscale_os(kap_os, wl.nc, wl.nc, wl.m, o)
    torch.cuda.synchronize()
    t_pl = _timed(lambda: sm.upscale_os(kap_os, wl.nc, wl.nc, wl.m, o, S=S_pl), reps=2)
    sc_pl = S_pl.abs().amax(dim=2)
    U_pl, _, _ = sm.coarse_solve_pg(S_pl[:n_trunc].contiguous(), wl.nc, wl.nc, load=gl)
    os_interp = {}
    # tensor grids of 5 and 7 nodes per parameter; sparse grids of levels 4
    # and 5 (401 and 1105 nodes in four parameters)
    for name, nn, level, nodes in (("nodes_5", 5, None, 5 ** 4), ("nodes_7", 7, None, 7 ** 4),
                                   ("sparse_level_4", 0, 4, 401), ("sparse_level_5", 0, 5, 1105)):
        t0 = time.perf_counter()
        model = sm.kl_interp_build(wl.nc, wl.nc, wl.m, mu_os_d, V_os_d, nn, wl.box, oversample=o, level=level)
        torch.cuda.synchronize()
        t_build = time.perf_counter() - t0
        S_i = torch.empty_like(S_pl)
        t_i = _timed(lambda: sm.kl_interp_apply(model, xi_os, kap_os, S=S_i), reps=3)
        _, nfb = sm.kl_interp_apply(model, xi_os, kap_os, S=S_i)
        U_i, _, _ = sm.coarse_solve_pg(S_i[:n_trunc].contiguous(), wl.nc, wl.nc, load=gl)
        ins = ~out_os.bool()
        os_interp[name] = {
            "nodes_per_class": nodes, "table_rows": 9 * nodes, "build_s": t_build, "apply_ms": t_i * 1e3,
            "pairs_per_s": pairs / t_i,
            "oversampled_plain_pairs_per_s": pairs / t_pl, "ratio_vs_oversampled_plain": t_pl / t_i,
            "ratio_vs_oversampled_plain_with_field": (t_field + t_pl) / (t_field + t_proj_os + t_i),
            "fallback_pairs": nfb,
            "max_S_rel_err_vs_sample_interpolated_pairs": float(
                ((S_i - S_pl).abs().amax(dim=2) / sc_pl)[ins].max().item()),
            "max_coarse_rel_err_vs_sample": float((torch.linalg.norm(U_i - U_pl, dim=1) /
                                                   torch.linalg.norm(U_pl, dim=1)).max().item())}
        model.free()
    patch_kl["interpolation_of_oversampled_stiffness"] = os_interp
    del beta_os, kap_os, S_pl
    out = {"workload": (f"kappa = 0.1 + exp(beta), Gaussian beta (l1={wl.l1}, l2={wl.l2}, {wl.nterms} spectral "
                        f"terms), {wl.nc}x{wl.nc} coarse, H/h={wl.m}, local KL on the coarse elements"),
           "interpolation_in_kl_parameters": interp,
           "samples": N, "field_ms": t_field * 1e3, "field_elements_per_s": N * wl.nfine**2 / t_field,
           "projection_ms": t_proj * 1e3, "pairs_per_s_projection": pairs / t_proj,
           "kept_fraction_4_terms": float(mu[:4].sum() / (wl.m * wl.m)),
           "outside_rate": rate, "outside_rate_gaussian": p_ref,
           "truncation": trunc,
           "oversampled_patch_kl": patch_kl}
    log(f"gaussian medium: {out}")
    return out


def measure_gauss_paper_mesh(log, N=8):
    """The Gaussian medium on the paper's own Sec. 5.3 mesh: h = 2^-11
    (2048 x 2048 fine elements), H/h = 32 (64 x 64 coarse elements),
    oversampling ratio 2 (patches of 2H = 64 fine cells, moved inside at the
    edge) and the local KL on those patches with l2 = H, four terms, source
    b = 2 + x1 x2.  N samples: field, projection, the oversampled
    Petrov-Galerkin solve of every pair, and the interpolation of the
    oversampled stiffness in the patch parameters (5 tensor nodes per
    parameter, nine class tables) with the oversampled solve as fallback
    outside the box; errors of S and of the coarse solution against the solve
    of every pair."""
    import math

    import torch

    from paper_1607_00693_amd import stomsfem as sm
    from paper_1607_00693_amd import workloads as W

    wl = W.GAUSS16
    nc, m, o = 64, 32, 16
    nfine, l2 = nc * m, 1.0 / nc
    pairs = N * nc * nc
    gl = sm.element_loads(nc, nc)
    z, u = W.spectral_draws(N, wl.nterms, wl.seed + 11)
    z, u = torch.from_numpy(z).cuda(), torch.from_numpy(u).cuda()
    t_field = _timed(lambda: sm.coef_gauss(z, u, nfine, wl.l1, l2, with_beta=True), reps=2)
    kap, beta = sm.coef_gauss(z, u, nfine, wl.l1, l2, with_beta=True)
    mu, V, _ = sm.local_kl(m + 2 * o, 1.0 / nfine, wl.l1, l2, wl.kl_terms)
    mu_d, V_d = torch.from_numpy(mu).cuda(), torch.from_numpy(V).cuda()
    t_proj = _timed(lambda: sm.kl_project(beta, nc, m, mu_d, V_d, wl.box, oversample=o))
    xi, out, count = sm.kl_project(beta, nc, m, mu_d, V_d, wl.box, oversample=o)
    S_pl = sm.upscale_os(kap, nc, nc, m, o)
    torch.cuda.synchronize()
    t_pl = _timed(lambda: sm.upscale_os(kap, nc, nc, m, o, S=S_pl), reps=1)
    log(f"paper mesh: oversampled solve of {pairs} pairs in {t_pl * 1e3:.1f} ms")
    U_pl, _, _ = sm.coarse_solve_pg(S_pl, nc, nc, load=gl)
    t0 = time.perf_counter()
    model = sm.kl_interp_build(nc, nc, m, mu_d, V_d, 5, wl.box, oversample=o)
    torch.cuda.synchronize()
    t_build = time.perf_counter() - t0
    S_i = torch.empty_like(S_pl)
    t_i = _timed(lambda: sm.kl_interp_apply(model, xi, kap, S=S_i), reps=1)
    _, nfb = sm.kl_interp_apply(model, xi, kap, S=S_i)
    U_i, _, _ = sm.coarse_solve_pg(S_i, nc, nc, load=gl)
    model.free()
    sc = S_pl.abs().amax(dim=2)
    ins = ~out.bool()
    res = {"workload": f"Gaussian medium on the paper's Sec. 5.3 mesh: h = 2^-11 ({nfine}x{nfine}), {nc}x{nc} coarse "
                       f"(H/h = {m}), oversampling ratio 2 (patches of {m + 2 * o} cells), local KL on the patches "
                       f"with l2 = H, {wl.kl_terms} terms, b = 2 + x1 x2, {N} samples",
           "pairs": pairs, "kept_fraction": float(mu.sum() / (m + 2 * o) ** 2),
           "outside_rate": int(count.item()) / pairs,
           "outside_rate_gaussian": 1.0 - math.erf(wl.box / math.sqrt(2.0)) ** wl.kl_terms,
           "field_ms": t_field * 1e3, "projection_ms": t_proj * 1e3,
           "oversampled_solve_ms": t_pl * 1e3, "oversampled_solve_pairs_per_s": pairs / t_pl,
           "interpolation_nodes_5": {"table_rows": 9 * 5 ** 4, "build_s": t_build, "apply_ms": t_i * 1e3,
                                     "pairs_per_s": pairs / t_i, "ratio_vs_oversampled_solve": t_pl / t_i,
                                     "fallback_pairs": nfb,
                                     "max_S_rel_err_interpolated_pairs": float(((S_i - S_pl).abs().amax(dim=2)
                                                                                / sc)[ins].max().item()),
                                     "max_coarse_rel_err": float((torch.linalg.norm(U_i - U_pl, dim=1) /
                                                                  torch.linalg.norm(U_pl, dim=1)).max().item())}}
    log(f"gaussian medium, paper mesh: {res}")
    return res


def measure_accelerations(log):
    """Reduced basis (8x8 coarse, H/h = 8, 256 training samples, r <= 8,
    16384 online samples, FP32 coefficients) and learned surrogate (same mesh,
    2048 training samples per patch, 65536 test samples, gate 1e-3) against
    the plain FP64 path at the same shapes.  Each comparison reports
    throughputs in pairs/s, their ratio and the worst per-sample relative
    error of the coarse solution against the plain path."""
    import numpy as np
    import torch

    from paper_1607_00693_amd import stomsfem as sm
    from paper_1607_00693_amd import workloads as W

    wl = W.MESH8
    out = {}

    def coarse_err(Sa, Sb):
        Ua, _, _ = sm.coarse_solve(Sa, wl.nc, wl.nc)
        Ub, _, _ = sm.coarse_solve(Sb, wl.nc, wl.nc)
        d = torch.linalg.norm(Ua - Ub, dim=1) / torch.linalg.norm(Ub, dim=1)
        return float(d.max().item())

    # --- reduced basis ---
    N = 16384
    xi_tr = torch.from_numpy(W.uniform_xi(256, wl.nxi, 2003)).cuda()
    a_tr = sm.coef_bumps(xi_tr, wl.nfine, **wl.coef_params())
    t0 = time.perf_counter()
    model = sm.reduce(a_tr, wl.nc, wl.nc, wl.m, r_max=8, tail_tol=1e-6)
    t_off = time.perf_counter() - t0
    xi = torch.from_numpy(W.uniform_xi(N, wl.nxi, 1003)).cuda()
    a32 = sm.coef_bumps(xi, wl.nfine, **wl.coef_params(), dtype=torch.float32)
    S_rb = torch.empty((N, wl.M, 10), dtype=torch.float64, device="cuda")
    S_pl = torch.empty_like(S_rb)
    t_rb = _timed(lambda: sm.reduce_apply(model, a32, S=S_rb))
    t_pl = _timed(lambda: sm.upscale(a32, wl.nc, wl.nc, wl.m, S=S_pl))
    out["reduced_basis"] = {
        "workload": f"8x8 coarse, H/h=8, 256 training samples, r<=8 (tail 1e-6), {N} online samples, FP32 a",
        "offline_s": t_off, "r": int(model.export("r").max()),
        "pairs_per_s": N * wl.M / t_rb, "plain_pairs_per_s": N * wl.M / t_pl, "ratio": t_pl / t_rb,
        "max_coarse_rel_err": coarse_err(S_rb, S_pl)}
    log(f"reduced basis: {out['reduced_basis']}")
    model.free()
    del a_tr, a32

    # --- random interpolation at the same mesh and samples (FP64 a for the plain side) ---
    a64 = sm.coef_bumps(xi, wl.nfine, **wl.coef_params())
    S_pl = sm.upscale(a64, wl.nc, wl.nc, wl.m)
    t_pl = _timed(lambda: (sm.coef_bumps(xi, wl.nfine, **wl.coef_params(), out=a64),
                           sm.upscale(a64, wl.nc, wl.nc, wl.m, S=S_pl)))
    out["random_interpolation"] = measure_interpolation(wl, xi, S_pl, t_pl * 1e3, (5, 7), log, sg_levels=(4, 5))
    out["random_interpolation"]["workload"] = (f"8x8 coarse, H/h=8, {N} samples, Chebyshev-Lobatto tensor "
                                               "nodes per local variable (k<=4), FP64")
    del a64

    # --- learned surrogate ---
    fam = sm.bump_family(wl)
    lv, _ = sm.local_vars_bumps(wl.nc, wl.nc, wl.m, fam)
    mdl = sm.mlp_create(wl.nc, wl.nc, wl.m, lv, W.mlp_init(wl.M, 4004), fam, 1.0)
    ntr = 2048
    t0 = time.perf_counter()
    xi_tr = torch.from_numpy(W.uniform_xi(ntr, wl.nxi, 2004)).cuda()
    S_tr = sm.upscale(sm.coef_bumps(xi_tr, wl.nfine, **wl.coef_params()), wl.nc, wl.nc, wl.m)
    sm.mlp_set_data(mdl, xi_tr, S_tr)
    perm = torch.from_numpy(W.permutation(ntr, 5004)).cuda()
    for steps, lr in ((8000, 2e-3), (8000, 5e-4), (8000, 1e-4)):
        sm.mlp_train(mdl, steps, lr, perm)
    torch.cuda.synchronize()
    t_train = time.perf_counter() - t0
    N = 65536
    xi = torch.from_numpy(W.uniform_xi(N, wl.nxi, 1004)).cuda()
    a = torch.empty((N, wl.nfine, wl.nfine), dtype=torch.float64, device="cuda")
    S_pl = torch.empty((N, wl.M, 10), dtype=torch.float64, device="cuda")
    S_su = torch.empty_like(S_pl)
    status = torch.empty((N, wl.M), dtype=torch.int32, device="cuda")

    def plain():
        sm.coef_bumps(xi, wl.nfine, **wl.coef_params(), out=a)
        sm.upscale(a, wl.nc, wl.nc, wl.m, S=S_pl)

    t_pl = _timed(plain)
    t_su = _timed(lambda: sm.upscale_surrogate(mdl, xi, 1e-3, sm.PREC_BF16, S=S_su, status=status))
    st = status.cpu().numpy()
    err_b = coarse_err(S_su, S_pl)
    # the FP16 single-term kernel on the same networks and samples
    t_h = _timed(lambda: sm.upscale_surrogate(mdl, xi, 1e-3, sm.PREC_F16, S=S_su, status=status))
    sth = status.cpu().numpy()
    out["learned_surrogate"] = {
        "workload": f"8x8 coarse, H/h=8, 64 per-patch MLPs (k<=4 -> 64x3 -> 2x10, GELU), {ntr} training "
                    f"samples/patch, {N} test samples, gate tau=1e-3, BF16 MFMA (3-term split)",
        "train_s": t_train, "pairs_per_s": N * wl.M / t_su, "plain_pairs_per_s": N * wl.M / t_pl,
        "ratio": t_pl / t_su, "accepted": float((st == 0).mean()), "fallback": float((st == 1).mean()),
        "audited": float((st == 2).mean()), "max_coarse_rel_err": err_b,
        "fp16_single_term": {"pairs_per_s": N * wl.M / t_h, "ratio": t_pl / t_h,
                             "accepted": float((sth == 0).mean()), "fallback": float((sth == 1).mean()),
                             "audited": float((sth == 2).mean()), "max_coarse_rel_err": coarse_err(S_su, S_pl)}}
    log(f"learned surrogate: {out['learned_surrogate']}")
    mdl.free()
    return out


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--workload", default="mesh32", choices=["mesh32", "mesh8"])
    ap.add_argument("--nsamples", type=int, default=0, help="override the sample count (0 = workload default)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-accelerations", action="store_true", help="skip the reduced-basis / surrogate comparison")
    ap.add_argument("--only", default="",
                    help="comma-separated subset of the extra measurements (ri_bench, rb_bench, two_level_bench, surrogate_bench, "
                         "mixed_bench, mesh8, coarse_bench, queue, channels, channels_surrogate, oversampling, oversampling_large, rb_os_sec52, rb_os_channels, "
                         "collocation, "
                         "two_level, gauss, gauss_paper_mesh); "
                         "default: all of them")
    ap.add_argument("--calib-copy", action="store_true",
                    help="run one 1 GiB device copy first (calibrates HBM byte counters in a profile)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(json.dumps({"error": "this build runs on one GPU only; --gpus must be 1 "
                          "(sharding over samples is described in the design notes)"}))
        sys.exit(2)

    import dataclasses

    import torch

    from paper_1607_00693_amd import stomsfem
    from paper_1607_00693_amd import workloads as W

    wl = W.MESH32 if args.workload == "mesh32" else W.MESH8
    if args.nsamples:
        wl = dataclasses.replace(wl, nsamples=args.nsamples)
    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    stream = torch.cuda.current_stream()

    xi = torch.from_numpy(W.uniform_xi(wl.nsamples, wl.nxi, wl.seed)).to(dev)
    a = torch.empty((wl.nsamples, wl.nfine, wl.nfine), dtype=torch.float64, device=dev)
    S = torch.empty((wl.nsamples, wl.M, 10), dtype=torch.float64, device=dev)
    nU = (wl.nc - 1) ** 2
    U = torch.empty((wl.nsamples, nU), dtype=torch.float64, device=dev)
    qm = torch.empty(nU, dtype=torch.float64, device=dev)
    qv = torch.empty(nU, dtype=torch.float64, device=dev)
    status = torch.empty((wl.nsamples, wl.M), dtype=torch.int32, device=dev)

    ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]

    def step(record):
        if record:
            ev[0].record(stream)
        stomsfem.coef_bumps(xi, wl.nfine, **wl.coef_params(), out=a, stream=stream)
        if record:
            ev[1].record(stream)
        stomsfem.upscale(a, wl.nc, wl.nc, wl.m, S=S, status=status, stream=stream)
        if record:
            ev[2].record(stream)
        stomsfem.coarse_solve(S, wl.nc, wl.nc, U=U, qoi_mean=qm, qoi_var=qv, stream=stream)
        if record:
            ev[3].record(stream)

    if args.calib_copy:
        src = torch.empty(1 << 27, dtype=torch.float64, device=dev)
        dst = torch.empty_like(src)
        dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst
    # the project's autotuner picks the launch shape (and checks the refined
    # FP32 variant) for this batch before anything is timed
    stomsfem.coef_bumps(xi, wl.nfine, **wl.coef_params(), out=a, stream=stream)
    tuning = stomsfem.autotune(a, wl.nc, wl.nc, wl.m, S=S, reps=2)
    print(f"[bench] autotune: {tuning}", file=sys.stderr, flush=True)
    for _ in range(args.warmup):
        step(False)
    torch.cuda.synchronize()
    print(f"[bench] warmup done ({args.warmup} steps)", file=sys.stderr, flush=True)

    t_gen = t_up = t_co = 0.0
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for k in range(args.steps):
        step(True)
        ev[3].synchronize()
        t_gen += ev[0].elapsed_time(ev[1])
        t_up += ev[1].elapsed_time(ev[2])
        t_co += ev[2].elapsed_time(ev[3])
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    bad = int((status != 0).sum().item())
    ms = (t1 - t0) * 1000.0 / args.steps
    pairs = wl.nsamples * wl.M
    t_up /= args.steps
    t_gen /= args.steps
    t_co /= args.steps
    flops = plain_flops_per_pair(wl.m) * pairs
    achieved = flops / (t_up * 1e-3) / 1e12
    bytes_alg = pairs * (wl.m * wl.m * 8 + 10 * 8 + 4)
    print(f"[bench] {args.steps} steps: {ms:.2f} ms/step (gen {t_gen:.2f}, upscale {t_up:.2f}, coarse {t_co:.2f} ms),"
          f" non-OK pairs {bad}", file=sys.stderr, flush=True)

    # the same step captured once in a HIP graph (an execution plan of one
    # stage: coefficient generation, upscaling, coarse solve and QoI) and
    # replayed: its time per step and its QoI against the eager step's
    qm_e = qm.clone()
    qm_p = torch.empty_like(qm)
    plan = stomsfem.plan_create([stomsfem.make_stage(wl.nc, wl.m, xi, bumps=stomsfem.bump_family(wl),
                                                     qoi_mean=qm_p)])
    plan.launch(-1, stream)
    torch.cuda.synchronize()
    ev[0].record(stream)
    for _ in range(3):
        plan.launch(-1, stream)
    ev[1].record(stream)
    ev[1].synchronize()
    t_graph = ev[0].elapsed_time(ev[1]) / 3
    graph = {"ms_per_step": t_graph, "pairs_per_s": pairs / (t_graph * 1e-3),
             "qoi_mean_equal_to_eager": bool(torch.equal(qm_p, qm_e))}
    plan.free()
    print(f"[bench] graph-captured step: {graph}", file=sys.stderr, flush=True)

    out = {
        "metric": "upscaled (patch x sample)/s, plain FP64 path",
        "value": pairs / (ms * 1e-3),
        "unit": "pairs/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64",
        "data": "synthetic",
        "config": {
            "workload": f"{wl.name}: {wl.nc}x{wl.nc} coarse, H/h={wl.m}, {wl.nsamples} samples, "
                        f"{wl.nxi} bumps (xi~U[-1,1]), f=1, zero Dirichlet",
            "nc": wl.nc, "m": wl.m, "nsamples": wl.nsamples, "pairs": pairs,
        },
        "kernel_ms": {"coef_bumps": t_gen, "upscale": t_up, "coarse_solve_qoi": t_co},
        "graph_captured_step": graph,
        "tuning": tuning,
        "roofline": {
            "bound": "alu",
            "achieved": achieved,
            "peak": FP64_VALU_PEAK_TFLOPS,
            "unit": "TFLOP/s",
            "frac": achieved / FP64_VALU_PEAK_TFLOPS,
            "traffic": (None if (tpp := profiled_traffic_per_pair()) is None or wl.m != 32 else tpp * pairs),
            "traffic_unit": "bytes per launch (rocprofv3 FETCH_SIZE + WRITE_SIZE, copy-calibrated)",
            "algorithmic_bytes": bytes_alg,
            "kernel": "local upscaling (FP64 VALU)",
            "flops_per_pair": plain_flops_per_pair(wl.m),
            "frac_with_scope_table_count": survey_flops_per_pair(wl.m) * pairs / (t_up * 1e-3) / 1e12
                                           / FP64_VALU_PEAK_TFLOPS,
            "scope_table_flops_per_pair": survey_flops_per_pair(wl.m),
            "hbm_frac_algorithmic": bytes_alg / (t_up * 1e-3) / 1e9 / HBM_PEAK_GBS,
        },
        "cpu_baseline": None,
    }
    if not args.no_accelerations:
        lg = lambda m: print(f"[bench] {m}", file=sys.stderr, flush=True)  # noqa: E731
        only = set(x for x in args.only.split(",") if x)
        want = lambda name: not only or name in only  # noqa: E731
        acc = {}
        if want("ri_bench"):
            lg("random interpolation at the benchmark mesh")
            ri_out = measure_interpolation(wl, xi, S, t_gen + t_up, (5, 7), lg, sg_levels=(4, 5))
            ri_out["workload"] = (f"{wl.nc}x{wl.nc} coarse, H/h={wl.m}, {wl.nsamples} samples (the benchmark's xi), "
                                  "Chebyshev-Lobatto tensor nodes per local variable (k<=4) and Smolyak "
                                  "Clenshaw-Curtis sparse grids, FP64; plain side = coefficient generation + "
                                  "upscaling kernels")
            acc["random_interpolation_bench_mesh"] = ri_out
        if want("rb_bench"):
            lg("reduced basis at the benchmark mesh")
            acc["reduced_basis_bench_mesh"] = measure_reduced_basis(wl, xi, S, t_gen + t_up, lg)
        if want("two_level_bench"):
            lg("two-level Monte Carlo at the benchmark mesh")
            acc["two_level_mc_bench_mesh"] = measure_two_level_bench(wl, S, lg)
        if want("surrogate_bench"):
            lg("learned surrogate at the benchmark mesh")
            acc["learned_surrogate_bench_mesh"] = measure_surrogate(wl, xi, S, t_gen + t_up, lg)
        if want("mixed_bench"):
            lg("FP32 factorisation + FP64 refinement on the first 64 samples")
            ns = min(64, wl.nsamples)
            a_sub, S_sub = a[:ns], S[:ns]
            S_mx = torch.empty_like(S_sub)
            st_mx = torch.empty((ns, wl.M), dtype=torch.int32, device=dev)
            t_mx = _timed(lambda: stomsfem.upscale(a_sub, wl.nc, wl.nc, wl.m, S=S_mx, status=st_mx,
                                                   precision=stomsfem.PREC_F32_REFINE64), reps=2)
            S_64 = torch.empty_like(S_sub)
            t_64 = _timed(lambda: stomsfem.upscale(a_sub, wl.nc, wl.nc, wl.m, S=S_64), reps=2)
            mixed = {"workload": f"first {ns} samples of the benchmark batch ({ns * wl.M} pairs)",
                     "pairs_per_s": ns * wl.M / t_mx, "fp64_pairs_per_s": ns * wl.M / t_64, "ratio": t_64 / t_mx,
                     "recomputed_fp64": int((st_mx == 1).sum().item()),
                     "max_S_rel_err_vs_fp64": float(((S_mx - S_64).abs().amax(dim=2)
                                                     / S_64.abs().amax(dim=2)).max())}
            lg(f"fp32+refinement: {mixed}")
            acc["fp32_solve_fp64_refinement_bench_mesh"] = mixed
        del a
        torch.cuda.empty_cache()
        if want("mesh8"):
            lg("reduced basis, interpolation and learned surrogate at the 8x8 mesh")
            acc.update(measure_accelerations(lg))
        out["accelerations"] = acc
        if want("coarse_bench"):
            lg("batched coarse solve at 64x64, 48x48, 33x33")
            out["coarse_solve_bench"] = measure_coarse(lg)
        if want("queue"):
            lg("mixed H/h: per-m kernels (sequential, concurrent streams) against one persistent launch")
            out["mixed_m_persistent_launch"] = measure_queue(lg)
        chan = None
        if want("channels"):
            lg("channels-and-inclusions workload through a graph plan")
            chan = measure_channels(lg)
            out["channels64_plan"] = {k: v for k, v in chan.items() if not k.startswith("_")}
        if want("channels_surrogate"):
            lg("channels-and-inclusions workload with the learned surrogate")
            out["channels64_surrogate"] = measure_channels_surrogate(lg, chan)
        if want("oversampling"):
            lg("oversampled Petrov-Galerkin upscaling at the 8x8 mesh")
            out["oversampled_petrov_galerkin"] = measure_oversampling(lg)
        if want("oversampling_large"):
            lg("oversampled Petrov-Galerkin upscaling with patches of 48 to 64 cells")
            out["oversampled_large_patches"] = measure_oversampling_large(lg)
        if want("rb_os_sec52"):
            lg("reduced basis on oversampled patches, Sec. 5.2 geometry")
            out["reduced_basis_oversampled_sec52"] = measure_rb_os_sec52(lg)
        if want("rb_os_channels"):
            lg("reduced basis on oversampled patches in the channels medium")
            out["reduced_basis_oversampled_channels"] = measure_rb_os_channels(lg)
        if want("collocation"):
            lg("sparse-grid collocation with dictionaries at the 8x8 mesh")
            from paper_1607_00693_amd import workloads as W
            out["sparse_grid_collocation"] = {"mesh8_level4": measure_collocation(lg, plain_chunk=1 << 20),
                                              "bench_mesh_level2": measure_collocation(lg, W.MESH32, 2, errors=False)}
        if want("two_level"):
            lg("two-level Monte Carlo at the 8x8 mesh")
            out["two_level_mc"] = measure_two_level(lg)
        if want("gauss"):
            lg("Gaussian medium and local KL")
            out["gaussian_local_kl"] = measure_gauss(lg)
        if want("gauss_paper_mesh"):
            lg("Gaussian medium on the paper's h = 2^-11 mesh with 64-cell oversampled patches")
            out["gaussian_paper_mesh"] = measure_gauss_paper_mesh(lg)
    if not args.no_cpu_baseline:
        print("[bench] timing the CPU oracle on a bounded sample", file=sys.stderr, flush=True)
        out["cpu_baseline"] = cpu_baseline(wl)
    print(json.dumps(out))


if __name__ == "__main__":
    main()
