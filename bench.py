#!/usr/bin/env python3
"""Training-step benchmark of the Defrise-Clack FBP path on one MI355X.

Workload (C2): sinusoidal orbit (source elevation amplitude 100 mm, 2 periods),
496 views, SID 750 / SDD 1200 mm, 512 x 512 detector at 0.6 mm, Radon grid
360 angles x 725 bins, 256^3 volume at 0.5 mm.  Data: 20 seeded random
ellipsoids, exact line integrals, Poisson noise at 1e5 photons per ray; target =
the voxelised phantom.  One step = forward (weighted Radon, filter, detector BP,
cone BP + ReLU), MSE loss gradient, backward through every adjoint kernel to
dL/dM, and an Adam update of M.  All inputs are resident in HBM before timing.

``--orbit circle`` runs the same grid on a 496-view circular orbit instead
(the cone stages then take their z-invariant form); the default is the
sinusoidal workload above.

Prints one JSON line: voxel-view updates per second (Nvox x V / step time) for
float32 storage (``value``) and bf16 storage of H / gF (``bf16``), per-kernel
times, the dominant kernel's roofline and the CPU oracle baseline.
"""
from __future__ import annotations

import argparse
import glob
import hashlib
import json
import math
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "voxel-view updates/s (fwd+bwd DC-FBP) at 256³; % HBM roofline; BF16 vs FP32"
HBM_PEAK_GBS = 8000.0
# float32 vector peak: 256 CU x 4 SIMD x 32 lanes/clk x 2 flops (FMA) x 2.4 GHz = 157.3 TFLOP/s;
# gfx950 issues a wave64 float32 VALU op in 2 cycles without packed math (measured)
FP32_PEAK_TFLOPS = 157.3

# algorithmic work per unit (flops) of each stage: pixel-angle pairs for the 2D
# stages, voxel-view pairs for the cone stages, sinogram bins for the filter
FLOPS_PER_UNIT = {"weight_radon": 9, "filter": 10, "detector_bp": 9, "cone_bp": 23,
                  "cone_bp_adjoint": 23, "detector_bp_adjoint": 9, "filter_adjoint": 10}
# LDS bytes per unit the algorithms move: one 8-byte (c, s) read per pixel-angle
# (interp), four 4-byte taps per voxel-view (cone BP), two 8-byte atomics per voxel-view
# (cone transpose), a row staged once per bin (filters, written and read); the gathers of
# the two Radon stages add three 4-byte sums per 16 rows of a column and angle, and the
# exact form reads one fraction per pixel-angle of four views.  Against 128 B per clock per
# CU (the CDNA3 LDS figure; no CDNA4 one is published), 78.6 TB/s over 256 CUs.
LDS_BYTES_PER_UNIT = {"weight_radon": 1.75, "filter": 8, "detector_bp": 8, "cone_bp": 16,
                      "cone_bp_adjoint": 16, "detector_bp_adjoint": 0.75, "filter_adjoint": 8}
LDS_PEAK_TBS = 256 * 128 * 2.4e9 / 1e12
# The Radon gathers are bound by vector instructions: wave instructions per 64
# pixel-angles from SQ_INSTS_VALU (the exact form: the weighted Radon, and the detector
# Radon stored in 16 bits; the float form: the detector Radon in float32), against the
# 1.7 per clock per CU that plain float32 instructions reach.
VALU_PER_UNIT = {"exact": 6.1, "float": 3.4}
VALU_PEAK_PER_CLK = 1.7


# HBM bytes per call of a stage, from FETCH_SIZE and WRITE_SIZE counter runs of this
# script (each scaled by what the counter reads for a 1 GiB copy; summaries in
# profiles/c2_<dtype>_hbm_traffic.md).  A figure holds only for the kernel sources it
# was measured on, identified by the digest of the stage's kernel sources (the file
# holding its kernels and launcher, and the shared internal header); after any change
# to them the roofline reports traffic as null until the counters are taken again.
STAGE_SOURCES = {
    "weight_radon": ("radon2d.hip", "splat_shear.hip"), "detector_bp": ("radon2d.hip",),
    "detector_bp_adjoint": ("radon2d.hip", "splat_shear.hip"),
    "filter": ("filter.hip",), "filter_adjoint": ("filter.hip",),
    "cone_bp": ("cone.hip",), "cone_bp_adjoint": ("cone.hip",),
}
MEASURED_TRAFFIC = {
    # (stage, storage dtype): (bytes per call, digest of the stage's kernel sources)
    ("cone_bp_adjoint", "f32"): (3_094_738_906 + 693_083_832,
                                 "ce2aba7cc86a44f5c5cac9d9caf9d50587afe4da7f93e755d12371c08a80aba9"),
    ("weight_radon", "f32"): (4_687_652_825 + 1_690_618_224,
                              "b9b97c4a4be6e5de3b802f2b8afa820a944e74f46d16ccbded62cddc1886ad5d"),
}


def kernel_sources_digest(stage):
    """sha256 over the names and bytes of the stage's kernel sources and dc_internal.h."""
    h = hashlib.sha256()
    for name in sorted(STAGE_SOURCES[stage] + ("dc_internal.h",)):
        h.update(name.encode())
        with open(os.path.join(ROOT, "paper_2410_14900_amd", "csrc", name), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()


def valu_issue(stage, store, units, t):
    """Vector instruction issue of a Radon stage's gather of `units` pixel-angles that
    takes t seconds (nothing for the other stages)."""
    if stage not in ("weight_radon", "detector_bp_adjoint"):
        return {}
    form = "float" if stage == "detector_bp_adjoint" and store == "f32" else "exact"
    rate = VALU_PER_UNIT[form] * units / 64.0 / (t * 256 * 2.4e9)
    return {"valu_per_unit": VALU_PER_UNIT[form], "valu_per_clk_cu": round(rate, 2),
            "valu_frac": round(rate / VALU_PEAK_PER_CLK, 3)}


def log(*a):
    print("[bench]", *a, file=sys.stderr, flush=True)


def stage_work(g, V, bpe_store):
    """(units, algorithmic HBM bytes) per launch over all V views."""
    npix, nbin, nvox = g.nu * g.nv, g.n_theta * g.n_s, g.nx * g.ny * g.nz
    pa = V * npix * g.n_theta            # pixel-angle pairs
    vv = V * nvox                        # voxel-view pairs
    return {
        "weight_radon": (pa, V * npix * 4 + V * nbin * 4),
        "filter": (V * nbin, V * nbin * (4 + 4 + bpe_store)),
        "detector_bp": (pa, V * nbin * bpe_store + V * npix * bpe_store),
        "cone_bp": (vv, V * npix * bpe_store + nvox * 4),
        "cone_bp_adjoint": (vv, nvox * 4 * 2 + V * npix * bpe_store),
        "detector_bp_adjoint": (pa, V * npix * bpe_store + V * nbin * bpe_store),
        "filter_adjoint": (V * nbin, V * nbin * (bpe_store + 4 + 4)),
    }


SLABS = 16   # the oracle worker's 3D stages run on one z-slab of 1/SLABS of the volume


def _oracle_step(args):
    """One view's forward + backward step of the float64 oracle (a worker of
    cpu_baseline), its 3D stages on one z-slab of the volume.  Returns (seconds
    of the 2D stages, seconds of the 3D stages on the slab)."""
    grid, sub, slab = args
    import numpy as np
    from threadpoolctl import threadpool_limits
    from oracle import pipeline as O
    with threadpool_limits(1):
        rng = np.random.Generator(np.random.PCG64(0))
        g = rng.uniform(0, 1, (1, grid.nv, grid.nu))
        M = np.full((1, grid.n_theta, grid.n_s), 0.5)
        nz = grid.nz // SLABS
        zz, yy, xx = np.meshgrid(np.arange(slab * nz, (slab + 1) * nz), np.arange(grid.ny), np.arange(grid.nx),
                                 indexing="ij")
        idx = np.stack([zz.ravel(), yy.ravel(), xx.ravel()], axis=1)
        t0 = time.perf_counter()
        R = O.weight_radon(g, grid, sub)
        H = O.filter_stack(R, M, grid, sub)
        gF = O.detector_bp(H, grid)
        t1 = time.perf_counter()
        f = O.cone_bp(gF, grid, sub, relu=True, points=O.voxel_centres(grid, idx))
        GgF = O.cone_bp_adjoint(f, grid, sub, relu_f=f, support=idx)
        t2 = time.perf_counter()
        GH = O.detector_bp_adjoint(GgF, grid)
        O.filter_stack_adjoint(GH, R, M, grid, sub)
        t3 = time.perf_counter()
        return (t1 - t0) + (t3 - t2), t2 - t1


def host_cpu():
    """(usable cores, logical CPUs, model name) of this host."""
    usable = len(os.sched_getaffinity(0)) if hasattr(os, "sched_getaffinity") else os.cpu_count()
    model = ""
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    return usable, os.cpu_count(), model


def cpu_baseline(grid, views, max_workers=16):
    """Times the float64 oracle on a bounded sample of the same step: one worker
    process per usable host core (at most max_workers, BLAS held to one thread
    each), all running at once.  Each runs one view's forward + backward (views
    spread over the orbit) with the 2D stages at full size and the two 3D stages
    on one z-slab of 1/16 of the 256^3 volume (their work is linear in the voxel
    count), so a worker's step time for a whole view is t_2D + 16 t_slab.  Run
    before the GPU is touched, so the workers are plain forks."""
    import multiprocessing as mp
    usable, logical, model = host_cpu()
    W = max(1, min(max_workers, usable))
    picks = [int(round(i * len(views) / W)) % len(views) for i in range(W)]
    jobs = [(grid, views.subset([v]), i % SLABS) for i, v in enumerate(picks)]
    t0 = time.perf_counter()
    with mp.get_context("fork").Pool(W) as pool:
        per = pool.map(_oracle_step, jobs)
    wall = time.perf_counter() - t0
    nvox = grid.nx * grid.ny * grid.nz
    step = [t2d + SLABS * t3d for t2d, t3d in per]           # seconds per whole view, per worker
    rate = sum(nvox / t for t in step)                         # all workers together
    return {"value": rate, "unit": "voxel-view updates/s", "cores": W, "kind": "oracle",
            "host": {"usable_cores": usable, "logical_cpus": logical, "cpu_model": model},
            "sample": "%d worker processes at once (BLAS 1 thread each), each one view of the same forward+backward "
                      "step: 2D stages at full size (512^2 detector, 360x725 sinogram), the 3D stages on a 1/%d z-slab "
                      "of the 256^3 volume scaled by %d; float64 NumPy; %.1f s wall; per view %.1f s (2D %.1f s + 3D "
                      "%.1f s)" % (W, SLABS, SLABS, wall, sum(step) / W, sum(p[0] for p in per) / W,
                                   SLABS * sum(p[1] for p in per) / W)}


def adam_(M, G, m, v, t, lr=1e-2, b1=0.9, b2=0.999, eps=1e-8):
    """Adam update of M in place from gradient G: the step count t (a float32 device
    scalar) is advanced, then the library's fused update runs (one pass over the
    arrays; both can sit in a captured graph)."""
    import paper_2410_14900_amd as P
    t.add_(1.0)
    P.dc_adam_step(M, G, m, v, t, lr, (b1, b2), eps)


class Trainer:
    """One training step of the DC-FBP network over a plan (one scan or a batch):
    R = A2d(w_cos g), H = D(W D R), gF = A2d^T H, f = ReLU(cone BP), the MSE
    gradient, the adjoint chain to dL/dM and an Adam update of M.  Buffers are
    allocated once, so the step can be captured in a graph."""

    STAGES = ["weight_radon", "filter", "detector_bp", "cone_bp", "cone_bp_adjoint", "detector_bp_adjoint",
              "filter_adjoint"]
    SMOOTH_STAGES = ["smooth", "smooth_adjoint"]

    def __init__(self, P, plan, g, target, store, smooth=None, keep_R=False):
        import torch
        self.P, self.plan, self.g, self.target = P, plan, g, target
        V, (K, S), det = plan.n_views, plan.sino_shape, plan.det_shape
        dev = g.device
        self.R = torch.empty((V, K, S), device=dev)
        self.H = torch.empty((V, K, S), device=dev, dtype=store)
        self.gF = torch.empty((V,) + det, device=dev, dtype=store)
        self.f = torch.empty(plan.vol_shape, device=dev)
        self.Gf = torch.empty_like(self.f)
        self.GgF = torch.empty_like(self.gF)
        self.GH = torch.empty_like(self.H)
        self.M = torch.full((V, K, S), 0.5, device=dev)
        self.GM = torch.empty_like(self.M)
        self.m, self.v = torch.zeros_like(self.M), torch.zeros_like(self.M)
        self.t = torch.zeros((), device=dev)
        self.gscale = 2.0 / target.numel()
        # the Gaussian filter layer on the weight (sigma, radius), applied before use
        self.smooth = smooth
        self.Mw = torch.empty_like(self.M) if smooth else self.M
        # R depends only on the projections: with keep_R it is formed once here and
        # the step starts at the filter
        self.keep_R = keep_R
        if keep_R:
            P.dc_weight_radon(plan, g, self.R)

    def step(self, timed=None):
        import torch
        P, pl = self.P, self.plan
        run = timed or (lambda name, fn: fn())
        if not self.keep_R:
            run("weight_radon", lambda: P.dc_weight_radon(pl, self.g, self.R))
        if self.smooth:
            run("smooth", lambda: P.dc_smooth_weights(pl, self.M, self.Mw, *self.smooth))
        run("filter", lambda: P.dc_filter(pl, self.R, self.Mw, self.H))
        run("detector_bp", lambda: P.dc_detector_bp(pl, self.H, self.gF))
        run("cone_bp", lambda: P.dc_cone_bp(pl, self.gF, self.f, relu=True))
        torch.sub(self.f, self.target, out=self.Gf)
        self.Gf.mul_(self.gscale)
        run("cone_bp_adjoint", lambda: P.dc_cone_bp_adjoint(pl, self.Gf, self.GgF, f_relu=self.f))
        run("detector_bp_adjoint", lambda: P.dc_detector_bp_adjoint(pl, self.GgF, self.GH))
        run("filter_adjoint", lambda: P.dc_filter_adjoint(pl, self.GH, self.R, self.Mw, GM=self.GM))
        if self.smooth:
            run("smooth_adjoint", lambda: P.dc_smooth_weights_adjoint(pl, self.GM, self.GM, *self.smooth))
        adam_(self.M, self.GM, self.m, self.v, self.t)

    def rel_error(self):
        """Relative L2 error of the current reconstruction against the phantom."""
        d = (self.f - self.target).double()
        return float(d.norm() / self.target.double().norm())


def time_eager(trainers, steps, warmup, per_stage=False):
    """ms per step of running every trainer's step once, eagerly; optional per-stage event times."""
    import torch
    stream = torch.cuda.current_stream()
    ev = {s: [] for s in Trainer.STAGES + Trainer.SMOOTH_STAGES}

    def timed(name, fn):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record(stream)
        fn()
        b.record(stream)
        ev[name].append((a, b))

    for _ in range(warmup):
        for tr in trainers:
            tr.step()
    torch.cuda.synchronize()
    start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    start.record(stream)
    for _ in range(steps):
        for tr in trainers:
            tr.step(timed if per_stage else None)
    end.record(stream)
    torch.cuda.synchronize()
    ms = start.elapsed_time(end) / steps
    kern = ({s: sum(a.elapsed_time(b) for a, b in ev[s]) / len(ev[s]) for s in ev if ev[s]}
            if per_stage else None)
    return ms, kern


def time_graph(trainer, steps, warmup):
    """ms per step of replaying the trainer's step captured in one HIP graph."""
    import torch
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        trainer.step()                       # warm-up on a side stream before capture
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        trainer.step()
    for _ in range(max(0, warmup - 1)):
        graph.replay()
    torch.cuda.synchronize()
    stream = torch.cuda.current_stream()
    start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    start.record(stream)
    for _ in range(steps):
        graph.replay()
    end.record(stream)
    torch.cuda.synchronize()
    return start.elapsed_time(end) / steps, graph


def batched_c4(P, synth, args):
    """The batched workload: 8 scans with mixed orbits (3002 views) on the C2 grid.
    FP32 storage with one plan per scan run eagerly, against BF16 storage with one
    batched plan whose whole step is one captured graph; same data, same number of
    steps, reconstruction error of both against the phantoms."""
    import torch
    grid, sets, seeds = synth.c4_scans()
    nvox = grid.nx * grid.ny * grid.nz
    gs, targets = [], []
    for views, seed in zip(sets, seeds):
        ell = synth.random_ellipsoids(20, grid.nx * grid.vx, seed)
        gs.append(synth.project_ellipsoids(ell, grid, views, device="cuda").float().contiguous())
        targets.append(synth.voxelize_torch(ell, grid, device="cuda"))
    Vt = sum(len(v) for v in sets)
    log("C4 inputs ready:", [len(v) for v in sets], "views")
    plans = [P.Plan(grid, v) for v in sets]
    if not args.no_autotune:
        for pl in plans:
            pl.autotune()
    singles = [Trainer(P, pl, g, t, torch.float32) for pl, g, t in zip(plans, gs, targets)]
    ms32, _ = time_eager(singles, args.batched_steps, args.warmup)
    err32 = sum(tr.rel_error() for tr in singles) / len(singles)
    log("C4 fp32 per-scan eager: %.2f ms/step, mean relative error %.5f" % (ms32, err32))
    del singles, plans
    torch.cuda.empty_cache()
    plan = P.Plan.batched(grid, sets)
    batched_knobs = plan.autotune()["knobs"] if not args.no_autotune else plan.knobs()
    g = torch.cat(gs)
    del gs
    tb = Trainer(P, plan, g, torch.stack(targets), torch.bfloat16)
    # one eager warm-up step, warmup - 1 untimed and `steps` timed replays: both forms
    # have taken warmup + steps Adam steps when their errors are compared
    msbg, _graph = time_graph(tb, args.batched_steps, args.warmup)
    errbg = sum(float((tb.f[s] - tb.target[s]).double().norm() / tb.target[s].double().norm())
                for s in range(plan.n_samples)) / plan.n_samples
    log("C4 bf16 batched graph: %.2f ms/step, mean relative error %.5f" % (msbg, errbg))
    return {
        "workload": "C4: 8 scans on the C2 grid (circle 248/496/372, sinusoid 496/248/372, circle+arc 100+360 "
                    "and 60+250 views; 3002 views), 20 seeded ellipsoids each, no noise",
        "views": Vt, "samples": len(sets),
        "fp32_per_scan_eager": {"value": nvox * Vt / (ms32 * 1e-3), "ms_per_step": round(ms32, 3),
                                "mean_rel_error": round(err32, 6)},
        "bf16_batched_graph": {"value": nvox * Vt / (msbg * 1e-3), "ms_per_step": round(msbg, 3),
                               "mean_rel_error": round(errbg, 6)},
        "speedup": round(ms32 / msbg, 3),
        "batched_knobs": batched_knobs,
        "steps": args.batched_steps,
    }


def c3_line(P, synth, args):
    """The circle-plus-arc workload (C3: 100 arc views at +-30 degrees, then 360
    circle views; the C2 grid), the same training step in FP32 and in BF16
    storage, eagerly."""
    import torch
    c = synth.CONFIGS["C3"]
    grid, views = synth.config_geometry("C3")
    ell = synth.random_ellipsoids(c["n_ell"], grid.nx * grid.vx, c["seed"])
    g = synth.project_ellipsoids(ell, grid, views, device="cuda").float().contiguous()
    target = synth.voxelize_torch(ell, grid, device="cuda")
    plan = P.Plan(grid, views)
    knobs = plan.autotune() if not args.no_autotune else {"knobs": plan.knobs()}
    V, nvox = len(views), grid.nx * grid.ny * grid.nz
    out = {"knobs": knobs["knobs"], "workload": "C3: circle+arc orbit, 100 arc views (+-30 deg) then 360 circle views, 512x512 detector "
                       "@0.6 mm, Radon 360x725, 256^3 volume @0.5 mm, forward+backward w.r.t. M + Adam step",
           "views": V}
    for store, dt in (("f32", torch.float32), ("bf16", torch.bfloat16)):
        tr = Trainer(P, plan, g, target, dt)
        ms, kern = time_eager([tr], args.steps, args.warmup, per_stage=True)
        out[store] = {"value": nvox * V / (ms * 1e-3), "ms_per_step": round(ms, 3),
                      "kernels_ms": {k: round(v, 3) for k, v in kern.items()}, "rel_error": round(tr.rel_error(), 6)}
        log("C3 %s: %.2f ms/step" % (store, ms), json.dumps(out[store]["kernels_ms"]))
        del tr
        torch.cuda.empty_cache()
    return out


def shard_line(P, grid, views, g, target, args, n_gpus=8):
    """One GPU's share of a view-sharded C2 step: every n_gpus-th view (62 of 496)
    into the full 256^3 volume, the same forward+backward step timed as is.  A
    sharded step would sum the partial volumes with one all-reduce before the ReLU
    and the loss; that exchange is not run here (one GPU), only modelled."""
    import torch
    idx = list(range(0, len(views), n_gpus))
    sub = views.subset(idx)
    plan = P.Plan(grid, sub)
    knobs = plan.autotune() if not args.no_autotune else {"knobs": plan.knobs()}
    gs = g[idx].contiguous()
    tr = Trainer(P, plan, gs, target, torch.float32)
    ms, kern = time_eager([tr], args.steps, args.warmup, per_stage=True)
    nvox = grid.nx * grid.ny * grid.nz
    vol_bytes = 4 * nvox
    # ring all-reduce over n_gpus: each GPU sends and receives 2 (n-1)/n of the volume
    # over its busiest link (about 153 GB/s per xGMI link)
    ring_ms = 2 * (n_gpus - 1) / n_gpus * vol_bytes / 153e9 * 1e3
    out = {"workload": "one GPU's share of C2 sharded by view over %d GPUs: every %dth view (%d of %d), full 256^3 "
                       "volume, forward+backward w.r.t. M + Adam step, FP32 storage" % (n_gpus, n_gpus, len(idx), len(views)),
           "views": len(idx), "knobs": knobs["knobs"], "ms_per_step": round(ms, 3),
           "value": nvox * len(idx) / (ms * 1e-3),
           "kernels_ms": {k: round(v, 3) for k, v in kern.items()},
           "allreduce_model": {"bytes": vol_bytes, "single_ring_ms": round(ring_ms, 3),
                               "note": "modelled, not measured: one ring over one xGMI link per GPU"}}
    log("one GPU's view share (%d views): %.2f ms/step" % (len(idx), ms), json.dumps(out["kernels_ms"]))
    del tr
    torch.cuda.empty_cache()
    return out


def c5_line(P, synth, args):
    """The full C-arm scale workload (C5: 512^3 at 0.25 mm, 976^2 detector at
    0.308 mm, Radon 720 x 1381, 496-view sinusoid): the training step with FP16
    storage of the filtered sinograms and detector images, the Radon stack
    recomputed every step, with the plan's default knobs and with the autotuner's."""
    import torch
    c = synth.CONFIGS["C5"]
    grid, views = synth.config_geometry("C5")
    ell = synth.random_ellipsoids(c["n_ell"], grid.nx * grid.vx, c["seed"])
    g = synth.project_ellipsoids(ell, grid, views, device="cuda").float().contiguous()
    target = synth.voxelize_torch(ell, grid, device="cuda")
    plan = P.Plan(grid, views)
    V, nvox = len(views), grid.nx * grid.ny * grid.nz
    out = {"workload": "C5: sinusoidal orbit, 496 views, 976x976 detector @0.308 mm, Radon 720x1381, 512^3 volume "
                       "@0.25 mm, FP16 storage, Radon stack recomputed every step, forward+backward + Adam step",
           "views": V, "default_knobs": plan.knobs()}
    steps, warm = max(2, args.steps // 2), 1
    tr = Trainer(P, plan, g, target, torch.float16)
    ms, kern = time_eager([tr], steps, warm, per_stage=True)
    out["default"] = {"value": nvox * V / (ms * 1e-3), "ms_per_step": round(ms, 3),
                      "kernels_ms": {k: round(v, 3) for k, v in kern.items()}}
    log("C5 default knobs: %.2f ms/step" % ms, json.dumps(out["default"]["kernels_ms"]))
    if not args.no_autotune:
        out["tuned_knobs"] = plan.autotune()
        ms, kern = time_eager([tr], steps, warm, per_stage=True)
        out["tuned"] = {"value": nvox * V / (ms * 1e-3), "ms_per_step": round(ms, 3),
                        "kernels_ms": {k: round(v, 3) for k, v in kern.items()}}
        log("C5 tuned knobs %s: %.2f ms/step" % (json.dumps(out["tuned_knobs"]["knobs"]), ms),
            json.dumps(out["tuned"]["kernels_ms"]))
    out["rel_error"] = round(tr.rel_error(), 6)
    del tr
    torch.cuda.empty_cache()
    return out


# The paper's own timing of this method (its Table 4, sinusoidal orbit): one
# reconstruction with trained weights, forward only, on an NVIDIA RTX 4080 Super,
# against 197 s for 300 iterations of AIR (the abstract's "more than 97%").
PAPER_FORWARD_S = 4.5
PAPER_AIR_S = 197.0


def paper_workload_line(P, synth, args):
    """The paper's reconstruction workload (its Tables 1-2 and the sinusoidal-orbit
    section): a 128 x 512 x 512 volume at 0.25 mm from 400 views of a 620 x 480
    detector at 0.616 mm (SID 750 mm, SDD 1200 mm) on the sinusoid with a 20 degree
    maximum tilt and frequency 5, Radon 360 x 785.  One forward reconstruction
    (weighted Radon, filter, detector BP, cone BP + ReLU) on synthetic projections of
    that shape, timed with HIP events; the paper's own figure is quoted beside it as
    context (other hardware, its trained weights and data)."""
    import torch
    grid, views = synth.paper_geometry()
    plan = P.Plan(grid, views)
    if not args.no_autotune:
        plan.autotune()
    V, nvox = len(views), grid.nx * grid.ny * grid.nz
    gen = torch.Generator(device="cuda").manual_seed(5)
    g = torch.rand((V, grid.nv, grid.nu), device="cuda", generator=gen)
    M = torch.full((V,) + plan.sino_shape, 0.5, device="cuda")
    R = torch.empty((V,) + plan.sino_shape, device="cuda")
    H = torch.empty_like(R)
    gF = torch.empty_like(g)
    f = torch.empty(plan.vol_shape, device="cuda")

    def forward():
        P.dc_weight_radon(plan, g, R)
        P.dc_filter(plan, R, M, H)
        P.dc_detector_bp(plan, H, gF)
        P.dc_cone_bp(plan, gF, f, relu=True)

    for _ in range(max(1, args.warmup)):
        forward()
    torch.cuda.synchronize()
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    n = max(3, args.steps)
    a.record()
    for _ in range(n):
        forward()
    b.record()
    torch.cuda.synchronize()
    ms = a.elapsed_time(b) / n
    out = {"workload": "the paper's: sinusoidal orbit (20 deg, f = 5), 400 views, 620x480 detector @0.616 mm, "
                       "Radon 360x785, 128x512x512 volume @0.25 mm, one forward reconstruction",
           "knobs": plan.knobs(), "ms": round(ms, 3), "value": nvox * V / (ms * 1e-3), "unit": "voxel-view updates/s",
           "paper_context": {"seconds": PAPER_FORWARD_S, "gpu": "NVIDIA RTX 4080 Super",
                             "value": nvox * V / PAPER_FORWARD_S,
                             "air_seconds": PAPER_AIR_S,
                             "source": "the paper's Table 4 (forward with trained weights; 300 AIR iterations 197 s)"}}
    log("paper workload: %.2f ms per forward reconstruction (the paper: %.1f s on an RTX 4080 Super)"
        % (ms, PAPER_FORWARD_S))
    del plan
    torch.cuda.empty_cache()
    return out


def crofton_baseline(P, plan, views, g, target):
    """The analytic smooth Crofton weight of eq. 9 generated on the device for all
    views (one timed call after a warm-up), and the reconstruction error it gives
    without any learning, beside that of the constant weight 1/2."""
    import torch
    V, (K, S) = plan.n_views, plan.sino_shape
    M = torch.empty((V, K, S), device="cuda")
    segs, sid = views.meta["segments"], views.meta["sid"]
    P.dc_crofton_weights(plan, segs, sid, M)
    torch.cuda.synchronize()
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record()
    P.dc_crofton_weights(plan, segs, sid, M)
    b.record()
    torch.cuda.synchronize()
    ms = a.elapsed_time(b)
    with torch.no_grad():
        errs = {}
        for name, W in (("crofton", M), ("half", torch.full_like(M, 0.5))):
            f = P.reconstruct(plan, W, g=g, relu=True)
            errs[name] = float((f - target).double().norm() / target.double().norm())
            del f
    return {"ms": round(ms, 2), "entries_per_s": V * K * S / (ms * 1e-3), "fine": 64,
            "rel_error_untrained": round(errs["crofton"], 6), "rel_error_untrained_half": round(errs["half"], 6)}


def crofton_oracle_rate(grid, views, n_bins=24):
    """Entries per second of the oracle's eq. 9 (per-bin crossing search) on view 0."""
    import numpy as np
    from oracle import crofton
    rng = np.random.Generator(np.random.PCG64(0))
    bins = [(int(rng.integers(grid.n_theta)), int(rng.integers(grid.n_s))) for _ in range(n_bins)]
    t0 = time.perf_counter()
    crofton.M_view(views, grid, 0, bins=bins)
    return n_bins / (time.perf_counter() - t0)


def main():
    ap = argparse.ArgumentParser(description=__doc__.split("\n")[0])
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--dtype", choices=["f32", "bf16", "both"], default="both")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--cpu-workers", type=int, default=16,
                    help="largest number of oracle worker processes (one per usable core up to this)")
    ap.add_argument("--no-batched", action="store_true", help="skip the batched 8-scan measurement")
    ap.add_argument("--no-c3", action="store_true", help="skip the circle-plus-arc (C3) line")
    ap.add_argument("--no-shard", action="store_true", help="skip the one-GPU view-share (62 of 496 views) line")
    ap.add_argument("--no-c5", action="store_true", help="skip the full C-arm scale (C5) line")
    ap.add_argument("--no-paper", action="store_true",
                    help="skip the forward reconstruction of the paper's own workload")
    ap.add_argument("--no-autotune", action="store_true", help="keep the plans' default knobs")
    ap.add_argument("--orbit", choices=["sinusoid", "circle"], default="sinusoid",
                    help="the C2 grid on its sinusoidal orbit (default) or on a 496-view circle")
    ap.add_argument("--batched-steps", type=int, default=3)
    ap.add_argument("--copy-calibration-mib", type=int, default=0,
                    help="first run one plain device copy of this many MiB (reference for HBM counters)")
    args = ap.parse_args()
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py runs on exactly one GPU: this path is single-GPU (views would shard across GPUs "
              "with one all-reduce of the volume, which is not built).", file=sys.stderr)
        sys.exit(2)

    import synth
    cpu = None
    if not args.no_cpu_baseline:
        # the oracle first, in forked worker processes, before anything touches the GPU
        g_c2, v_c2 = synth.config_geometry("C2")
        log("cpu baseline (oracle) ...")
        cpu = cpu_baseline(g_c2, v_c2, args.cpu_workers)
        log("cpu baseline:", json.dumps(cpu))

    import torch
    import paper_2410_14900_amd as P

    if not torch.cuda.is_available():
        print("bench.py needs a GPU", file=sys.stderr)
        sys.exit(2)
    torch.cuda.set_device(0)
    cfg = synth.CONFIGS["C2"]
    grid, views = synth.config_geometry("C2")
    if args.orbit == "circle":
        views = synth.circle_orbit(len(views), cfg["sid"], cfg["sdd"])
    V = len(views)
    nvox = grid.nx * grid.ny * grid.nz
    log("geometry C2", grid.as_dict(), "views", V, "orbit", args.orbit)

    ell = synth.random_ellipsoids(cfg["n_ell"], grid.nx * grid.vx, cfg["seed"])
    p32 = synth.project_ellipsoids(ell, grid, views, device="cuda").float().contiguous()
    # Poisson noise from the library's counter-based generator (one warm-up, one timed call)
    g = torch.empty_like(p32)
    P.dc_poisson_noise(p32, g, cfg["noise"], synth.MU_WATER_PER_MM, seed=cfg["seed"])
    torch.cuda.synchronize()
    ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    ev0.record()
    P.dc_poisson_noise(p32, g, cfg["noise"], synth.MU_WATER_PER_MM, seed=cfg["seed"])
    ev1.record()
    torch.cuda.synchronize()
    noise_ms = ev0.elapsed_time(ev1)
    noise = {"ms": round(noise_ms, 3), "elements_per_s": p32.numel() / (noise_ms * 1e-3),
             "photons": cfg["noise"], "generator": "Philox4x64-10"}
    log("Poisson noise:", json.dumps(noise))
    del p32
    target = synth.voxelize_torch(ell, grid, device="cuda")
    plan = P.Plan(grid, views)
    if args.copy_calibration_mib:
        n = args.copy_calibration_mib * (1 << 20) // 4
        src = torch.rand(n, device="cuda")
        dst = torch.empty_like(src)
        torch.cuda.synchronize()
        dst.copy_(src)
        torch.cuda.synchronize()
        log("copy calibration: %d MiB read + %d MiB written" % (args.copy_calibration_mib, args.copy_calibration_mib))
        del src, dst
    torch.cuda.synchronize()
    log("inputs ready")
    # the step with the plan's default knobs, then the autotuner's choice (used below)
    tr = Trainer(P, plan, g, target, torch.float32)
    default_ms, _ = time_eager([tr], args.steps, args.warmup)
    del tr
    tuned = {"default_knobs": plan.knobs(), "default_knobs_ms_per_step": round(default_ms, 3)}
    if not args.no_autotune:
        t0 = time.perf_counter()
        tuned.update(plan.autotune())
        tuned["tune_s"] = round(time.perf_counter() - t0, 3)
    log("knobs:", json.dumps(tuned))

    results = {}
    for store in (["f32", "bf16"] if args.dtype == "both" else [args.dtype]):
        sdt = torch.float32 if store == "f32" else torch.bfloat16
        tr = Trainer(P, plan, g, target, sdt)
        ms, kern = time_eager([tr], args.steps, args.warmup, per_stage=True)
        log(store, "ms/step %.2f" % ms, json.dumps(kern), "rel error %.5f" % tr.rel_error())
        work = stage_work(grid, V, 4 if store == "f32" else 2)
        per_kernel = {}
        for st in Trainer.STAGES:
            units, byts = work[st]
            t = kern[st] * 1e-3
            per_kernel[st] = {"ms": round(kern[st], 3), "GB/s": round(byts / t / 1e9, 1),
                              "TFLOP/s": round(units * FLOPS_PER_UNIT[st] / t / 1e12, 2),
                              "lds_TB/s": round(units * LDS_BYTES_PER_UNIT[st] / t / 1e12, 2),
                              "lds_frac": round(units * LDS_BYTES_PER_UNIT[st] / t / 1e12 / LDS_PEAK_TBS, 3),
                              "units_per_s": units / t}
            per_kernel[st].update(valu_issue(st, store, units, t))
        results[store] = dict(ms=ms, kern=kern, per_kernel=per_kernel, work=work, rel_error=tr.rel_error())
        del tr
        torch.cuda.empty_cache()
    # the step with the paper's Gaussian filter layer on the weight (sigma 20, 121 taps)
    tr = Trainer(P, plan, g, target, torch.float32, smooth=(20.0, 60))
    sm_ms, sm_kern = time_eager([tr], args.steps, args.warmup, per_stage=True)
    smoothing = {"ms_per_step": round(sm_ms, 3), "smooth_ms": round(sm_kern["smooth"], 3),
                 "smooth_adjoint_ms": round(sm_kern["smooth_adjoint"], 3), "sigma": 20.0, "taps": 121,
                 "rel_error": round(tr.rel_error(), 6)}
    log("f32 with the Gaussian weight layer: ms/step %.2f" % sm_ms, json.dumps(smoothing))
    del tr
    torch.cuda.empty_cache()
    # the step with R stored (it depends only on the projections, not on M)
    tr = Trainer(P, plan, g, target, torch.float32, keep_R=True)
    kr_ms, _ = time_eager([tr], args.steps, args.warmup)
    r_stored = {"ms_per_step": round(kr_ms, 3), "value": nvox * V / (kr_ms * 1e-3),
                "note": "R = A2d(w_cos g) formed once before timing; the step runs from the filter to the Adam update"}
    log("f32 with R stored: ms/step %.2f" % kr_ms)
    del tr
    torch.cuda.empty_cache()
    crof = crofton_baseline(P, plan, views, g, target)
    log("Crofton weight (eq. 9) for all views:", json.dumps(crof))
    torch.cuda.empty_cache()
    graph_ms = None
    if args.dtype != "f32":
        tr = Trainer(P, plan, g, target, torch.bfloat16)
        graph_ms, _graph = time_graph(tr, args.steps, args.warmup)
        log("bf16 graph ms/step %.2f" % graph_ms)
        del tr, _graph
        torch.cuda.empty_cache()

    main_store = "f32" if "f32" in results else "bf16"
    r = results[main_store]
    dom = max(r["kern"], key=r["kern"].get)
    units, byts = r["work"][dom]
    t = r["kern"][dom] * 1e-3
    # measured on the sinusoidal C2 step only
    meas = MEASURED_TRAFFIC.get((dom, main_store)) if args.orbit == "sinusoid" else None
    traffic = meas[0] if meas and meas[1] == kernel_sources_digest(dom) else None
    if dom.startswith("filter"):
        roof = {"bound": "hbm", "kernel": dom, "achieved": round(byts / t / 1e9, 1), "peak": HBM_PEAK_GBS,
                "unit": "GB/s", "frac": round(byts / t / 1e9 / HBM_PEAK_GBS, 4), "traffic": traffic,
                "algorithmic_bytes": byts}
    else:
        ach = units * FLOPS_PER_UNIT[dom] / t / 1e12
        roof = {"bound": "alu", "kernel": dom, "achieved": round(ach, 3), "peak": FP32_PEAK_TFLOPS,
                "unit": "TFLOP/s", "frac": round(ach / FP32_PEAK_TFLOPS, 4), "traffic": traffic,
                "algorithmic_bytes": byts,
                "hbm_GBps": round(byts / t / 1e9, 1), "hbm_frac": round(byts / t / 1e9 / HBM_PEAK_GBS, 5),
                "lds_TBps": round(units * LDS_BYTES_PER_UNIT[dom] / t / 1e12, 2),
                "lds_frac": round(units * LDS_BYTES_PER_UNIT[dom] / t / 1e12 / LDS_PEAK_TBS, 3)}
        roof.update(valu_issue(dom, main_store, units, t))
    out = {
        "metric": METRIC,
        "value": nvox * V / (r["ms"] * 1e-3),
        "unit": "voxel-view updates/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": round(r["ms"], 3),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f32" if main_store == "f32" else "bf16-storage/f32-accumulate",
        "data": "synthetic: 20 seeded random ellipsoids, exact line integrals, Poisson noise at 1e5 photons/ray (Philox4x64-10)",
        "config": {"workload": ("C2: sinusoidal orbit" if args.orbit == "sinusoid" else
                                "C2 grid on a circular orbit") +
                               ", 496 views, 512x512 detector @0.6 mm, Radon 360x725, "
                               "256^3 volume @0.5 mm, forward+backward w.r.t. M + Adam step",
                   "views": V, "detector": [grid.nv, grid.nu], "radon": [grid.n_theta, grid.n_s],
                   "volume": [grid.nz, grid.ny, grid.nx]},
        "knobs": tuned,
        "roofline": roof,
        "kernels": r["per_kernel"],
        "rel_error": round(r["rel_error"], 6),
    }
    if "bf16" in results and main_store == "f32":
        b = results["bf16"]
        out["bf16"] = {"value": nvox * V / (b["ms"] * 1e-3), "ms_per_step": round(b["ms"], 3),
                       "kernels": b["per_kernel"], "speedup_vs_f32": round(r["ms"] / b["ms"], 3),
                       "rel_error": round(b["rel_error"], 6)}
    out["with_weight_smoothing"] = smoothing
    out["r_stored"] = r_stored
    out["crofton_weight"] = crof
    out["poisson_noise"] = noise
    if graph_ms is not None:
        out["bf16_graph"] = {"value": nvox * V / (graph_ms * 1e-3), "ms_per_step": round(graph_ms, 3),
                             "speedup_vs_f32": round(r["ms"] / graph_ms, 3) if main_store == "f32" else None}
    if not args.no_shard:
        out["view_shard"] = shard_line(P, grid, views, g, target, args)
    if not args.no_c3:
        out["c3"] = c3_line(P, synth, args)
        torch.cuda.empty_cache()
    if not args.no_paper:
        out["paper_workload"] = paper_workload_line(P, synth, args)
    if not args.no_c5:
        del plan
        torch.cuda.empty_cache()
        out["c5"] = c5_line(P, synth, args)
        torch.cuda.empty_cache()
        plan = None
    if not args.no_batched:
        plan = None
        torch.cuda.empty_cache()
        out["batched"] = batched_c4(P, synth, args)
    if cpu is not None:
        out["cpu_baseline"] = cpu
        out["crofton_weight"]["oracle_entries_per_s"] = round(crofton_oracle_rate(grid, views), 1)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
