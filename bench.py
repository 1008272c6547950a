"""Throughput benchmark of the per-object radiance-field training step.

Prints one JSON line: trained rays/s (draw, forward, loss, backward, dense
Adam) summed over all objects of the workload, measured on the batched path
(all objects per launch, one hipGraph per step), with the roofline of the
dominant kernel, the plain path (FP32, one launch per object per phase, no
graph) beside it, PSNR of both after training, and the CPU oracle timed on a
bounded sample of the same workload.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload objects24|objects24-fp32|torus1|stream128]

The default workload is the 24-object batched BF16 one (the metric's).  HBM
traffic per launch comes from rocprofv3 counter runs of this script (one per
pass of PMC_PASSES, with --copy-probe so that a plain copy calibrates the
request sizes and a random gather checks them), turned into a committed
summary by

    python bench.py --pmc-summary <rocprofv3 output dir> --workload <name>

The summary records a hash of the kernel source: once the kernels change,
the traffic is reported as null until the counters are taken again.

Inputs are seeded synthetic scenes (the paper's datasets are not available).
Only one GPU is used; --gpus above 1 exits with a message.
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

METRIC = "trained rays/s (fwd+bwd+Adam) all objects, batched BF16 vs plain FP32 @ equal PSNR"
HBM_PEAK_GBS = 8000.0     # MI355X HBM3E
BF16_PEAK_TFLOPS = 2500.0  # dense
FP32_MFMA_PEAK_TFLOPS = 157.3


KERNEL_SRC = os.path.join(ROOT, "paper_2304_05735_amd", "csrc", "romap_kernels.hip")
def log(*a):
    print("[bench]", *a, file=sys.stderr, flush=True)


def build_workload(name, frames=300):
    import scenes
    if name == "torus1":
        return scenes.torus_scene()
    if name in ("objects24", "objects24-fp32"):
        return scenes.room_scene(n_obj=24)
    if name == "stream128":
        return scenes.stream_scene(n_frames=frames)
    raise SystemExit(f"unknown workload {name}")


def run_stream(wl, args):
    """Incremental mapping stream: keyframes arrive one by one (25 Hz in the
    scene's timeline); every 10th frame (f % 10 == 5) is held out for
    evaluation and never trained on; an object is registered on the first
    training frame where its mask has >= 200 pixels; objects seen in the last
    50 frames are active; each frame trains every active object for 4 steps
    of 2^16 rays in total (2^18 rays per frame), split in proportion to the
    mask pixels seen so far (at least 64 each), with the BF16 MLP and 128
    samples per ray; the occupancy bitfield of an object is refreshed every
    25 frames once it has trained for 25 frames (unless --no-occupancy).

    Quality over time: each object is evaluated on a fixed set of up to 4
    held-out frames of the whole stream that show at least 500 of its pixels
    (PSNR over its mask pixels), every --eval-every frames, for the objects
    registered by then; the per-object curves and their mean are reported."""
    import numpy as np
    import paper_2304_05735_amd as pk
    import scenes
    cfg = pk.default_config(samples_per_ray=128, precision=pk.PREC_BF16, batch_mode=pk.BATCH_ALL,
                            use_graph=1, autotune=0, streams=STREAMS)
    ctx = pk.Context(cfg)
    spec = {o.instance: o for o in wl.objects}
    held = [f for f in range(len(wl.frames)) if f % 10 == 5]
    evalset = {}
    for f in held:
        ids, counts = np.unique(wl.frames[f][2], return_counts=True)
        for i, c in zip(ids, counts):
            if int(i) in spec and c >= 500:
                evalset.setdefault(int(i), []).append(f)
    for i in evalset:  # up to 4, spread over the stream
        fs = evalset[i]
        evalset[i] = [fs[j] for j in sorted({round(k * (len(fs) - 1) / 3) for k in range(4)})]
    oid_of, first, last_seen, pix, has_kf = {}, {}, {}, {}, {}
    budget, steps_per_frame = 1 << 16, 4
    frame_ms, train_ms, kf_ms, curve = [], [], [], []
    rays_trained = 0

    def evaluate(f):
        per = {}
        for inst, oid in oid_of.items():
            vals = []
            for v in evalset.get(inst, []):
                cam, rgb, mask, _ = wl.frames[v]
                pred, _, _ = ctx.render(oid, cam)
                vals.append(scenes.psnr(pred, rgb / 255.0, mask == inst))
            if vals:
                per[inst] = round(float(np.mean(vals)), 3)
        return per

    for f, (cam, rgb, mask, depth) in enumerate(wl.frames):
        if f % args.eval_every == args.eval_every - 1 and oid_of:
            per = evaluate(f)
            curve.append({"frame": f, "objects": len(per),
                          "mean_psnr": round(float(np.mean(list(per.values()))), 3) if per else None,
                          "per_object": per})
            log(f"frame {f}: mean PSNR {curve[-1]['mean_psnr']} over {len(per)} objects")
        if f % 10 == 5:
            continue  # held out
        ids, counts = np.unique(mask, return_counts=True)
        ctx.sync()
        t0 = time.perf_counter()
        for inst, cnt in zip(ids, counts):
            inst = int(inst)
            if inst == 0 or inst not in spec:
                continue
            if inst not in oid_of and cnt >= 200:
                ob = spec[inst]
                oid_of[inst] = ctx.add_object(inst, ob.t, ob.yaw, ob.half, ob.log2T)
                first[inst], pix[inst], has_kf[inst] = f, 0, False
            if inst in oid_of:
                last_seen[inst] = f
                pix[inst] += int(cnt)
                has_kf[inst] = True
        tk = time.perf_counter()
        ctx.add_keyframe(cam, rgb, mask, depth)
        ctx.sync()
        kf_ms.append((time.perf_counter() - tk) * 1e3)
        active = [i for i in oid_of if f - last_seen[i] <= 50 and has_kf[i]]
        if active:
            w = np.array([pix[i] for i in active], np.float64)
            r = np.maximum(64, np.floor(budget * w / w.sum())).astype(np.int32)
            t1 = time.perf_counter()
            ctx.train(steps_per_frame, [oid_of[i] for i in active], r, stats=False)
            rays_trained += int(r.sum()) * steps_per_frame
            if not args.no_occupancy:
                for i in active:
                    if f - first[i] >= 25 and (f - first[i]) % 25 == 0:
                        ctx.update_occupancy(oid_of[i], 0.05)
            ctx.sync()
            train_ms.append((time.perf_counter() - t1) * 1e3)
        frame_ms.append((time.perf_counter() - t0) * 1e3)
        if f % 25 == 0:
            log(f"frame {f}: {len(oid_of)} objects, {len(active)} active, "
                f"{frame_ms[-1]:.2f} ms")
    per = evaluate(len(wl.frames))
    curve.append({"frame": len(wl.frames), "objects": len(per),
                  "mean_psnr": round(float(np.mean(list(per.values()))), 3) if per else None,
                  "per_object": per})
    # objects evaluated at every checkpoint since their first: how many end
    # higher than they started, and the mean over a fixed set (those
    # registered by the first checkpoint)
    base = curve[0]["per_object"]
    fixed = [{"frame": c["frame"], "mean_psnr": round(float(np.mean([c["per_object"][i] for i in base
                                                                     if i in c["per_object"]])), 3)}
             for c in curve if base]
    rises = sum(1 for i in per if i in base and per[i] > base[i])
    fm = np.array(frame_ms)
    tm = np.array(train_ms)
    return dict(frames=len(wl.frames), frames_trained=len(frame_ms),
                objects_registered=len(oid_of), occupancy=not args.no_occupancy,
                ms_per_frame_mean=round(float(fm.mean()), 3),
                ms_per_frame_p50=round(float(np.percentile(fm, 50)), 3),
                ms_per_frame_p95=round(float(np.percentile(fm, 95)), 3),
                frames_over_40ms=int((fm > 40.0).sum()),
                keyframe_ms_mean=round(float(np.mean(kf_ms)), 3),
                train_rays_per_s=round(rays_trained / (tm.sum() * 1e-3), 1) if tm.size else None,
                psnr_mean_over_time=[(c["frame"], c["objects"], c["mean_psnr"]) for c in curve],
                psnr_fixed_objects_over_time=fixed,
                fixed_objects=len(base), fixed_objects_improved=rises,
                psnr_per_object_over_time=curve)


STREAMS = 2  # --streams: 1 for profiler runs (one launch per kernel and phase)


def make_ctx(wl, precision, batch_mode, use_graph, autotune=1, profile=0, **kw):
    import paper_2304_05735_amd as pk
    N = 64
    kw.setdefault("streams", STREAMS)
    cfg = pk.default_config(samples_per_ray=N, precision=precision, batch_mode=batch_mode,
                            use_graph=use_graph, autotune=autotune, profile_phases=profile, **kw)
    ctx = pk.Context(cfg)
    ids = []
    for ob in wl.objects:
        ids.append(ctx.add_object(ob.instance, ob.t, ob.yaw, ob.half, ob.log2T))
    ctx.sync()
    held_out = set(wl.eval_views)
    t0 = time.perf_counter()
    for f, (cam, rgb, mask, depth) in enumerate(wl.frames):
        if f not in held_out:  # evaluation views are never trained on
            ctx.add_keyframe(cam, rgb, mask, depth)
    ctx.sync()
    ctx.keyframe_seconds = time.perf_counter() - t0  # host buffers -> HBM, training frames
    keep, rays = [], []
    for i, ob in zip(ids, wl.objects):
        if ctx.object_info(i).n_keyframes > 0:
            keep.append(i)
            rays.append(wl.rays[ob.instance])
    return ctx, keep, rays


def timed_steps(ctx, ids, rays, warmup, steps):
    if warmup:
        ctx.train(warmup, ids, rays, stats=False)
    ctx.sync()
    t0 = time.perf_counter()
    ctx.train(steps, ids, rays, stats=False)
    ctx.sync()
    return time.perf_counter() - t0


def mean_psnr(ctx, wl, ids):
    import scenes
    vals = []
    for v in wl.eval_views:
        cam, rgb, mask, _ = wl.frames[v]
        for i, ob in zip(ids, wl.objects):
            m = mask == ob.instance
            if m.sum() < 50:
                continue
            pred, _, _ = ctx.render(i, cam)
            vals.append(scenes.psnr(pred, rgb / 255.0, m))
    return float(sum(vals) / max(len(vals), 1))


def psnr_curve(ctx, wl, ids, rays, steps, chunk):
    """PSNR on the held-out views after every `chunk` training steps."""
    curve = []
    done = 0
    while done < steps:
        n = min(chunk, steps - done)
        ctx.train(n, ids, rays, stats=False)
        done += n
        curve.append((done, mean_psnr(ctx, wl, ids)))
    return curve


def equal_psnr(wl, ids, rays, prec, steps, chunk, ms_batched, ms_plain, seeds=(0,), extend=2):
    """Batched path vs the plain FP32 path from the same initialisation, PSNR
    on the held-out views (never keyframes) every `chunk` steps, averaged over
    `seeds` (each seed changes the initialisation and the ray draws of both
    paths alike).  When the PSNRs after `steps` steps differ by at most 0.1
    dB the two are equal and the speedup is the ratio of their rates at equal
    step counts; otherwise it is the ratio of the times to reach the plain
    path's PSNR after `steps` steps (each path's first evaluated step count at
    or above it, times its measured time per step).  The batched path trains
    on to `extend` times the steps so that its time to that PSNR is found when
    it ends below it (null if it has not reached it by then); its PSNR at
    `steps` is the one compared.  The batched path with the FP32 MLP is run beside them
    (same launches as the batched path), which separates what the BF16 MLP
    changes from what batching changes."""
    import numpy as np
    import paper_2304_05735_amd as pk
    curves = {"batched": [], "plain_fp32": [], "batched_fp32": []}
    for sd in seeds:
        runs = [("batched", prec, pk.BATCH_ALL, 1), ("plain_fp32", pk.PREC_FP32, pk.BATCH_PER_OBJECT, 0)]
        if prec != pk.PREC_FP32:
            runs.append(("batched_fp32", pk.PREC_FP32, pk.BATCH_ALL, 1))
        for name, pr, mode, graph in runs:
            q, _, _ = make_ctx(wl, pr, mode, graph, seed=sd)
            n = steps * extend if name == "batched" else steps
            curves[name].append(psnr_curve(q, wl, ids, rays, n, chunk))
            del q
    mean = {k: [(c[0][j][0], float(np.mean([cc[j][1] for cc in c]))) for j in range(len(c[0]))]
            for k, c in curves.items() if c}
    ca_all, cb = mean["batched"], mean["plain_fp32"]
    ca = [c for c in ca_all if c[0] <= steps]
    pa, pb = ca[-1][1], cb[-1][1]
    out = dict(steps=steps, seeds=list(seeds), eval_views=list(wl.eval_views),
               psnr_batched=round(pa, 3), psnr_plain_fp32=round(pb, 3),
               delta_psnr=round(pa - pb, 3))
    if "batched_fp32" in mean:
        out["psnr_batched_fp32"] = round(mean["batched_fp32"][-1][1], 3)
    if len(seeds) > 1:
        out["final_psnr_per_seed"] = {k: [round(next(p for st, p in c if st == steps), 3) for c in v]
                                      for k, v in curves.items() if v}
    if abs(pa - pb) <= 0.1:
        out.update(rule="equal PSNR (|delta| <= 0.1 dB): ratio of rates at equal steps",
                   speedup_at_equal_psnr=round(ms_plain / ms_batched, 3))
    else:
        sa = next((k for k, v in ca_all if v >= pb), None)
        sb = next(k for k, v in cb if v >= pb)
        out.update(rule="time to the plain path's PSNR after the steps", target_psnr=round(pb, 3),
                   steps_batched_to_target=sa, steps_plain_to_target=sb,
                   batched_steps_run=steps * extend,
                   speedup_at_equal_psnr=None if sa is None else
                   round((sb * ms_plain) / (sa * ms_batched), 3))
    for k, c in mean.items():
        out[f"curve_{k}"] = [(st, round(v, 3)) for st, v in c]
    return out


def mesh_timing(ctx, ids, res=64, iso=10.0, reps=3):
    """Marching cubes of every object at res^3 (Sec. VI: 64^3 per object):
    density on the box corners, mesh, world placement, triangles copied to
    the host; wall time per object (best of reps, after one untimed call)."""
    import numpy as np
    per, ntri = [], []
    for i in ids:
        ctx.extract_mesh(i, res, iso)
        best = 1e9
        for _ in range(reps):
            t0 = time.perf_counter()
            tri = ctx.extract_mesh(i, res, iso)
            best = min(best, time.perf_counter() - t0)
        per.append(best * 1e3)
        ntri.append(len(tri))
    return dict(res=res, iso=iso, objects=len(ids), ms_per_object_mean=round(float(np.mean(per)), 4),
                ms_per_object_max=round(float(np.max(per)), 4),
                triangles_mean=int(np.mean(ntri)),
                paper_ms_per_object_rtx4090=2.84)


def table_sweep(wl, steps=200, warmup=20):
    """Table 4's model-size study on one object: time per step (graph, FP32
    and BF16) of 4096 rays x 32 samples (the paper's N) and of 4096 x 64, for
    T = 2^14 .. 2^20 with the one-hidden-layer density MLP, and for T = 2^16
    with density MLPs of 2 and 3 hidden layers, on the single-object scene."""
    import paper_2304_05735_amd as pk
    ob = wl.objects[0]
    rows = []
    models = [(lt, 1) for lt in (14, 16, 18, 20)] + [(16, 2), (16, 3)]
    for N in (32, 64):
        for prec in (pk.PREC_FP32, pk.PREC_BF16):
            for lt, layers in models:
                cfg = pk.default_config(samples_per_ray=N, precision=prec, use_graph=1, autotune=1,
                                        mlp_layers=layers)
                ctx = pk.Context(cfg)
                i = ctx.add_object(ob.instance, ob.t, ob.yaw, ob.half, lt)
                for cam, rgb, mask, depth in wl.frames:
                    ctx.add_keyframe(cam, rgb, mask, depth)
                dt = timed_steps(ctx, [i], [4096], warmup, steps)
                rows.append(dict(N=N, precision="bf16" if prec else "fp32", log2T=lt,
                                 mlp_layers=layers, ms_per_step=round(dt / steps * 1e3, 4)))
                log("table sweep", rows[-1])
                del ctx
    return dict(rows=rows, paper_rtx4090_ms={"2^14": 0.658, "2^16": 0.706, "2^18": 0.921,
                                              "2^20": 1.495, "2^16, 2 layers": 0.862,
                                              "2^16, 3 layers": 1.052})


def density_ablation(wl, ids, rays, prec, steps):
    """The loss ablation of the paper's Fig. 8 on this workload: training with
    and without the density term of the background rays (lambda_2 = 0.01 vs
    0).  Reported per setting: PSNR on the objects' pixels of the held-out
    views, and the mean rendered opacity over the pixels of those views that
    do not belong to the rendered object (mass floating in its box's empty
    space, which the term is meant to remove)."""
    import numpy as np
    import paper_2304_05735_amd as pk
    import scenes
    out = {}
    for lam in (0.01, 0.0):
        ctx, _, _ = make_ctx(wl, prec, pk.BATCH_ALL, 1, lambda_density=lam)
        ctx.train(steps, ids, rays, stats=False)
        ps, fl = [], []
        for v in wl.eval_views:
            cam, rgb, mask, _ = wl.frames[v]
            for i, ob in zip(ids, wl.objects):
                m = mask == ob.instance
                if m.sum() < 50:
                    continue
                pred, _, opac = ctx.render(i, cam)
                ps.append(scenes.psnr(pred, rgb / 255.0, m))
                fl.append(float(np.mean(opac[~m])))
        out[f"lambda2={lam}"] = {"psnr": round(float(np.mean(ps)), 3),
                                 "empty_space_opacity": float(np.mean(fl))}
        del ctx
    out["steps"] = steps
    return out


# Algorithmic work per the method (per evaluated sample: L levels x 8 corners
# x F = 2 features x 4 B gathered, the same scattered; e and its adjoint
# L x F x 4 B; dense Adam 32 B per parameter: p, g, m, v read, p, m, v, g
# written; MLP 6 flops per weight and sample: forward, input and weight
# adjoints).
def evaluated_samples(ctx, ids, rays):
    """Samples the method evaluates in one step: the draw of the context's
    current step, rays that hit their box and are not occluders (classes 1,
    2; misses and occluder rays carry no loss and are never evaluated)."""
    n = 0
    for i, B in zip(ids, rays):
        _, cls, _, _ = ctx.debug_rays(i, B)
        n += int(((cls == 1) | (cls == 2)).sum())
    return n * ctx.cfg.samples_per_ray


def method_work(ctx, ids, S):
    """Bytes (or flops) of one step per phase, for S evaluated samples."""
    L = ctx.cfg.n_levels
    grid = sum(ctx.object_info(i).n_grid_params for i in ids)
    per_obj_mlp = ctx.object_info(ids[0]).n_mlp_params  # the same MLP shape for every object
    payload = S * L * 8 * 2 * 4
    ebytes = S * L * 2 * 4
    return dict(
        gather=payload + ebytes,                    # A5: corners gathered, e written
        scatter_adam=payload + ebytes + 32 * grid,  # A12 + A13: adjoint read, corners scattered, Adam
        field_bytes=2 * ebytes,                     # e read, adjoint written
        mlp_flops=6 * per_obj_mlp * S,              # A6, A7, A11
        grid_params=grid)


def kernel_src_hash():
    import hashlib
    with open(KERNEL_SRC, "rb") as f:
        return hashlib.sha256(f.read()).hexdigest()[:16]


def traffic_file(workload):
    return os.path.join(ROOT, "profiles", f"hbm_traffic_{workload}.txt")


def _kernel_key(name):
    """'void k_field<0, 64, 32>(StepArgs)' -> 'k_field'"""
    n = name.replace("void ", "").strip()
    for sep in ("<", "("):
        n = n.split(sep)[0]
    return n.strip()


# Counter passes of a profiled run (rocprofv3 --pmc, one pass per run: a pass
# holds at most 4 TCC, 8 SQ and 2 GRBM counters).
PMC_PASSES = {
    "rd": "TCC_EA0_RDREQ_sum TCC_EA0_RDREQ_32B_sum TCC_EA0_RDREQ_64B_sum TCC_EA0_RDREQ_128B_sum",
    "wr": "TCC_EA0_WRREQ_sum TCC_EA0_WRREQ_64B_sum TCC_EA0_WRREQ_DRAM_sum TCC_EA0_RDREQ_DRAM_sum",
    "l2": "TCC_HIT_sum TCC_MISS_sum",
    # MfmaUtil: MFMA-busy cycles summed over SIMDs / (active cycles x SIMDs)
    "sq": "MfmaUtil SQ_BUSY_CYCLES SQ_INSTS_VALU_MFMA_MOPS_BF16 SQ_INSTS_VALU "
          "SQ_INSTS_LDS SQ_INSTS_MFMA SQ_WAVES SQ_WAIT_INST_ANY",
    # where waves spend their time (wave-cycles) and what the LDS does
    "st": "SQ_WAVE_CYCLES SQ_BUSY_CU_CYCLES SQ_WAIT_ANY SQ_WAIT_INST_LDS SQ_LDS_BANK_CONFLICT "
          "SQ_LDS_ADDR_CONFLICT SQ_ACTIVE_INST_LDS SQ_ACTIVE_INST_VMEM",
    "st2": "SQ_ACTIVE_INST_VALU SQ_ACTIVE_INST_ANY SQ_INSTS_LDS_ATOMIC SQ_LDS_ATOMIC_RETURN "
           "SQ_INSTS_VMEM_RD SQ_INSTS_VMEM_WR SQ_INSTS_SALU SQ_INSTS_SMEM",
}
STALL_TABLE_HEADER = "# where the waves' time goes"
COPY_MIB = 512          # --copy-probe: a plain copy of this size
GATHER_TABLE_MIB = 1024  # and a gather of random 4-byte words from a table this large
GATHER_N = 1 << 24


def _probe_kind(name):
    n = name.lower()
    if "copy" in n:
        return "copy"
    if "index" in n or "gather" in n:
        return "gather"
    return None


def _find_csv(d, name):
    """rocprofv3 writes <d>/<name> or nests it under host and process folders."""
    import glob
    hits = sorted(glob.glob(os.path.join(d, "**", name), recursive=True))
    if not hits:
        raise SystemExit(f"no {name} under {d}")
    return hits[0]


WORKLOAD_NOTES = {
    "objects24": "24 objects, 16 levels, T 2^15..2^19 by box volume, 25201 rays x 64 samples "
                 "per step, BF16 MLP, batched, step graph",
    "objects24-fp32": "the objects24 scene and rays with the FP32 MLP, batched, step graph",
    "torus1": "1 object, 16 levels, T 2^19, 4096 rays x 64 samples per step, FP32 MLP, step graph",
    "stream128": "128-object keyframe stream, 4 steps of 2^16 rays x 128 samples per frame over "
                 "the active objects, BF16 MLP, 64^3 occupancy, T 2^19",
}


def trace_summary(d, workload, steps, warmup, frames=300):
    """Kernel-time table (calls, average/min/max us, share) of a rocprofv3
    --kernel-trace --stats run of bench.py --only-headline --streams 1 (the
    stream: bench.py --frames F --streams 1), written to
    profiles/step_kernels_<workload>.txt."""
    import csv
    rows = list(csv.DictReader(open(_find_csv(d, "run_kernel_stats.csv"))))
    if workload == "stream128":
        run = f"--workload stream128 --frames {frames} --streams 1"
        what = (f"# the first {frames} frames of the stream on one stream (frames train eagerly: "
                "new shapes every frame); k_bin_scatter / k_bin_acc run once per bin group; "
                "k_field / k_encode_fwd also serve the PSNR renders")
    else:
        run = f"--workload {workload} --steps {steps} --warmup {warmup} --only-headline --streams 1"
        what = (f"# {steps + warmup} steps ({warmup} warm-up + {steps} timed) replay the step graph "
                "on one stream; extra calls of k_field / k_encode_fwd / k_raygen come "
                "from the autotuner and the graph capture; k_field<PREC, NS, K1, layers>")
    out = [f"# rocprofv3 kernel-trace summary: training-step kernels, workload {workload} "
           f"({WORKLOAD_NOTES.get(workload, workload)})",
           "# command (from the repository root, after __graft_entry__.build()):",
           "#   export TMPDIR=/tmp",
           f"#   rocprofv3 --kernel-trace --stats -d <out> -o run -f csv -- python3 bench.py {run}",
           f"#   python bench.py --trace-summary <out> {run.replace(' --only-headline', '').replace(' --streams 1', '')}",
           what,
           f"kernel_source_sha256_16 {kernel_src_hash()}",
           "# columns: kernel | calls | average us | min us | max us | share of kernel time %"]
    rows.sort(key=lambda r: -float(r["TotalDurationNs"]))
    for r in rows:
        name = r["Name"].replace("void ", "").strip()
        if "(" in name and "<" in name:
            name = name.split("(")[0]
        out.append(f"{name[:48]:48s} {int(r['Calls']):6d} {float(r['AverageNs']) / 1e3:10.2f} "
                   f"{float(r['MinNs']) / 1e3:10.2f} {float(r['MaxNs']) / 1e3:10.2f} "
                   f"{float(r['Percentage']):7.2f}")
    path = os.path.join(ROOT, "profiles", f"step_kernels_{workload}.txt")
    with open(path, "w") as fh:
        fh.write("\n".join(out) + "\n")
    print("\n".join(out))
    log("wrote", path)


def pmc_summary(d, workload, steps):
    """Per-kernel counter summary from the rocprofv3 --pmc runs in <d>/<pass>
    (PMC_PASSES) of bench.py --only-headline --copy-probe.  HBM bytes come
    from read requests counted by size (32, 64 and 128 bytes) and write
    requests (64 bytes, else 32).  The copy probe (COPY_MIB read and written)
    checks that these sizes account for its bytes; read requests of no
    counted size (none expected) would take the size that balances the copy.
    The random-gather probe and every kernel are checked against the copy's
    rate: bytes that imply more than it are flagged.  Also the L2 hit rate
    and, per kernel, MFMA utilisation, BF16 MFMA flops and instruction
    counts."""
    import csv
    import glob
    vals = {}  # (kernel, counter) -> [per-dispatch values]
    dur = {}   # kernel or probe -> [ns]
    missing = [sub for sub in PMC_PASSES if not glob.glob(
        os.path.join(d, sub, "**", "run_counter_collection.csv"), recursive=True)]
    for sub in PMC_PASSES:
        if sub in missing:
            continue
        path = _find_csv(os.path.join(d, sub), "run_counter_collection.csv")
        for r in csv.DictReader(open(path)):
            name = r["Kernel_Name"]
            key = _kernel_key(name) if _kernel_key(name).startswith("k_") else _probe_kind(name)
            if key is None:
                continue
            vals.setdefault((key, r["Counter_Name"]), []).append(float(r["Counter_Value"]))
        for ktrace in glob.glob(os.path.join(d, sub, "**", "run_kernel_trace.csv"), recursive=True)[:1]:
            for r in csv.DictReader(open(ktrace)):
                name = r["Kernel_Name"]
                key = _kernel_key(name) if _kernel_key(name).startswith("k_") else _probe_kind(name)
                if key:
                    dur.setdefault(key, []).append(float(r["End_Timestamp"]) -
                                                   float(r["Start_Timestamp"]))

    def mean(key, c):
        x = vals.get((key, c))
        if not x:
            return 0.0
        if key in ("copy", "gather"):  # the probe itself: the largest such dispatch
            return max(x)
        return sum(x) / len(x)

    def avg_us(key):
        x = dur.get(key, [])
        if key in ("copy", "gather"):  # the median of the probe's repeats (all passes)
            top = sorted(t for t in x if t >= 0.5 * max(x)) if x else []
            return top[len(top) // 2] / 1e3 if top else 0.0
        return sum(x) / len(x) / 1e3 if x else 0.0

    def reads(key):
        n, n32, n64, n128 = (mean(key, "TCC_EA0_RDREQ_sum"), mean(key, "TCC_EA0_RDREQ_32B_sum"),
                             mean(key, "TCC_EA0_RDREQ_64B_sum"), mean(key, "TCC_EA0_RDREQ_128B_sum"))
        return 32 * n32 + 64 * n64 + 128 * n128, max(n - n32 - n64 - n128, 0.0)

    def writes(key):
        w, w64 = mean(key, "TCC_EA0_WRREQ_sum"), mean(key, "TCC_EA0_WRREQ_64B_sum")
        return 64 * w64 + 32 * (w - w64)

    copy_bytes = COPY_MIB * 2 ** 20
    cr, crest = reads("copy")
    rsize = (copy_bytes - cr) / crest if crest > 0 else 0.0

    def hbm(key):
        r, rest = reads(key)
        return r + rsize * rest, writes(key), rest

    cw = writes("copy")
    copy_us = avg_us("copy")
    copy_gbs = (sum(hbm("copy")[:2])) / (copy_us * 1e-6) / 1e9 if copy_us > 0 else 0.0
    out = [f"# HBM traffic and counters per dispatch, workload {workload}",
           "# passes (one rocprofv3 run each; <pass> in " + ", ".join(PMC_PASSES) + "):",
           f"#   rocprofv3 --pmc <counters of the pass> --kernel-trace -d <dir>/<pass> -o run -f csv "
           f"-- python3 bench.py --steps {steps} --warmup 3 --only-headline --copy-probe "
           f"--streams 1 --workload {workload}",
           f"# then: python bench.py --pmc-summary <dir> --workload {workload} --steps {steps}",
           "# counters of the passes: " + "; ".join(f"{k}: {v}" for k, v in PMC_PASSES.items()),
           "# passes not taken: " + (", ".join(missing) or "none"),
           f"# read bytes = 32 n32 + 64 n64 + 128 n128 (+ unsized requests at the size that "
           f"balances the copy); write bytes = 64 n64 + 32 (n - n64)",
           "# these are the requests that leave the L2s; lines that the 256 MB Infinity Cache "
           "serves count too, so a kernel that fetches the same lines into several XCDs' L2s "
           "(or again soon after) can imply more than the copy's HBM rate",
           f"# copy probe ({COPY_MIB} MiB read and written): counted reads {cr / copy_bytes:.4f}, "
           f"writes {cw / copy_bytes:.4f} of its bytes; unsized read requests {crest:.0f}"
           + (f" (taken at {rsize:.1f} B)" if crest > 0 else "")
           + f"; {copy_us:.1f} us, {copy_gbs:.0f} GB/s"]
    gr, gw, _ = hbm("gather")
    want = GATHER_N * 4
    g_us = avg_us("gather")
    g_gbs = (gr + gw) / (g_us * 1e-6) / 1e9 if g_us > 0 else 0.0
    out.append(f"# random-gather probe ({GATHER_N} words from {GATHER_TABLE_MIB} MiB, int64 "
               f"indices): {gr / 1e6:.1f} MB read for {want / 1e6:.1f} MB of words, "
               f"{gw / 1e6:.1f} MB written; {g_us:.1f} us, {g_gbs:.0f} GB/s"
               + (" (above the copy's rate: part of the table's lines come from the Infinity "
                  "Cache)" if g_gbs > copy_gbs > 0 else " (within the copy's rate)"))
    out.append(f"kernel_source_sha256_16 {kernel_src_hash()}")
    out.append("# kernel dispatches read_bytes write_bytes hbm_bytes avg_us implied_GB/s "
               "l2_hit_rate mfma_util bf16_mfma_flops valu_insts lds_insts mfma_insts "
               "wait_inst_any_quads waves")
    keys = sorted(k for k in {k for k, _ in vals} if k not in ("copy", "gather"))
    over = []
    for k in keys:
        r_, w_, _ = hbm(k)
        n = len(vals.get((k, "TCC_EA0_RDREQ_sum"), [0]))
        us = avg_us(k)
        gbs = (r_ + w_) / (us * 1e-6) / 1e9 if us > 0 else 0.0
        if copy_gbs > 0 and gbs > copy_gbs:
            over.append(k)
        hit, miss = mean(k, "TCC_HIT_sum"), mean(k, "TCC_MISS_sum")
        mu = mean(k, "MfmaUtil") / 100.0
        bf16_flops = 512.0 * mean(k, "SQ_INSTS_VALU_MFMA_MOPS_BF16")
        out.append(f"{k} {n} {r_:.0f} {w_:.0f} {r_ + w_:.0f} {us:.1f} {gbs:.0f} "
                   f"{hit / max(hit + miss, 1):.3f} {mu:.4f} {bf16_flops:.4g} "
                   f"{mean(k, 'SQ_INSTS_VALU'):.0f} {mean(k, 'SQ_INSTS_LDS'):.0f} "
                   f"{mean(k, 'SQ_INSTS_MFMA'):.0f} {mean(k, 'SQ_WAIT_INST_ANY'):.4g} "
                   f"{mean(k, 'SQ_WAVES'):.0f}")
    out.append("# kernels whose request bytes imply more than the copy's rate (served in part by "
               "the Infinity Cache): " + (", ".join(over) or "none"))
    out.append(STALL_TABLE_HEADER + " (ratios of wave-cycle counters; per wave: averages "
               "over the dispatch's waves)")
    out.append("# kernel wave_cycles_per_wave wait_any wait_inst_lds active_valu active_vmem "
               "active_lds lds_bank_conflict_per_lds_cycle lds_addr_conflict_per_lds_cycle "
               "lds_atomic_insts vmem_rd_insts vmem_wr_insts salu_insts")
    for k in keys:
        wc = mean(k, "SQ_WAVE_CYCLES")
        if wc <= 0:
            continue
        nw = max(mean(k, "SQ_WAVES"), 1.0)
        lds = max(mean(k, "SQ_ACTIVE_INST_LDS"), 1.0)
        out.append(f"{k} {wc / nw:.0f} {mean(k, 'SQ_WAIT_ANY') / wc:.3f} "
                   f"{mean(k, 'SQ_WAIT_INST_LDS') / wc:.3f} {mean(k, 'SQ_ACTIVE_INST_VALU') / wc:.3f} "
                   f"{mean(k, 'SQ_ACTIVE_INST_VMEM') / wc:.3f} {mean(k, 'SQ_ACTIVE_INST_LDS') / wc:.3f} "
                   f"{mean(k, 'SQ_LDS_BANK_CONFLICT') / lds:.3f} "
                   f"{mean(k, 'SQ_LDS_ADDR_CONFLICT') / lds:.3f} "
                   f"{mean(k, 'SQ_INSTS_LDS_ATOMIC'):.0f} {mean(k, 'SQ_INSTS_VMEM_RD'):.0f} "
                   f"{mean(k, 'SQ_INSTS_VMEM_WR'):.0f} {mean(k, 'SQ_INSTS_SALU'):.0f}")
    path = traffic_file(workload)
    with open(path, "w") as fh:
        fh.write("\n".join(out) + "\n")
    print("\n".join(out))
    log("wrote", path)


def copy_bandwidth(nbytes=1 << 30, reps=10):
    """Device-to-device copy rate (GB/s, bytes read + written) of a plain
    tensor copy: the achievable HBM bandwidth the roofline is also quoted
    against (besides the datasheet peak)."""
    import torch
    src = torch.ones(nbytes // 4, device="cuda")
    dst = torch.empty_like(src)
    for _ in range(3):
        dst.copy_(src)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    e0.record()
    for _ in range(reps):
        dst.copy_(src)
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / reps
    del src, dst
    return 2 * nbytes / (ms * 1e-3) / 1e9


def traffic_of(workload, kernels):
    """Calibrated HBM bytes per step of the given kernels from the committed
    counter summary, or None if it is missing or the kernels changed since."""
    path = traffic_file(workload)
    if not os.path.exists(path):
        return None
    tab, src = {}, None
    for line in open(path):
        if line.startswith("kernel_source_sha256_16"):
            src = line.split()[1]
        elif line.startswith(STALL_TABLE_HEADER):
            break  # the byte table ends here (the stall table repeats the kernel names)
        elif line.strip() and not line.startswith("#"):
            f = line.split()
            tab[f[0]] = float(f[4])
    if src != kernel_src_hash():
        return None
    return sum(tab.get(k, 0.0) for k in kernels)


def cpu_model():
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return None


def cpu_baseline(wl, seconds_target=12.0):
    """The oracle as it stands on the host cores, on a bounded sample: as many
    full training steps of the first object as fit in ~seconds_target, on
    every core this process may use and then on one core."""
    import oracle
    ob = wl.objects[0]
    B = wl.rays[ob.instance]
    held_out = set(wl.eval_views)
    runs = {}
    for threads in (oracle.host_threads(), 1):
        cfg = oracle.make_config(N=64, log2T=ob.log2T)
        o = oracle.OracleContext(cfg, nthreads=threads)
        oid = o.add_object(ob.instance, ob.t, ob.yaw, ob.half, ob.log2T)
        for f, (cam, rgb, mask, depth) in enumerate(wl.frames):
            if f not in held_out:
                o.add_keyframe(cam, rgb, mask, depth)
        t0 = time.perf_counter()
        steps = 0
        while time.perf_counter() - t0 < seconds_target and steps < 50:
            o.train(oid, 1, B)
            steps += 1
        dt = time.perf_counter() - t0
        runs[threads] = (steps * B / dt, steps)
        log(f"cpu oracle, {threads} threads: {steps} steps in {dt:.1f} s")
        del o
    allc = oracle.host_threads()
    v, n = runs[allc]
    v1, n1 = runs[1]
    return dict(value=round(v, 1), unit="rays/s", cores=allc, kind="oracle",
                sample=f"{n} full training steps x {B} rays x 64 samples of object instance "
                       f"{ob.instance} (2^{ob.log2T} table, FP64) on {allc} threads; "
                       f"{n1} such steps on 1 thread",
                cpu_model=cpu_model(), one_core={"value": round(v1, 1), "cores": 1})


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=200)
    ap.add_argument("--warmup", type=int, default=20)
    ap.add_argument("--workload", default="objects24",
                    choices=("objects24", "objects24-fp32", "torus1", "stream128"))
    ap.add_argument("--psnr-steps", type=int, default=2000)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-psnr", action="store_true")
    ap.add_argument("--table-sweep", action="store_true",
                    help="time one object for T = 2^14..2^20 and for 2- and 3-layer density MLPs "
                         "(the paper's Table 4 study) and exit")
    ap.add_argument("--no-ablation", action="store_true",
                    help="skip the lambda_2 = 0 training run (PSNR and empty-space opacity)")
    ap.add_argument("--psnr-chunk", type=int, default=250)
    ap.add_argument("--psnr-seeds", type=int, default=2,
                    help="seeds the equal-PSNR comparison is averaged over")
    ap.add_argument("--only-headline", action="store_true",
                    help="time the batched path only (for profiler runs)")
    ap.add_argument("--frames", type=int, default=300, help="frames of the stream128 workload")
    ap.add_argument("--eval-every", type=int, default=50,
                    help="stream128: evaluate the registered objects every this many frames")
    ap.add_argument("--no-occupancy", action="store_true",
                    help="stream128: train without the occupancy skip")
    ap.add_argument("--streams", type=int, default=2, choices=(1, 2),
                    help="streams of a batched step (1 for profiler runs: kernel traces and "
                         "counters then describe one launch per kernel and phase)")
    ap.add_argument("--copy-probe", action="store_true",
                    help="first copy 512 MiB three times (calibrates the HBM byte counters)")
    ap.add_argument("--pmc-summary", metavar="DIR",
                    help="write the HBM traffic summary from rocprofv3 counter runs and exit")
    ap.add_argument("--trace-summary", metavar="DIR",
                    help="write the kernel-time summary of a rocprofv3 --kernel-trace --stats "
                         "run and exit")
    args = ap.parse_args()
    global STREAMS
    STREAMS = args.streams
    if args.pmc_summary:
        pmc_summary(args.pmc_summary, args.workload, args.steps)
        return
    if args.trace_summary:
        trace_summary(args.trace_summary, args.workload, args.steps, args.warmup, args.frames)
        return
    if args.gpus != 1:
        print(f"bench.py measures one GPU only (asked for {args.gpus}): the path is the "
              "single-GPU share of the workload; sharding across GPUs is not built.",
              file=sys.stderr)
        sys.exit(2)

    import torch
    import paper_2304_05735_amd as pk
    # the scene renders in forked worker processes: build it before this
    # process opens the GPU (afterwards it would render serially)
    log("workload", "torus1 (table sweep)" if args.table_sweep else args.workload)
    t = time.perf_counter()
    wl = build_workload("torus1" if args.table_sweep else args.workload, args.frames)
    log(f"scene ready in {time.perf_counter() - t:.1f}s: {len(wl.objects)} objects, "
        f"{len(wl.frames)} frames")
    assert torch.cuda.is_available(), "no GPU visible"
    if args.copy_probe:
        src = torch.ones(COPY_MIB << 18, device="cuda")  # COPY_MIB MiB of floats
        dst = torch.empty_like(src)
        for _ in range(3):
            dst.copy_(src)
        del src, dst
        tab = torch.ones(GATHER_TABLE_MIB << 18, device="cuda")
        idx = torch.randint(0, tab.numel(), (GATHER_N,), device="cuda")
        for _ in range(3):
            out = torch.index_select(tab, 0, idx)
        torch.cuda.synchronize()
        log(f"copy probe: 3 x {COPY_MIB} MiB copied, 3 x {GATHER_N} random words gathered")
        del tab, idx, out
    if args.table_sweep:
        print(json.dumps({"table_sweep": table_sweep(wl)}), flush=True)
        return
    if args.workload == "stream128":
        st = run_stream(wl, args)
        log("stream", json.dumps(st))
        out = {"metric": METRIC, "value": st["train_rays_per_s"], "unit": "rays/s", "n_gpus": 1,
               "steps": None, "warmup": 0, "ms_per_step": None, "higher_is_better": True,
               "scaling": "weak", "vs_baseline": None, "dtype": "bf16-mfma/fp32",
               "data": "synthetic", "config": {"workload": wl.name}, "stream": st}
        print(json.dumps(out), flush=True)
        return
    prec = pk.PREC_BF16 if args.workload == "objects24" else pk.PREC_FP32
    # ---- headline: batched path, one hipGraph per step (captured by the
    # untimed warm-up call, replayed by the timed one)
    ctx, ids, rays = make_ctx(wl, prec, pk.BATCH_ALL, 2)
    rays_per_step = sum(rays)
    # RGB8, int32 mask, float depth where given
    kf_bytes = sum(rgb.shape[0] * rgb.shape[1] * (3 + 4 + (4 if depth is not None else 0))
                   for f, (_, rgb, _, depth) in enumerate(wl.frames) if f not in wl.eval_views)
    keyframes = {"frames": len(wl.frames) - len(wl.eval_views),
                 "ms": round(ctx.keyframe_seconds * 1e3, 3), "MB": round(kf_bytes / 1e6, 1),
                 "GB_per_s": round(kf_bytes / ctx.keyframe_seconds / 1e9, 2)}
    log("keyframes", json.dumps(keyframes))
    log(f"{len(ids)} trained objects, {rays_per_step} rays/step")
    dt = timed_steps(ctx, ids, rays, max(args.warmup, 1), args.steps)
    value = rays_per_step * args.steps / dt
    ms_step = dt / args.steps * 1e3
    log(f"batched: {ms_step:.4f} ms/step, {value / 1e6:.3f} M rays/s")
    if args.only_headline:
        print(json.dumps({"value": value, "ms_per_step": ms_step}), flush=True)
        return
    mesh = mesh_timing(ctx, ids)
    log("mesh", json.dumps(mesh))
    del ctx
    batched_fp32 = None
    if prec == pk.PREC_BF16:  # the same batched path with the FP32 MLP
        fctx, _, _ = make_ctx(wl, pk.PREC_FP32, pk.BATCH_ALL, 2)
        dtf = timed_steps(fctx, ids, rays, max(args.warmup, 1), args.steps)
        batched_fp32 = {"value": round(rays_per_step * args.steps / dtf, 1), "unit": "rays/s",
                        "ms_per_step": round(dtf / args.steps * 1e3, 5)}
        log("batched FP32", json.dumps(batched_fp32))
        del fctx
    # ---- per-kernel durations (HIP events on the context stream, same kernels)
    pctx, _, _ = make_ctx(wl, prec, pk.BATCH_ALL, 0, profile=1)
    pctx.train(args.warmup, ids, rays, stats=False)
    S = evaluated_samples(pctx, ids, rays)
    pctx.train(args.steps, ids, rays, stats=False)
    phases, nph = pctx.phase_times()
    records = pctx.step_records()
    log("phase ms:", json.dumps({k: round(v, 5) for k, v in phases.items()}))
    work = method_work(pctx, ids, S)
    copy_gbs = copy_bandwidth()
    log(f"copy bandwidth {copy_gbs:.0f} GB/s")

    def hbm(name, kernels, byt):
        ms = sum(phases[k] for k in kernels)
        a = byt / (ms * 1e-3) / 1e9
        return dict(bound="hbm", kernels=["k_" + k for k in kernels], avg_ms=round(ms, 5),
                    algorithmic_bytes=int(byt), achieved=round(a, 1), peak=HBM_PEAK_GBS,
                    unit="GB/s", frac=round(a / HBM_PEAK_GBS, 4), frac_of_copy=round(a / copy_gbs, 4))

    peak_f = BF16_PEAK_TFLOPS if prec == pk.PREC_BF16 else FP32_MFMA_PEAK_TFLOPS
    tf = work["mlp_flops"] / (phases["field"] * 1e-3) / 1e12
    mfma_measured = pk.debug_mfma_rate(prec)  # what the matrix cores sustain here
    log(f"measured MFMA rate ({'BF16' if prec == pk.PREC_BF16 else 'FP32'}): "
        f"{mfma_measured:.0f} TFLOP/s")
    units = {
        "scatter_adam": hbm("scatter_adam", ["bin_scatter", "bin_acc", "bin_finish"],
                            work["scatter_adam"]),
        "gather": hbm("gather", ["encode_fwd"], work["gather"]),
        "mlp": dict(bound="mfma", kernels=["k_field"], avg_ms=round(phases["field"], 5),
                    algorithmic_flops=int(work["mlp_flops"]), achieved=round(tf, 2),
                    peak=peak_f, unit="TFLOP/s", frac=round(tf / peak_f, 4),
                    peak_measured=round(mfma_measured, 1),
                    frac_of_measured=round(tf / mfma_measured, 4),
                    hbm_bytes=int(work["field_bytes"])),
    }
    dominant = max(units, key=lambda k: units[k]["avg_ms"])
    roofline = dict(units[dominant])
    tr = traffic_of(args.workload, roofline["kernels"])
    roofline.update(unit_name=dominant, traffic=None if tr is None else int(tr),
                    copy_gbs=round(copy_gbs, 1), units=units,
                    evaluated_samples=S, samples_drawn=rays_per_step * pctx.cfg.samples_per_ray,
                    grid_params=work["grid_params"],
                    records_per_step=int(records), record_bytes_per_step=int(8 * records),
                    phase_ms={k: round(v, 5) for k, v in phases.items()})
    del pctx
    # ---- plain path: FP32, one launch per object per phase, no graph
    plain_ctx, _, _ = make_ctx(wl, pk.PREC_FP32, pk.BATCH_PER_OBJECT, 0)
    dtp = timed_steps(plain_ctx, ids, rays, args.warmup, args.steps)
    plain = rays_per_step * args.steps / dtp
    log(f"plain FP32 per-object: {dtp / args.steps * 1e3:.4f} ms/step, {plain / 1e6:.3f} M rays/s")
    del plain_ctx
    quality = None
    if not args.no_psnr:
        quality = equal_psnr(wl, ids, rays, prec, args.psnr_steps, args.psnr_chunk, ms_step,
                             dtp / args.steps * 1e3, seeds=tuple(range(args.psnr_seeds)))
        log("psnr", json.dumps(quality))
    ablation = None
    if not args.no_ablation and not args.no_psnr:
        ablation = density_ablation(wl, ids, rays, prec, args.psnr_steps)
        log("ablation", json.dumps(ablation))
    cpu = None
    if not args.no_cpu_baseline:
        log("cpu baseline (oracle) ...")
        cpu = cpu_baseline(wl)
        log("cpu", cpu)
    dtype = "bf16-mfma/fp32" if prec == pk.PREC_BF16 else "fp32"
    out = {
        "metric": METRIC, "value": round(value, 1), "unit": "rays/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": round(ms_step, 5),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": dtype,
        "data": "synthetic",
        "config": {"workload": wl.name, "objects": len(ids), "rays_per_step": rays_per_step,
                   "samples_per_ray": 64, "levels": 16, "batched": True, "graph": True},
        "roofline": roofline,
        "batched_fp32": batched_fp32,
        "plain_fp32": {"value": round(plain, 1), "unit": "rays/s",
                       "ms_per_step": round(dtp / args.steps * 1e3, 5),
                       "ratio_at_equal_steps": round(value / plain, 3)},
        "quality": quality,
        "ablation_density": ablation,
        "mesh": mesh,
        "cpu_baseline": cpu,
        "keyframe_upload": keyframes,
    }
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
