#!/usr/bin/env python3
"""Benchmark of the BEV-pooling forward pass on one MI355X.

One step is one bevpool_forward over one batch: the fused lift (P x F) and
per-cell sum for every BEV cell. This is the whole per-frame hot path. The
plan is built once beforehand and timed separately.

The default workload is the nuScenes-shaped frame: 6 cameras x 118 depth
bins x 32x88 features, C = 80 fp32, pooled to a 360x360 grid. Inputs are
seeded synthetic data already resident in device memory.

Timing: before every timed step a 1 GiB read (a sum over a scratch buffer)
evicts the L2s and the Infinity Cache, so each forward reads its inputs from
HBM. A read leaves no dirty lines behind whose write-back would be charged
to the forward. The forward's GPU time comes from HIP events that its own
first and last kernel dispatch record (bevpool_forward_timed, on the stream
that runs the kernels): events recorded as separate stream entries add
several microseconds of queue gap, which is reported beside it
(outer_events_mean). The headline `value` is algorithmic bytes (P + F read
once, the BEV map written once) divided by the mean forward time. The warm
figure (back-to-back, no eviction) is reported too.

Prints one JSON line. See `--help` for the knobs.
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import platform
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = ("BEV-pool forward ms + HBM GB/s, 6cam×118D×32×88×C80"
          "→360×360 BEV, 1 GPU")
HBM_PEAK_GBS = 8000.0          # MI355X HBM3E, AMD published figure
FLUSH_BYTES = 1 << 30
PLAN_REBUILDS = 4               # plan builds timed after the first
TRAFFIC_FILE = os.path.join(ROOT, "profiles", "forward_traffic.json")
KERNEL_SOURCE = os.path.join(ROOT, "paper_2205_13542_amd", "csrc", "forward.hip")
# Every file that shapes the forward's memory traffic: the kernels, the
# device helpers and constants they use, the plan builder that lays out the
# work partition, and the build flags. A counter record is tied to their
# combined hash.
FORWARD_SOURCES = [os.path.join(ROOT, "paper_2205_13542_amd", *p) for p in (
    ("csrc", "forward.hip"), ("csrc", "device.h"), ("csrc", "internal.h"), ("csrc", "plan.hip"),
    ("build.py",))]
BWD_SOURCE = os.path.join(ROOT, "paper_2205_13542_amd", "csrc", "backward.hip")

WORKLOAD_TEXT = {
    "nuscenes": "nuScenes-shaped frame: 6 cams x 118 depth bins x 32x88, C=80 fp32 -> 360x360 BEV at 0.3 m",
    "nuscenes_bf16": "nuScenes-shaped frame, bf16 P and F, fp32 accumulate/output -> 360x360",
    "nuscenes_f16": "nuScenes-shaped frame, fp16 P and F, fp32 accumulate/output -> 360x360",
    "nuscenes_b8": "8 nuScenes-shaped frames sharing one plan, C=80 fp32 -> 8 x 360x360",
    "highres": "6 cams x 236 bins x 64x176, C=128 fp32, 90% one-hot depth -> 720x720 at 0.15 m",
    "nuscenes_tilted": "nuScenes-shaped frame, every camera pitched 5 deg and rolled 2 deg (generic cells), C=80 fp32 -> 360x360",
    "nuscenes_tilt1": "nuScenes-shaped frame, every camera pitched 1 deg and rolled 0.5 deg, C=80 fp32 -> 360x360",
}


def parse_args():
    ap = argparse.ArgumentParser(description=__doc__, formatter_class=argparse.RawDescriptionHelpFormatter)
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=100)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--workload", default="nuscenes", choices=sorted(WORKLOAD_TEXT))
    ap.add_argument("--no-cpu-baseline", action="store_true",
                    help="skip the oracle timing on the host cores")
    ap.add_argument("--cpu-seconds", type=float, default=10.0,
                    help="approximate CPU time budget of the oracle sample")
    ap.add_argument("--reduce", default="sum", choices=["sum", "mean", "max"],
                    help="aggregation (mean/max, and --slabs, are timed by reduce_bench)")
    ap.add_argument("--slabs", type=int, default=1,
                    help="z slabs of 4 m from z = -8 m, flattened by channel concatenation")
    ap.add_argument("--cumsum", action="store_true",
                    help="time the prior-art prefix-sum pooling beside the forward (speed ratio)")
    ap.add_argument("--nchw", action="store_true",
                    help="time the channel-major copy of the pooled map (bevpool_to_nchw)")
    ap.add_argument("--backward", action="store_true",
                    help="time bevpool_backward (gradients of P and F) instead of the forward; "
                         "prints its own JSON line")
    ap.add_argument("--floor", action="store_true",
                    help="time a plain streaming kernel that moves the workload's compulsory "
                         "bytes (inputs read once, map written once) and an empty launch")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="only run a plain device-to-device copy of 256 MiB five times (the "
                         "reference kernel for scaling the FETCH_SIZE / WRITE_SIZE counters)")
    return ap.parse_args()


COPY_BYTES = 256 << 20


def copy_calibration():
    """A plain copy of COPY_BYTES, five times. Under rocprofv3 --pmc its
    FETCH_SIZE and WRITE_SIZE per dispatch give the counter's reading for a
    known number of HBM bytes."""
    import torch
    dev = torch.device("cuda:0")
    src = torch.ones(COPY_BYTES // 4, dtype=torch.float32, device=dev)
    dst = torch.empty_like(src)
    torch.cuda.synchronize()
    for _ in range(5):
        dst.copy_(src)
    torch.cuda.synchronize()
    print(json.dumps({"copy_calibration": True, "bytes_read": COPY_BYTES,
                      "bytes_written": COPY_BYTES, "launches": 5}), flush=True)


def floor_bench(args):
    """The streaming floor of the workload on this device: a plain kernel
    (paper_2205_13542_amd/csrc/floor.hip, 16-byte accesses, 8 workgroups per
    CU, each streaming one contiguous share) that reads the inputs' bytes
    once and writes the map's bytes once, the read and write halves alone,
    and an empty launch of the same shape. Timed like the forward: a 1 GiB
    cache-evicting read before each launch, dispatch-attached events."""
    import ctypes
    import numpy as np
    import torch
    import workloads as wl
    from paper_2205_13542_amd import build as pkg_build
    if not os.path.exists(pkg_build.FLOOR_LIB_PATH):
        raise ImportError(f"{pkg_build.FLOOR_LIB_PATH} is not built")
    lib = ctypes.CDLL(pkg_build.FLOOR_LIB_PATH)
    lib.bevpool_floor.argtypes = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_void_p, ctypes.c_int64,
                                  ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p]
    lib.bevpool_floor.restype = ctypes.c_int
    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    w = wl.make(args.workload, seed=0)
    nbytes = algorithmic_bytes(w)
    out_bytes = w.batch * w.rig.n_cells * w.channels * 4
    in_bytes = (nbytes - out_bytes + 15) // 16 * 16
    src = torch.ones(in_bytes // 4, dtype=torch.float32, device=dev)
    dst = torch.empty(out_bytes // 4, dtype=torch.float32, device=dev)
    flush = torch.zeros(FLUSH_BYTES // 4, dtype=torch.float32, device=dev)
    flush_out = torch.zeros((), dtype=torch.float32, device=dev)
    stream = torch.cuda.current_stream(dev)
    res = {}
    for name, mode in (("empty", 0), ("read", 1), ("write", 2), ("read_write", 3)):
        times = []
        for k in range(args.warmup + args.steps):
            torch.sum(flush, dim=0, out=flush_out)
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record(stream)               # torch creates the HIP events on first record;
            e1.record(stream)               # the launch then records both again
            rc = lib.bevpool_floor(src.data_ptr(), in_bytes, dst.data_ptr(), out_bytes, mode,
                                   stream.cuda_stream, e0.cuda_event, e1.cuda_event)
            if rc != 0:
                raise RuntimeError(f"bevpool_floor mode {mode} failed")
            if k >= args.warmup:
                times.append((e0, e1))
        torch.cuda.synchronize()
        us = np.array([a.elapsed_time(b) for a, b in times]) * 1e3
        res[name] = {"mean_us": round(float(us.mean()), 2), "median_us": round(float(np.median(us)), 2),
                     "min_us": round(float(us.min()), 2)}
    rw = res["read_write"]["mean_us"]
    rec = {"floor": True, "workload": WORKLOAD_TEXT[args.workload], "name": args.workload,
           "read_bytes": in_bytes, "write_bytes": out_bytes, "steps": args.steps,
           "launch": "8 workgroups of 256 per CU, 16-byte accesses", **res,
           "read_write_gbs": round(nbytes / (rw * 1e-6) / 1e9, 1),
           "read_write_frac_of_peak": round(nbytes / (rw * 1e-6) / 1e9 / HBM_PEAK_GBS, 4),
           "device": torch.cuda.get_device_name(dev)}
    print(json.dumps(rec), flush=True)


def algorithmic_bytes(w) -> int:
    """P and F read once, the BEV map written once (fp32)."""
    rig = w.rig
    esize = 4 if w.dtype == "f32" else 2
    p = w.batch * rig.n_points * esize
    f = w.batch * rig.n_pixels * w.channels * esize
    o = w.batch * rig.n_cells * w.channels * 4
    return p + f + o


def kernel_hash(paths=None) -> str:
    """sha256[:16] over the forward's sources (names and contents, in order)."""
    h = hashlib.sha256()
    for path in (FORWARD_SOURCES if paths is None else paths):
        with open(path, "rb") as fh:
            h.update(os.path.relpath(path, ROOT).encode() + b"\0" + fh.read() + b"\0")
    return h.hexdigest()[:16]


def load_traffic(workload: str):
    """Counter-measured HBM bytes per launch, if they were taken for the
    current kernel source (else None)."""
    try:
        with open(TRAFFIC_FILE) as fh:
            rec = json.load(fh)
    except (OSError, ValueError):
        return None
    entry = rec.get("workloads", {}).get(workload)
    if not entry or rec.get("kernel_sha256_16") != kernel_hash():
        return None
    return entry.get("hbm_bytes_per_launch")


def cpu_model() -> str:
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return platform.processor() or "unknown"


def cpu_baseline(w, nbytes: int, budget_s: float):
    """The oracle as it stands (C, gcc -O3, fp64 accumulation), on the host
    cores: whole frames of the same workload, first with OpenMP over every
    host thread (channels split across threads) for about half of budget_s,
    then single-threaded for the rest (at least one frame each). `value` is
    the faster leg and `cores` its thread count; both legs are reported."""
    import oracle
    omp_threads = oracle.max_threads()
    t0 = time.perf_counter()
    cop = oracle.cell_map(w.rig)
    plan_s = time.perf_counter() - t0
    per_frame_bytes = nbytes / w.batch

    def leg(threads: int, seconds: float):
        oracle.set_threads(threads)
        frames, spent = 0, 0.0
        while frames == 0 or (spent < seconds and frames < 64):
            b = frames % w.batch
            t0 = time.perf_counter()
            oracle.pool(w.rig, cop, w.P[b:b + 1], w.F[b:b + 1])
            spent += time.perf_counter() - t0
            frames += 1
        return frames, spent

    try:
        f_omp, s_omp = leg(omp_threads, budget_s / 2)
        f_one, s_one = leg(1, budget_s / 2)
    finally:
        oracle.set_threads(omp_threads)
    model = cpu_model()
    # the faster of the two legs is the baseline (channel-sliced threads each
    # scan every point, which can lose to one thread)
    omp_rate, one_rate = per_frame_bytes * f_omp / s_omp, per_frame_bytes * f_one / s_one
    best_threads = omp_threads if omp_rate >= one_rate else 1
    return {
        "value": round(max(omp_rate, one_rate) / 1e9, 4),
        "unit": "GB/s",
        "cores": best_threads,
        "kind": "oracle",
        "sample": f"{f_omp} whole frame(s) of the same workload on {omp_threads} OpenMP threads, "
                  f"{s_omp:.1f} s of pooling ({s_omp / f_omp * 1e3:.0f} ms/frame); single-threaded "
                  f"{f_one} frame(s), {s_one:.1f} s ({s_one / f_one * 1e3:.0f} ms/frame); value is the "
                  f"faster leg ({best_threads} thread(s)); cell map "
                  f"{plan_s * 1e3:.0f} ms; host CPU {model}, os.cpu_count()={os.cpu_count()}",
        "omp_threads": omp_threads,
        "omp": {"value": round(omp_rate / 1e9, 4), "unit": "GB/s", "cores": omp_threads,
                "ms_per_frame": round(s_omp / f_omp * 1e3, 1), "frames": f_omp},
        "single_thread": {"value": round(per_frame_bytes * f_one / s_one / 1e9, 4), "unit": "GB/s",
                          "cores": 1, "ms_per_frame": round(s_one / f_one * 1e3, 1),
                          "frames": f_one},
        "cell_map_ms": round(plan_s * 1e3, 1),
        "cpu_model": model,
        "os_cpu_count": os.cpu_count(),
        "build": "gcc -O3 -ffp-contract=off -fno-fast-math -fopenmp",
    }


BWD_METRIC = ("BEV-pool backward ms + HBM GB/s (gradients of P and F), 6cam×118D×32×88×C80"
              "→360×360 BEV, 1 GPU")


def backward_list_bytes(rig, cells):
    """Bytes of a plan's backward lists for the cell map ``cells``: one list for
    each camera, 4 columns and 16 rows, 36 bytes for each of its slots and 4 for
    its place. A depth bin has as many slots as the most pieces that its rows form
    in one of the columns (a piece ends where a kept row's cell is another one),
    and lies within 16 slots: empty slots before it fill the 16."""
    import numpy as np
    N, D, H, W = rig.n_cams, rig.n_depth, rig.feat_h, rig.feat_w
    hb, wb = -(-H // 16), -(-W // 4)
    x = np.full((N, D, hb * 16, wb * 4), -1, np.int32)
    x[:, :, :H, :W] = np.asarray(cells).reshape(N, D, H, W)
    x = x.reshape(N, D, hb, 16, wb * 4)
    last = np.full((N, D, hb, wb * 4), -1, np.int32)
    pieces = np.zeros(last.shape, np.int64)
    for r in range(16):
        c = x[:, :, :, r]
        pieces += (c >= 0) & (c != last)
        last = np.where(c >= 0, c, last)
    most = np.maximum(1, pieces.reshape(N, D, hb, wb, 4).max(axis=-1))
    at = np.zeros((N, hb, wb), np.int64)
    for d in range(D):
        n = most[:, d]
        at = np.where(at % 16 + n > 16, (at // 16 + 1) * 16, at) + n
    return int(36 * at.sum() + 4 * (N * hb * wb + 1))


def backward_bench(args):
    """bevpool_backward on the workload: P, F and a standard-normal gradient
    of the BEV map resident in HBM; each timed call after a cache-evicting
    read, timed by events recorded as stream entries around the call.
    Algorithmic bytes: P, F and the gradient rows of the non-empty cells
    read, dP and dF written (the plan's combo table is reported beside them)."""
    import numpy as np
    import torch
    import workloads as wl
    import paper_2205_13542_amd as bp
    import oracle

    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    w = wl.make(args.workload, seed=0)
    tdt = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[w.dtype]
    P = torch.from_numpy(w.P).to(dev).to(tdt).contiguous()
    F = torch.from_numpy(w.F).to(dev).to(tdt).contiguous()
    rng = np.random.default_rng(1)
    G_host = rng.standard_normal((w.batch, w.rig.ny, w.rig.nx, w.channels)).astype(np.float32)
    G = torch.from_numpy(G_host).to(dev)
    flush = torch.zeros(FLUSH_BYTES // 4, dtype=torch.float32, device=dev)
    flush_out = torch.zeros((), dtype=torch.float32, device=dev)
    stream = torch.cuda.current_stream(dev)
    plan = bp.Plan.from_rig(w.rig, stream=stream)
    info = plan.info
    for _ in range(args.warmup):
        torch.sum(flush, dim=0, out=flush_out)
        plan.backward(G, P, F, stream=stream)
    torch.cuda.synchronize()
    ms = []
    for _ in range(args.steps):
        torch.sum(flush, dim=0, out=flush_out)
        s0, s1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        s0.record(stream)
        plan.backward(G, P, F, stream=stream)
        s1.record(stream)
        torch.cuda.synchronize()
        ms.append(s0.elapsed_time(s1))
    ms = np.array(ms)
    esize = 4 if w.dtype == "f32" else 2
    per_frame = (w.rig.n_points * esize + w.rig.n_pixels * w.channels * esize
                 + info.n_nonempty * w.channels * 4
                 + w.rig.n_points * 4 + w.rig.n_pixels * w.channels * 4)
    nbytes = per_frame * w.batch
    mean_ms = float(ms.mean())
    gbs = nbytes / (mean_ms * 1e-3) / 1e9
    rec = {
        "metric": BWD_METRIC, "value": round(gbs, 2), "unit": "GB/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": round(mean_ms, 5),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": w.dtype,
        "data": "synthetic",
        "config": {"workload": WORKLOAD_TEXT[args.workload], "name": args.workload,
                   "batch": w.batch, "outputs": "dP and dF"},
        "roofline": {"bound": "hbm", "achieved": round(gbs, 2), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": round(gbs / HBM_PEAK_GBS, 4), "traffic": None},
        "backward_us": {"mean": round(mean_ms * 1e3, 2),
                        "median": round(float(np.median(ms)) * 1e3, 2),
                        "min": round(float(ms.min()) * 1e3, 2)},
        "algorithmic_bytes": nbytes,
        # the lists of the matrix-core kernel, which takes every workload here:
        # cells, masks and bin of each slot, and the lists' first slots
        "plan_bytes_read": backward_list_bytes(w.rig, plan.export()[0]),
        "kernel_sha256_16": kernel_hash([BWD_SOURCE]),
    }
    if not args.no_cpu_baseline:
        cop = oracle.cell_map(w.rig)
        frames, spent = 0, 0.0
        while frames == 0 or (spent < args.cpu_seconds / 2 and frames < 16):
            b = frames % w.batch
            t0 = time.perf_counter()
            oracle.backward(w.rig, cop, w.P[b:b + 1], w.F[b:b + 1], G_host[b:b + 1])
            spent += time.perf_counter() - t0
            frames += 1
        rec["cpu_baseline"] = {
            "value": round(per_frame * frames / spent / 1e9, 4), "unit": "GB/s",
            "cores": oracle.max_threads(), "kind": "oracle",
            "sample": f"{frames} whole frame(s) of the same workload, {spent:.1f} s "
                      f"({spent / frames * 1e3:.0f} ms/frame); host CPU {cpu_model()}, "
                      f"os.cpu_count()={os.cpu_count()}"}
    plan.close()
    print(json.dumps(rec), flush=True)


def reduce_bench(args):
    """bevpool_forward_ex with --reduce mean/max, or --slabs nz z slabs
    (one plan per slab, each writing its channel block of one map): timed by
    events recorded as stream entries around the call, each call after a
    cache-evicting read. Algorithmic bytes: P and F read once, the map
    (nz x C channels per cell) written once; each slab's call reads P and F
    again, which the figure does not credit."""
    import dataclasses
    import numpy as np
    import torch
    import workloads as wl
    import paper_2205_13542_amd as bp
    import oracle

    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    w = wl.make(args.workload, seed=0)
    nz = args.slabs
    rig = w.rig if nz == 1 else dataclasses.replace(w.rig, z_min=-8.0, z_cell=4.0)
    tdt = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[w.dtype]
    P = torch.from_numpy(w.P).to(dev).to(tdt).contiguous()
    F = torch.from_numpy(w.F).to(dev).to(tdt).contiguous()
    flush = torch.zeros(FLUSH_BYTES // 4, dtype=torch.float32, device=dev)
    flush_out = torch.zeros((), dtype=torch.float32, device=dev)
    stream = torch.cuda.current_stream(dev)
    sp = bp.SlabPlan.from_rig(rig, nz, stream=stream)
    out = torch.empty((w.batch, rig.ny, rig.nx, nz * w.channels), dtype=torch.float32, device=dev)
    for _ in range(args.warmup):
        torch.sum(flush, dim=0, out=flush_out)
        sp.forward(P, F, out=out, stream=stream, reduce=args.reduce)
    torch.cuda.synchronize()
    ms = []
    for _ in range(args.steps):
        torch.sum(flush, dim=0, out=flush_out)
        s0, s1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        s0.record(stream)
        sp.forward(P, F, out=out, stream=stream, reduce=args.reduce)
        s1.record(stream)
        torch.cuda.synchronize()
        ms.append(s0.elapsed_time(s1))
    ms = np.array(ms)
    esize = 4 if w.dtype == "f32" else 2
    per_frame = (rig.n_points * esize + rig.n_pixels * w.channels * esize
                 + rig.n_cells * nz * w.channels * 4)
    nbytes = per_frame * w.batch
    mean_ms = float(ms.mean())
    gbs = nbytes / (mean_ms * 1e-3) / 1e9
    what = f"{args.reduce}" + (f", {nz} z slabs of 4 m from -8 m (C x {nz} channels)" if nz > 1 else "")
    rec = {
        "metric": f"BEV-pool forward ({what}) ms + HBM GB/s, 1 GPU", "value": round(gbs, 2),
        "unit": "GB/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": round(mean_ms, 5), "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": w.dtype, "data": "synthetic",
        "config": {"workload": WORKLOAD_TEXT[args.workload], "name": args.workload,
                   "batch": w.batch, "reduce": args.reduce, "slabs": nz},
        "roofline": {"bound": "hbm", "achieved": round(gbs, 2), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": round(gbs / HBM_PEAK_GBS, 4), "traffic": None},
        "forward_us": {"mean": round(mean_ms * 1e3, 2),
                       "median": round(float(np.median(ms)) * 1e3, 2),
                       "min": round(float(ms.min()) * 1e3, 2)},
        "algorithmic_bytes": nbytes,
        "kernel_sha256_16": kernel_hash(),
    }
    if not args.no_cpu_baseline:
        frames, spent = 0, 0.0
        cop = oracle.cell_map(rig, nz)
        grid = oracle.slab_grid(rig, nz)
        while frames == 0 or (spent < args.cpu_seconds / 2 and frames < 16):
            b = frames % w.batch
            t0 = time.perf_counter()
            if args.reduce == "sum":
                oracle.pool(grid, cop, w.P[b:b + 1], w.F[b:b + 1])
            else:
                oracle.pool_reduce(grid, cop, w.P[b:b + 1], w.F[b:b + 1], args.reduce)
            spent += time.perf_counter() - t0
            frames += 1
        rec["cpu_baseline"] = {
            "value": round(per_frame * frames / spent / 1e9, 4), "unit": "GB/s",
            "cores": oracle.max_threads(), "kind": "oracle",
            "sample": f"{frames} whole frame(s) of the same workload, {spent:.1f} s "
                      f"({spent / frames * 1e3:.0f} ms/frame); host CPU {cpu_model()}, "
                      f"os.cpu_count()={os.cpu_count()}"}
    sp.close()
    print(json.dumps(rec), flush=True)


def cumsum_trick_pool(P, F, sorted_point, cell_start, rig, C, inner_scan=False):
    """The prior art the paper compares against (Sec. III-B, "Interval
    Reduction"): lift every kept point in cell order into a K x C array,
    take the prefix sum over all points, and subtract the prefix at each
    cell's interval boundaries. Written with PyTorch tensor ops on the GPU,
    as that implementation is; it reuses the plan's association (the sort
    is not timed), so only the aggregation is compared. P [1][N][D][H][W],
    F [1][N][H][W][C] fp32 device tensors; sorted_point, cell_start int64
    device tensors. Returns fp32 [1][ny][nx][C]. inner_scan: run the prefix
    sum along the innermost dimension of a transposed copy (PyTorch's
    parallel scan) instead of along the points dimension as laid out."""
    import torch
    HW = rig.feat_h * rig.feat_w
    DHW = rig.n_depth * HW
    pix = (sorted_point // DHW) * HW + sorted_point % HW
    x = P.reshape(-1)[sorted_point].unsqueeze(1) * F.reshape(-1, C)[pix]
    if inner_scan:
        prefix = torch.cumsum(x.t().contiguous(), dim=1).t()
    else:
        prefix = torch.cumsum(x, dim=0)
    counts = cell_start[1:] - cell_start[:-1]
    nonempty = torch.nonzero(counts > 0).squeeze(1)
    ends = prefix[cell_start[1:][nonempty] - 1]
    sums = torch.cat((ends[:1], ends[1:] - ends[:-1]))
    out = torch.zeros((rig.n_cells, C), dtype=torch.float32, device=P.device)
    out[nonempty] = sums
    return out.view(1, rig.ny, rig.nx, C)


def cumsum_bench(args):
    """The prefix-sum pooling and the forward on the same frame (cold caches,
    events around each call): the speed ratio the paper reports between the
    two (500 ms -> 2 ms on its GPU) measured on MI355X."""
    import numpy as np
    import torch
    import workloads as wl
    import paper_2205_13542_amd as bp

    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    w = wl.make(args.workload, seed=0)
    assert w.batch == 1 and w.dtype == "f32"
    stream = torch.cuda.current_stream(dev)
    plan = bp.Plan.from_rig(w.rig, stream=stream)
    _, sp, cs = plan.export()
    spd = torch.from_numpy(sp.astype(np.int64)).to(dev)
    csd = torch.from_numpy(cs.astype(np.int64)).to(dev)
    P = torch.from_numpy(w.P).to(dev)
    F = torch.from_numpy(w.F).to(dev)
    flush = torch.zeros(FLUSH_BYTES // 4, dtype=torch.float32, device=dev)
    flush_out = torch.zeros((), dtype=torch.float32, device=dev)

    def timed(fn, steps):
        ms = []
        for _ in range(steps):
            torch.sum(flush, dim=0, out=flush_out)
            s0, s1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            s0.record(stream)
            fn()
            s1.record(stream)
            torch.cuda.synchronize()
            ms.append(s0.elapsed_time(s1))
        return np.array(ms)

    run_cs = lambda: cumsum_trick_pool(P, F, spd, csd, w.rig, w.channels)
    run_ci = lambda: cumsum_trick_pool(P, F, spd, csd, w.rig, w.channels, inner_scan=True)
    run_fw = lambda: plan.forward(P, F, stream=stream)
    timed(run_cs, args.warmup)
    timed(run_ci, args.warmup)
    timed(run_fw, args.warmup)
    cs_ms = timed(run_cs, max(5, args.steps // 5))
    ci_ms = timed(run_ci, args.steps)
    fw_ms = timed(run_fw, args.steps)
    a, ai, b = run_cs(), run_ci(), run_fw()
    torch.cuda.synchronize()
    diff = float((a - b).abs().max())
    diff_i = float((ai - b).abs().max())
    K = int(cs[-1])
    rec = {
        "metric": "BEV-pool aggregation: prefix-sum pooling vs interval forward, ms, 1 GPU",
        "value": round(float(cs_ms.mean()) / float(fw_ms.mean()), 1), "unit": "x (speed ratio)",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": round(float(fw_ms.mean()), 5), "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": WORKLOAD_TEXT[args.workload], "name": args.workload,
                   "kept_points": K, "lifted_bytes": K * w.channels * 4},
        "prefix_sum_ms": {"mean": round(float(cs_ms.mean()), 4),
                          "median": round(float(np.median(cs_ms)), 4)},
        "prefix_sum_inner_scan_ms": {"mean": round(float(ci_ms.mean()), 4),
                                     "median": round(float(np.median(ci_ms)), 4),
                                     "ratio_to_forward": round(float(ci_ms.mean()) / float(fw_ms.mean()), 1),
                                     "max_abs_difference": diff_i},
        "forward_ms": {"mean": round(float(fw_ms.mean()), 5),
                       "median": round(float(np.median(fw_ms)), 5)},
        "max_abs_difference": diff,
        "paper": "500 ms -> 2 ms (250x) on an RTX 3090, Sec. III-B",
    }
    plan.close()
    print(json.dumps(rec), flush=True)


def nchw_bench(args):
    """bevpool_to_nchw of the workload's pooled map, alone: [B][ny][nx][C]
    rows to [B][C][ny][nx] planes, each call after a cache-evicting read,
    timed by events around the call. Algorithmic bytes: the map read once
    and written once."""
    import numpy as np
    import torch
    import workloads as wl
    import paper_2205_13542_amd as bp

    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    w = wl.make(args.workload, seed=0)
    stream = torch.cuda.current_stream(dev)
    plan = bp.Plan.from_rig(w.rig, stream=stream)
    bev = plan.forward(torch.from_numpy(w.P).to(dev), torch.from_numpy(w.F).to(dev), stream=stream)
    out = torch.empty((w.batch, w.channels, w.rig.ny, w.rig.nx), dtype=torch.float32, device=dev)
    flush = torch.zeros(FLUSH_BYTES // 4, dtype=torch.float32, device=dev)
    flush_out = torch.zeros((), dtype=torch.float32, device=dev)
    for _ in range(args.warmup):
        torch.sum(flush, dim=0, out=flush_out)
        bp.to_nchw(bev, out=out, stream=stream)
    torch.cuda.synchronize()
    ms = []
    for _ in range(args.steps):
        torch.sum(flush, dim=0, out=flush_out)
        s0, s1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        s0.record(stream)
        bp.to_nchw(bev, out=out, stream=stream)
        s1.record(stream)
        torch.cuda.synchronize()
        ms.append(s0.elapsed_time(s1))
    ms = np.array(ms)
    nbytes = 2 * bev.numel() * 4
    mean_ms = float(ms.mean())
    gbs = nbytes / (mean_ms * 1e-3) / 1e9
    rec = {
        "metric": "BEV map NHWC->NCHW copy ms + HBM GB/s, 1 GPU", "value": round(gbs, 2),
        "unit": "GB/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": round(mean_ms, 5), "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": WORKLOAD_TEXT[args.workload], "name": args.workload,
                   "batch": w.batch, "map": [w.batch, w.rig.ny, w.rig.nx, w.channels]},
        "roofline": {"bound": "hbm", "achieved": round(gbs, 2), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": round(gbs / HBM_PEAK_GBS, 4), "traffic": None},
        "copy_us": {"mean": round(mean_ms * 1e3, 2), "median": round(float(np.median(ms)) * 1e3, 2),
                    "min": round(float(ms.min()) * 1e3, 2)},
        "algorithmic_bytes": nbytes,
    }
    plan.close()
    print(json.dumps(rec), flush=True)


def main():
    args = parse_args()
    if args.gpus != 1:
        print(f"bench.py: this build runs on one GPU only; --gpus {args.gpus} is not supported "
              "(the pooling shards by BEV tiles or frames without a collective; see the design "
              "notes)", file=sys.stderr)
        sys.exit(2)
    if args.copy_calibration:
        copy_calibration()
        return
    if args.floor:
        floor_bench(args)
        return
    if args.backward:
        backward_bench(args)
        return
    if args.nchw:
        nchw_bench(args)
        return
    if args.cumsum:
        cumsum_bench(args)
        return
    if args.reduce != "sum" or args.slabs != 1:
        reduce_bench(args)
        return

    import numpy as np
    import torch
    import workloads as wl
    import paper_2205_13542_amd as bp

    if not torch.cuda.is_available():
        print("bench.py: no GPU visible", file=sys.stderr)
        sys.exit(1)
    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)

    w = wl.make(args.workload, seed=0)
    tdt = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[w.dtype]
    P = torch.from_numpy(w.P).to(dev).to(tdt).contiguous()
    F = torch.from_numpy(w.F).to(dev).to(tdt).contiguous()
    out = torch.empty((w.batch, w.rig.ny, w.rig.nx, w.channels), dtype=torch.float32, device=dev)
    flush = torch.zeros(FLUSH_BYTES // 4, dtype=torch.float32, device=dev)
    flush_out = torch.zeros((), dtype=torch.float32, device=dev)

    def evict():
        torch.sum(flush, dim=0, out=flush_out)
    stream = torch.cuda.current_stream(dev)

    # plan build (once per calibration; reported separately, not the metric):
    # the first build, then PLAN_REBUILDS more, each synchronous, and the
    # export of the association to host arrays
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    plan = bp.Plan.from_rig(w.rig, stream=stream)
    plan_ms = [(time.perf_counter() - t0) * 1e3]
    for _ in range(PLAN_REBUILDS):
        t0 = time.perf_counter()
        extra = bp.Plan.from_rig(w.rig, stream=stream)
        plan_ms.append((time.perf_counter() - t0) * 1e3)
        extra.close()
    t0 = time.perf_counter()
    cop_host, _, _ = plan.export()
    export_ms = (time.perf_counter() - t0) * 1e3
    # a plan from the stored association (bevpool_plan_import), as a cache would
    t0 = time.perf_counter()
    bp.Plan.from_cells(cop_host, w.rig, stream=stream).close()
    import_ms = (time.perf_counter() - t0) * 1e3
    info = plan.info

    for _ in range(args.warmup):
        evict()
        plan.forward(P, F, out=out, stream=stream)
    torch.cuda.synchronize()

    # Timed region: each forward runs after a cache-evicting read. Its GPU
    # time comes from kernel-boundary events, recorded by the forward's own
    # first and last kernel dispatch (bevpool_forward_timed).
    starts = [torch.cuda.Event(enable_timing=True) for _ in range(args.steps)]
    ends = [torch.cuda.Event(enable_timing=True) for _ in range(args.steps)]
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for k in range(args.steps):
        evict()
        plan.forward(P, F, out=out, stream=stream, events=(starts[k], ends[k]))
    torch.cuda.synchronize()
    wall_s = time.perf_counter() - t0
    cold_ms = np.array([s.elapsed_time(e) for s, e in zip(starts, ends)])

    # The same, bracketed by events recorded as stream entries before and
    # after the call (includes the queue gaps around the dispatch).
    outer_ms = []
    for k in range(min(args.steps, 20)):
        evict()
        s0, s1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        s0.record(stream)
        plan.forward(P, F, out=out, stream=stream)
        s1.record(stream)
        torch.cuda.synchronize()
        outer_ms.append(s0.elapsed_time(s1))

    # warm: back-to-back launches, no eviction (the whole working set fits
    # the 256 MB Infinity Cache); secondary figure
    warm_steps = max(10, args.steps)
    ws = torch.cuda.Event(enable_timing=True)
    we = torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    ws.record(stream)
    for _ in range(warm_steps):
        plan.forward(P, F, out=out, stream=stream)
    we.record(stream)
    torch.cuda.synchronize()
    warm_ms = ws.elapsed_time(we) / warm_steps

    nbytes = algorithmic_bytes(w)
    mean_ms = float(cold_ms.mean())
    gbs = nbytes / (mean_ms * 1e-3) / 1e9
    traffic = load_traffic(args.workload)
    rec = {
        "metric": METRIC,
        "value": round(gbs, 2),
        "unit": "GB/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(mean_ms, 5),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": w.dtype,
        "data": "synthetic",
        "config": {
            "workload": WORKLOAD_TEXT[args.workload],
            "name": args.workload,
            "batch": w.batch,
            "cameras": w.rig.n_cams, "depth_bins": w.rig.n_depth,
            "feat_hw": [w.rig.feat_h, w.rig.feat_w], "channels": w.channels,
            "bev": [w.rig.ny, w.rig.nx],
            "points": info.n_points, "kept": info.n_kept,
            "nonempty_cells": info.n_nonempty, "max_per_cell": info.max_per_cell,
            "column_cells": info.n_column, "generic_cells": info.n_generic,
            "generic_runs": info.n_runs, "empty_cells": info.n_empty,
        },
        "roofline": {
            "bound": "hbm",
            "achieved": round(gbs, 2),
            "peak": HBM_PEAK_GBS,
            "unit": "GB/s",
            "frac": round(gbs / HBM_PEAK_GBS, 4),
            "traffic": traffic,
        },
        "forward_us": {"mean": round(mean_ms * 1e3, 2),
                       "median": round(float(np.median(cold_ms)) * 1e3, 2),
                       "min": round(float(cold_ms.min()) * 1e3, 2),
                       "p90": round(float(np.percentile(cold_ms, 90)) * 1e3, 2),
                       "outer_events_mean": round(float(np.mean(outer_ms)) * 1e3, 2),
                       "warm_mean": round(warm_ms * 1e3, 2)},
        "algorithmic_bytes": nbytes,
        # the HBM bytes the counters measured for these kernel sources, per
        # unit time and against the algorithmic bytes
        "counter_traffic": None if traffic is None else {
            "bytes": traffic, "GBps": round(traffic / (mean_ms * 1e-3) / 1e9, 2),
            "vs_algorithmic": round(traffic / nbytes, 3)},
        "plan_bytes_read": 8 * info.n_planes * info.n_cams * info.n_depth * info.feat_w
                           + 16 * info.n_generic
                           + 16 * info.n_runs + 4 * info.n_empty
                           + 4 * (info.n_multi * (10 + 8) + 1),
        "frames_per_s": round(w.batch / (mean_ms * 1e-3), 1),
        # a plan is built once per calibration; this many frames' forward
        # time equals one rebuild
        "plan_rebuild_in_frames": round(float(np.median(plan_ms[1:])) / (mean_ms / w.batch), 1),
        "plan_build_ms": round(plan_ms[0], 2),
        "plan": {"build_ms_first": round(plan_ms[0], 2),
                 "build_ms_median": round(float(np.median(plan_ms[1:])), 2),
                 "build_ms_min": round(float(np.min(plan_ms[1:])), 2),
                 "rebuilds": PLAN_REBUILDS,
                 "export_ms": round(export_ms, 2),
                 "import_ms": round(import_ms, 2)},
        "wall_s_timed_loop": round(wall_s, 4),
        "kernel_sha256_16": kernel_hash(),
        "device": torch.cuda.get_device_name(dev),
    }
    if not args.no_cpu_baseline:
        rec["cpu_baseline"] = cpu_baseline(w, nbytes, args.cpu_seconds)
    plan.close()
    print(json.dumps(rec), flush=True)


if __name__ == "__main__":
    main()
