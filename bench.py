"""Benchmark: TOD samples/s per PCG iteration of the map-making solve on one MI355X.

Workload (default, the largest single-GPU configuration): TQU polarisation,
256 detectors x 2^22 samples = 2^30 samples, a 4096 x 12288 (12 x 2048^2)
pixel raster, a 2 Hz half-wave plate, stationary intervals log-uniform in
[2^16, 2^22], per-detector 1/f noise, correlation length 8192, and 8 noise
realisations solved together as right-hand sides; float32 TOD and weights,
mixed-precision PCG (float32 filtering and scatter, float64 CG, float64
residual replacement) to relative residual 1e-8.  The inputs are generated on
the device (synthetic; they stand in for the paper's simulated focal planes).

One step = the whole hot path on inputs resident in HBM: plan (pixel sort,
observed compaction, filters, preconditioner) in a workspace from torch's
caching allocator, right-hand sides, PCG iterations of every RHS to
tolerance, maps out.  value = samples x (iterations summed over RHS) / step
time, i.e. TOD samples per second per PCG iteration, whole job.

Also reported (JSON keys):
  iteration_roofline  one PCG iteration of all RHS (fixed-iteration solves on a
                      persistent plan) against the staged model's bytes and the
                      fused-floor ceiling, at 8 TB/s and against a device copy;
  roofline            the dominant kernel, the overlap-save N^-1 transform, timed
                      alone (HIP events on its launch stream) and placed on the
                      HBM roofline with the method's work at the paper's n_f
                      (4 n_f/m + 4 bytes and (5 n_f log2 n_f + n_f)/m flops per
                      sample); the flops it executes at the library's n_f beside;
                      traffic from the HBM counters when they were taken for this
                      kernel source and workload;
  time_to_solution    plain FP64 PCG vs mixed at the same map error (measured
                      against an FP64 map at 1e-11), on a stated RHS subset when
                      the two plans do not fit beside the full batch;
  cpu_baseline        the FP64 oracle's H on a host copy of one detector, and
                      its direct-convolution N^-1 on a bounded prefix.

--workload c2 / c3 run the smaller configurations.  --profile-filter only
launches the filter (for counter runs); --traffic-from turns the counter CSVs
of such runs into the traffic record this script reads.
"""

from __future__ import annotations

import argparse
import csv
import glob
import hashlib
import json
import math
import os
import subprocess
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0
FP32_PEAK_TFLOPS = 157.3                               # published dense vector FP32 (packed)
# Non-packed FP32 (and FP64) vector FMA issue rate: 256 CUs x 64 lanes x 2 flop x 2.4 GHz.
# Packed FP32 is not generated by this build.
VALU_NONPACKED_TFLOPS = 256 * 64 * 2 * 2.4e9 / 1e12
WORKLOADS = {
    "c2": "TQU 4 det x 2^22 samples, 256x256 px, HWP 2 Hz, intervals 2^20, n_c 8192",
    "c3": "TQU 64 det x 2^22 samples (2^28), 2^20 px, intervals log-uniform [2^14, 2^21], per-det 1/f, n_c 8192",
    "c5": "TQU 256 det x 2^22 samples (2^30), 12x2048^2 px, intervals log-uniform [2^16, 2^22], per-det 1/f, "
          "8 noise realisations as RHS, n_c 8192",
}
KERNEL_SOURCES = [os.path.join(ROOT, "paper_0906_1775_amd", "csrc", f)
                  for f in ("k_filter.hip", "k_ols_wave.hip", "fft.hpp", "sky.hpp")]


def traffic_file(workload: str) -> str:
    return os.path.join(ROOT, "profiles", f"ols_filter_{workload}_traffic.json")


def kernel_source_hash() -> str:
    h = hashlib.sha256()
    for f in KERNEL_SOURCES:
        h.update(open(f, "rb").read())
    return h.hexdigest()[:16]


def log(msg):
    print(f"[bench] {msg}", file=sys.stderr, flush=True)


def cpu_model() -> str:
    try:
        out = subprocess.run(["lscpu"], capture_output=True, text=True, timeout=10).stdout
        for line in out.splitlines():
            if line.startswith("Model name:"):
                return line.split(":", 1)[1].strip()
    except Exception:
        pass
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


# ---------------------------------------------------------------- workload

def load_workload(name, dev, n_rhs=None):
    """Device tensors and host tables of a workload."""
    import torch
    import synth
    if name == "c2":
        p = synth.make_problem("c2")
        w = dict(pix=torch.from_numpy(p.pix).to(dev), w=torch.from_numpy(p.w).to(dev), n_pix=p.n_pix,
                 iv_start=p.iv_start, iv_filter=p.iv_filter, filter_params=p.filter_params, f_samp=p.f_samp,
                 n_c=p.n_c, tod=torch.from_numpy(p.tod).to(dev), det_start=p.det_start)
    else:
        from synth.gpu import make_device_problem
        dp = make_device_problem(name, device=dev, n_rhs=n_rhs)
        w = dict(pix=dp.pix, w=dp.w, n_pix=dp.n_pix, iv_start=dp.iv_start, iv_filter=dp.iv_filter,
                 filter_params=dp.filter_params, f_samp=dp.f_samp, n_c=dp.n_c, tod=dp.tod,
                 det_start=dp.det_start)
        del dp
    torch.cuda.synchronize()
    return w


FFT_SHAPE = 0   # transform shape of every plan (--fft-shape; 0 = the library default)
N_F = 0         # FFT length of every plan (--n-f; 0 = the library's choice)


def make_plan(wl, precision, n_rhs):
    from paper_0906_1775_amd import MapMaker
    return MapMaker(wl["pix"], wl["w"], wl["n_pix"], 3, wl["iv_start"], wl["iv_filter"],
                    filter_params=wl["filter_params"], f_samp=wl["f_samp"], n_c=wl["n_c"],
                    precision=precision, n_rhs=n_rhs, fft_shape=FFT_SHAPE, n_f=N_F)


# ---------------------------------------------------------------- CPU baseline

def cpu_baseline(wl, budget_s: float = 20.0):
    """The FP64 oracle's H = P^T N^-1 P on a host copy of detector 0 (its N^-1 is a
    library-FFT convolution of each stationary interval), and, labelled separately,
    the same H with the oracle's direct-convolution N^-1 on a bounded prefix."""
    import numpy as np
    from oracle import Oracle
    n = int(wl["det_start"][1])
    iv = np.asarray(wl["iv_start"])
    nb = int(np.searchsorted(iv, n))
    iv0 = iv[:nb + 1].copy()
    used = np.unique(np.asarray(wl["iv_filter"])[:nb])
    remap = {int(f): k for k, f in enumerate(used)}
    fl0 = np.array([remap[int(f)] for f in np.asarray(wl["iv_filter"])[:nb]], np.int32)
    fp0 = np.asarray(wl["filter_params"])[used]
    pix = wl["pix"][:n].cpu().numpy()
    w = wl["w"][:n].cpu().numpy()
    orc = Oracle(pix, w, wl["n_pix"], 3, iv0, fl0, fp0, wl["f_samp"], wl["n_c"])
    x = np.random.default_rng(0).standard_normal(orc.n_unknowns)
    orc.apply_H(x)                          # warm-up
    reps, t0 = 0, time.perf_counter()
    while True:
        orc.apply_H(x)
        reps += 1
        if time.perf_counter() - t0 > budget_s / 2 or reps >= 40:
            break
    dt = (time.perf_counter() - t0) / reps
    # direct convolution (O(n_c) per sample) on a prefix of the same detector
    nd = min(n, 1 << 19)
    kd = int(np.searchsorted(iv0, nd))
    ivd = np.append(iv0[:kd][iv0[:kd] < nd], nd).astype(np.int64)
    od = Oracle(pix[:nd], w[:nd], wl["n_pix"], 3, ivd, fl0[:ivd.shape[0] - 1], fp0, wl["f_samp"], wl["n_c"])
    xd = np.random.default_rng(1).standard_normal(od.n_unknowns)
    t1 = time.perf_counter()
    od.apply_At(od.apply_ninv(od.apply_A(xd), direct=True))
    tdir = time.perf_counter() - t1
    cores = os.cpu_count()
    return dict(value=n / dt, unit="TOD samples/s per PCG iteration", cores=cores, kind="oracle",
                cpu_model=cpu_model(),
                sample=f"one H = P^T N^-1 P of the FP64 oracle on a host copy of detector 0 ({n} samples, "
                       f"{nb} stationary intervals, N^-1 by a library FFT of each interval with "
                       f"{cores} FFT worker threads, sparse products on one thread), mean of {reps}",
                direct_convolution=dict(
                    value=nd / tdir, unit="TOD samples/s per PCG iteration",
                    sample=f"the same H with the oracle's direct-convolution N^-1 (2 n_c - 1 = {2 * wl['n_c'] - 1} "
                           f"taps per sample, one thread) on the first {nd} samples of detector 0, one run"))


# ---------------------------------------------------------------- measurements

def copy_bandwidth(dev, n: int = 1 << 28, reps: int = 10):
    """Achievable HBM bandwidth: a plain device copy of n float32 (read + write bytes per second)."""
    import torch
    x = torch.ones(n, dtype=torch.float32, device=dev)
    y = torch.empty_like(x)
    for _ in range(2):
        y.copy_(x)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(reps):
        y.copy_(x)
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / reps
    del x, y
    return 2 * n * 4 / (ms * 1e-3) / 1e9


def paper_nf(n_c, iv_start):
    from paper_0906_1775_amd import fft_length_rule
    longest = int(max(b - a for a, b in zip(iv_start[:-1], iv_start[1:])))
    return fft_length_rule(n_c, longest)


def time_filter(mm, tod, precision, s, n_launch=20):
    """Mean launch time (ms) of the overlap-save N^-1 kernel: mm_weight launches only the filter;
    HIP events on the stream it is launched on."""
    import ctypes
    import torch
    from paper_0906_1775_amd import _lib as L
    y_in = tod if precision == "mixed" else tod.double()
    y_out = torch.empty_like(y_in)
    lib = L.load()
    dt = L.MM_F32 if y_in.dtype == torch.float32 else L.MM_F64

    def launch():
        L.check(lib.mm_weight(mm._h, ctypes.c_void_p(y_in.data_ptr()), ctypes.c_void_p(y_out.data_ptr()),
                              dt, ctypes.c_void_p(s.cuda_stream)), lib)
    for _ in range(3):
        launch()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record(s)
    for _ in range(n_launch):
        launch()
    e1.record(s)
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / n_launch
    del y_out, y_in
    return ms


def filter_kernel_name(precision, lib_nf, shape):
    """The overlap-save kernel a plan launches: the wavefront-private transforms for shape 1 up to
    2^13 points (float64: 2^14) and shape 10 beyond, the batched four-step one past 2^16 samples,
    the Stockham shapes otherwise."""
    logn, fp64 = lib_nf.bit_length() - 2, precision != "mixed"
    if lib_nf > 1 << 16:
        return "k_long_columns, k_long_rows, k_long_output"
    wave = shape == 10 or (shape <= 1 and 10 <= logn <= (14 if fp64 else 13))
    return "k_ols_wave" if wave else "k_ols"


def filter_roofline(ols_ms, workload, precision, n_t, R, n_c, iv_start, lib_nf, shape=0):
    """The overlap-save N^-1 kernel on the HBM roofline, with the method's work at the
    paper's FFT length: per sample and RHS, 4 n_f/m bytes read (each transform reads its
    2 n_c halo) + 4 written, and (5 n_f log2 n_f + n_f)/m flops (a real FFT of n_f points
    forward and back, 2.5 n_f log2 n_f each, and the symbol product), m = n_f - 2 n_c.  At
    the paper's n_f that is ~12 flop/B, below the FP32 ridge (157.3 / 8 = 19.7), so the
    bound is HBM.  The flops executed at the library's shorter on-chip n_f are reported
    beside it."""
    esz = 4 if precision == "mixed" else 8
    nf = paper_nf(n_c, iv_start)
    m = nf - 2 * n_c
    units = n_t * R
    b_per = esz * nf / m + esz
    f_per = (5 * nf * math.log2(nf) + nf) / m
    lm = lib_nf - 2 * n_c
    fx_per = (5 * lib_nf * math.log2(lib_nf) + lib_nf) / lm
    t = ols_ms * 1e-3
    achieved = units * b_per / t / 1e9
    traffic = None
    tf = traffic_file(workload)
    if os.path.exists(tf):
        tr = json.load(open(tf))
        if tr.get("kernel_source_hash") == kernel_source_hash() and tr.get("precision") == precision \
                and tr.get("n_sample_rhs") == units:
            traffic = tr.get("bytes_per_launch")
    name = filter_kernel_name(precision, lib_nf, shape)
    return dict(kernel=f"{name} (overlap-save N^-1; library n_f={lib_nf}, paper n_f={nf})", bound="hbm",
                achieved=round(achieved, 1), peak=HBM_PEAK_GBS, unit="GB/s", frac=round(achieved / HBM_PEAK_GBS, 4),
                traffic=traffic, launch_ms=round(ols_ms, 4), units_per_launch=units,
                bytes_per_unit=round(b_per, 4), algorithmic_bytes=round(units * b_per),
                paper_n_f=nf, flops_per_unit_paper_nf=round(f_per, 2),
                achieved_TFLOPs_paper_nf=round(units * f_per / t / 1e12, 2), fp32_peak_TFLOPs=FP32_PEAK_TFLOPS,
                library_n_f=lib_nf, executed_flops_per_unit=round(fx_per, 2),
                executed_TFLOPs=round(units * fx_per / t / 1e12, 2),
                executed_frac_of_nonpacked_valu=round(units * fx_per / t / 1e12 / VALU_NONPACKED_TFLOPS, 4))


def iteration_roofline(t_iter_ms, n_t, R, n_obs, n_c, iv_start, copy_gbs):
    """One mixed PCG iteration of all R RHS on the HBM roofline.  Staged model bytes (each
    stream moved once): the gather reads 12 B of pointing per sample (shared by the RHS)
    and writes 4 B per sample and RHS; the filter reads 4 B per sample and RHS times the
    halo ratio n_f/m of the paper's FFT-length rule and writes 4 B; the scatter reads 12 B
    of pointing and 4 B of TOD; the pixel side is 14 float64 vector passes of 3 values per
    observed pixel and RHS.  The fused floor moves the pointing once (12 B per sample) and
    no TOD, plus the same pixel side: its rate is a ceiling for any staging."""
    nf = paper_nf(n_c, iv_start)
    halo = nf / (nf - 2 * n_c)
    pixel = n_obs * R * 14 * 8 * 3
    model = n_t * (12 + 4 * R + R * (4 * halo + 4) + 12 + 4 * R) + pixel
    floor = n_t * 12 + pixel
    t = t_iter_ms * 1e-3
    gbs = model / t / 1e9
    return dict(bound="hbm", model_bytes=round(model), achieved_GBs=round(gbs, 1), peak_GBs=HBM_PEAK_GBS,
                frac=round(gbs / HBM_PEAK_GBS, 4), copy_GBs=round(copy_gbs, 1), frac_of_copy=round(gbs / copy_gbs, 4),
                staged_ceiling_sample_rhs_per_s=n_t * R / (model / (HBM_PEAK_GBS * 1e9)),
                fused_floor_bytes=round(floor),
                fused_floor_ceiling_sample_rhs_per_s=n_t * R / (floor / (HBM_PEAK_GBS * 1e9)),
                fused_floor_frac=round(floor / t / 1e9 / HBM_PEAK_GBS, 4), paper_n_f=nf)


def time_to_solution(wl, tol, n_sub):
    """Wall time to the same map error: plain FP64 PCG at tol vs the loosest mixed tolerance
    whose map is at least as close to an FP64 map at 1e-11, on the first n_sub RHS."""
    import torch
    tod = wl["tod"][:n_sub]
    ref_plan = make_plan(wl, "fp64", n_sub)
    ref, _ = ref_plan.solve(tod, tol=1e-11, max_iter=3000)
    nref = torch.linalg.norm(ref)

    def err(m):
        return float(torch.linalg.norm(m - ref) / nref)

    def tts_of(plan, t):
        plan.solve(tod, tol=t, max_iter=3000)      # warm (graph capture)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        m, inf = plan.solve(tod, tol=t, max_iter=3000)
        torch.cuda.synchronize()
        return time.perf_counter() - t0, err(m), sum(inf["iters"])
    t64, e64, i64 = tts_of(ref_plan, tol)
    ref_plan.close()
    del ref_plan
    log(f"time to solution: fp64 {t64:.3f}s at map error {e64:.3e} ({i64} iterations)")
    mx = make_plan(wl, "mixed", n_sub)
    tmx = emx = imx = None
    mtol = tol
    for mtol in (tol * 10, tol * 3, tol, tol / 3, tol / 10, tol / 30, tol / 100):
        tmx, emx, imx = tts_of(mx, mtol)
        log(f"time to solution: mixed tol {mtol:g} {tmx:.3f}s at map error {emx:.3e} ({imx} iterations)")
        if emx <= e64:
            break
    _, inf = mx.solve(tod, tol=mtol, max_iter=3000, map_error=True)
    mx.close()
    return dict(rhs=n_sub, target_map_error=e64, fp64_s=round(t64, 5), fp64_iters=i64, mixed_tol=mtol,
                mixed_s=round(tmx, 5), mixed_iters=imx, mixed_map_error=emx,
                mixed_map_error_estimate=[float(v) for v in inf["map_error"]],
                speedup=round(t64 / tmx, 3), reached=bool(emx <= e64))


# ---------------------------------------------------------------- counter runs

def traffic_from(fetch_dir, write_dir, workload, precision, n_sample_rhs, alg_bytes, command_lines):
    """Traffic record of the filter kernel from two rocprofv3 --pmc runs of --profile-filter
    (FETCH_SIZE, then WRITE_SIZE; KiB per dispatch), each scaled by what the counter reads
    for the calibration copy of 2^28 float32 that --profile-filter makes first."""
    def read(d, counter):
        rows = []
        for f in glob.glob(os.path.join(d, "**", "*counter_collection.csv"), recursive=True):
            with open(f) as fh:
                for r in csv.DictReader(fh):
                    if r.get("Counter_Name") == counter:
                        rows.append((int(r["Dispatch_Id"]), r["Kernel_Name"], float(r["Counter_Value"])))
        rows.sort()
        copies = [v for _, k, v in rows if "copyBuffer" in k][:3]
        ols = sorted(v for _, k, v in rows if "k_ols" in k)
        if len(copies) < 3 or not ols:
            raise SystemExit(f"no calibration copies or filter dispatches for {counter} under {d}")
        return sorted(copies)[1], ols[len(ols) // 2]
    cf, of = read(fetch_dir, "FETCH_SIZE")
    cw, ow = read(write_dir, "WRITE_SIZE")
    copy_bytes = (1 << 28) * 4
    fs, ws = copy_bytes / (cf * 1024), copy_bytes / (cw * 1024)
    rec = dict(kernel="k_ols_wave (overlap-save N^-1)", workload=WORKLOADS[workload], precision=precision,
               n_sample_rhs=n_sample_rhs, kernel_source_hash=kernel_source_hash(),
               fetch_kib_per_dispatch=round(of, 2), write_kib_per_dispatch=round(ow, 2),
               dispatches_used="median over the filter dispatches of the run",
               calibration=dict(kernel="copyBuffer (torch copy_ of 2^28 float32, the run's first three copies)",
                                bytes_read=copy_bytes, bytes_written=copy_bytes, fetch_kib=round(cf, 2),
                                write_kib=round(cw, 2), fetch_scale=round(fs, 4), write_scale=round(ws, 4)),
               bytes_per_launch=round(of * 1024 * fs + ow * 1024 * ws), algorithmic_bytes_per_launch=alg_bytes,
               commands=command_lines)
    json.dump(rec, open(traffic_file(workload), "w"), indent=1)
    print(json.dumps(rec))


# ---------------------------------------------------------------- main

def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=3)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--precision", default="mixed", choices=["mixed", "fp64"])
    ap.add_argument("--tol", type=float, default=1e-8)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-tts", action="store_true", help="skip the time-to-solution comparison")
    ap.add_argument("--workload", default="c5", choices=["c2", "c3", "c5"],
                    help="c5: 256 det, 2^30 samples, 8 realisations (default); c3: 64 det, 2^28 samples, "
                         "uneven intervals; c2: 4 det x 2^22 TQU")
    ap.add_argument("--tts-rhs", type=int, default=2,
                    help="RHS of the time-to-solution comparison for c5 (the FP64 and mixed plans of all 8 "
                         "do not fit beside each other)")
    ap.add_argument("--n-f", type=int, default=0,
                    help="overlap-save FFT length of the plans (mm.h n_f; 0 = library choice, -1 = autotune)")
    ap.add_argument("--fft-shape", type=int, default=0,
                    help="workgroup shape of the overlap-save transform (mm.h fft_shape; 0 = library default)")
    ap.add_argument("--profile-filter", action="store_true",
                    help="calibration copy, then plan and 3 filter launches only (for counter runs)")
    ap.add_argument("--profile-iteration", action="store_true",
                    help="calibration copy, then plan and a 2-iteration fixed solve only (for counter runs)")
    ap.add_argument("--traffic-from", nargs=2, metavar=("FETCH_DIR", "WRITE_DIR"),
                    help="write the filter's traffic record from two --pmc runs of --profile-filter")
    args = ap.parse_args()
    global FFT_SHAPE, N_F
    FFT_SHAPE = args.fft_shape
    N_F = args.n_f
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py runs on one GPU only: this build has no multi-GPU path "
              "(see the sharding design); use --gpus 1", file=sys.stderr)
        sys.exit(2)

    import torch
    dev = torch.device("cuda:0")
    if args.traffic_from:
        wl = load_workload(args.workload, dev)
        n_t, R = int(wl["pix"].shape[0]), int(wl["tod"].shape[0])
        nf = paper_nf(wl["n_c"], wl["iv_start"])
        esz = 4 if args.precision == "mixed" else 8
        alg = round(n_t * R * (esz * nf / (nf - 2 * wl["n_c"]) + esz))
        cmds = ["export TMPDIR=/tmp   # then, from the repository root:"] + [
            f"timeout -s KILL 300 rocprofv3 --pmc {c} --kernel-include-regex 'k_ols|copyBuffer' --output-format csv "
            f"-d $PWD/gpurun_out/{d} -o ols -- "
            f"python -u bench.py --workload {args.workload} --precision {args.precision} --profile-filter"
            for c, d in (("FETCH_SIZE", os.path.basename(args.traffic_from[0].rstrip("/"))),
                         ("WRITE_SIZE", os.path.basename(args.traffic_from[1].rstrip("/"))))] + [
            f"python bench.py --workload {args.workload} --precision {args.precision} --traffic-from "
            f"{args.traffic_from[0]} {args.traffic_from[1]}"]
        traffic_from(args.traffic_from[0], args.traffic_from[1], args.workload, args.precision, n_t * R, alg, cmds)
        return

    t_gen = time.perf_counter()
    if args.profile_filter or args.profile_iteration:
        copy_bandwidth(dev, reps=1)          # the calibration copies come first in the run
    wl = load_workload(args.workload, dev)
    tod = wl["tod"]
    n_t, R, n_c = int(wl["pix"].shape[0]), int(tod.shape[0]), int(wl["n_c"])
    log(f"generated {args.workload} inputs in {time.perf_counter() - t_gen:.1f}s "
        f"({n_t} samples x {R} RHS)")
    if args.profile_filter:
        mm = make_plan(wl, args.precision, R)
        ms = time_filter(mm, tod, args.precision, torch.cuda.current_stream(), n_launch=1)
        log(f"filter launch {ms:.3f} ms")
        mm.close()
        return
    if args.profile_iteration:
        mm = make_plan(wl, args.precision, R)
        mm.solve(tod, fixed_iters=2, check_every=2, use_graph=False)
        torch.cuda.synchronize()
        log("plan and 2 iterations done")
        mm.close()
        return
    copy_gbs = copy_bandwidth(dev)
    log(f"device copy {copy_gbs:.0f} GB/s (read + write)")

    def step():
        mm = make_plan(wl, args.precision, R)
        m, info = mm.solve(tod, tol=args.tol, max_iter=1000, check_every=8)
        mm.close()
        return info

    for _ in range(args.warmup):
        info = step()
        log(f"warmup step: {info['iters']} iterations, status {info['status']}")
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    iters = 0
    for _ in range(args.steps):
        info = step()
        iters += sum(info["iters"])
        log(f"step: {info['iters']} iterations")
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    ms_per_step = elapsed / args.steps * 1e3
    value = n_t * iters / elapsed
    log(f"timed {args.steps} steps: {ms_per_step:.2f} ms/step, {iters / args.steps:.1f} iterations/step")

    # ---- per-iteration time and the dominant kernel, on a persistent plan
    torch.cuda.synchronize()
    t_plan0 = time.perf_counter()
    mm = make_plan(wl, args.precision, R)
    torch.cuda.synchronize()
    plan_ms = (time.perf_counter() - t_plan0) * 1e3
    pinfo = mm.info()
    s = torch.cuda.current_stream()

    def timed_solve(k):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record(s)
        mm.solve(tod, fixed_iters=k, check_every=8)
        e1.record(s)
        torch.cuda.synchronize()
        return e0.elapsed_time(e1)

    timed_solve(8)
    t_a, t_b = timed_solve(8), timed_solve(40)
    t_iter_ms = (t_b - t_a) / 32.0
    log(f"per iteration {t_iter_ms:.3f} ms")
    ols_ms = time_filter(mm, tod, args.precision, s)
    roofline = filter_roofline(ols_ms, args.workload, args.precision, n_t, R, n_c, wl["iv_start"], pinfo["n_f"],
                               pinfo["fft_shape"])
    log(f"filter roofline {roofline}")
    iter_roof = iteration_roofline(t_iter_ms, n_t, R, pinfo["n_obs"], n_c, wl["iv_start"], copy_gbs)
    log(f"iteration roofline {iter_roof}")
    mm.close()
    del mm

    tts = None
    if not args.no_tts:
        n_sub = min(R, args.tts_rhs) if args.workload == "c5" else R
        tts = time_to_solution(wl, args.tol, n_sub)
        log(f"time to solution {tts}")

    cpu = None if args.no_cpu_baseline else cpu_baseline(wl)
    if cpu:
        log(f"cpu baseline {cpu}")

    out = {
        "metric": "TOD samples/s per PCG iteration (% HBM roofline); time-to-solution at fixed error",
        "value": value,
        "unit": "TOD samples/s per PCG iteration",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_per_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32+f64" if args.precision == "mixed" else "f64",
        "data": "synthetic (device-generated scan, HWP angles, 1/f noise of the configuration's shape)",
        "config": {"workload": WORKLOADS[args.workload] + f", {args.precision} PCG to {args.tol:g}",
                   "n_samples": n_t, "n_rhs": R, "n_obs": pinfo["n_obs"], "n_f": pinfo["n_f"], "n_c": n_c},
        "iters_per_step": iters / args.steps,
        "t_iter_ms": round(t_iter_ms, 4),
        "iter_sample_rhs_per_s": n_t * R / (t_iter_ms * 1e-3),
        "plan_ms": round(plan_ms, 2),
        "iteration_roofline": iter_roof,
        "time_to_solution": tts,
        "roofline": roofline,
        "cpu_baseline": cpu,
    }
    print(json.dumps(out))


if __name__ == "__main__":
    main()
