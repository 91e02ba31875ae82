"""Benchmark of the Lomb-Scargle periodogram hot path on one MI355X.

Default workload (lsst_200k): 200,000 objects, N_t uniform in 20..500 with
seasonal gaps, 60% sinusoids, 30% with a second harmonic, 10% pure noise;
N_f = 250,000 frequencies over [0.5, 24) cycles/day; every object's peak.
Three forms run on the same device-resident input (Section 3.4's batch mode):
  * the FP32 form with FP64 phase reduction on the whole grid -- one timed
    step is one lsp_batch call (prep, main kernel, FP64 fix-up, peaks); its
    evals/s is the line's value and its main kernel carries the roofline;
  * the learned band proposal (features, network, top bands, refine,
    fallback), trained and calibrated on independent objects before the
    timed region, under three proposal rules (network, coarse power, hybrid);
  * the plain FP64 form on the whole grid, the reference every other form's
    peaks are judged against, object by object.
The CPU oracle (FP64) checks both whole-grid forms on a sample of the first
2,000 objects and is timed on that sample on this host's cores.

Other workloads: single_4096 / single_256 (one object, full FP32 periodogram
plus peak) and batch_10k time the FP32 and FP64 forms; --method generalized
times the generalized periodogram (Section 4.11); --host-return and
--recovery run the host-return and period-recovery studies.

Prints ONE JSON line.
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

METRIC = "LS obs×freq evals/s and objects/s vs plain FP64 kernel at peak-bin agreement"
# FP32 form, algorithmic flops per eval: 4 FMA for the sums (8 flops) plus the
# recurrence, 2 mul + 2 FMA for a rotation (6 flops) or 2 FMA for the
# three-term (Chebyshev) recurrence (4 flops).
FLOPS_PER_EVAL = {"rotation": 14, "chebyshev": 12}
# Generalized FP32 form: 6 FMA for the sums (12 flops) plus the three-term
# recurrence's 2 FMA (4 flops).
FLOPS_PER_EVAL_GEN = 16
# MI355X FP32 vector peak: 256 CUs x 4 SIMDs x 2.4 GHz x 64 flops/clock/SIMD
# (32 FMA lanes per clock), the published 157.3 TFLOP/s.
PEAK_FP32_TFLOPS = 256 * 4 * 2.4e9 * 64 / 1e12
# Matrix-core form (what runs when every tuning option is left to the library):
# 4 multiply-adds per evaluation (6 generalized), each as three products of
# 11-bit halves on the FP16 matrix instructions, against their dense peak
# (1,024 flops per clock and SIMD).
FLOPS_PER_EVAL_MATRIX = {"standard": 24, "generalized": 36}
PEAK_FP16_MATRIX_TFLOPS = 256 * 4 * 2.4e9 * 1024 / 1e12
# VALU instructions per observation and lane in the compiled gfx950 loop, for
# K frequencies per lane: 4K for the sums, the recurrence (4(K-1) for rotations;
# 4 + 2(K-2) for Chebyshev), and 9-10 per-observation instructions (FP64
# phase, cvt, 2 transcendentals, moves).  K = 16 compiles to 133 and 106.
def valu_ops_per_eval(rec, k):
    if rec == "chebyshev":
        return (4 * k + 4 + 2 * (k - 2) + 10) / k
    return (4 * k + 4 * (k - 1) + 9) / k


# Generalized form: 6K for the sums, 4 + 2(K-2) for the recurrence and about
# 12 per observation (the standard form's 10 plus the two seed scalings).
def valu_ops_per_eval_gen(k):
    return (6 * k + 4 + 2 * (k - 2) + 12) / k


def roofline(args, gen, rec_name, k_lane, evals, k_ms, workload, variant=False):
    """The dominant kernel's rate against the peak of the units that it uses."""
    matrix = not (variant or args.k or args.waves or args.t_split) and \
        args.recurrence == args.wave_split == args.schedule == "auto"
    if matrix:
        flops_eval = FLOPS_PER_EVAL_MATRIX["generalized" if gen else "standard"]
        peak, valu = PEAK_FP16_MATRIX_TFLOPS, None
    else:
        flops_eval = FLOPS_PER_EVAL_GEN if gen else FLOPS_PER_EVAL[rec_name]
        peak = PEAK_FP32_TFLOPS
        valu = (valu_ops_per_eval_gen(k_lane) if gen else valu_ops_per_eval(rec_name, k_lane)) \
            * evals / (k_ms * 1e-3)
    vector = None if variant else valu
    achieved = flops_eval * evals / (k_ms * 1e-3) / 1e12
    return {
        "bound": "alu",
        "achieved": achieved,
        "peak": peak,
        "unit": "TFLOP/s",
        "frac": achieved / peak,
        "traffic": None if variant or matrix else measured_traffic(args.method, workload),
        "kernel": ("mx_gen_kernel" if gen else "mx_kernel") if matrix
        else "gen_fp32p_kernel" if gen else "fp32p_kernel",
        "kernel_ms": k_ms,
        "flops_per_eval": flops_eval,
        "evals_per_launch": int(evals),
        "matrix_cores": matrix,
        "recurrence": None if matrix else rec_name,
        "k_per_lane": None if matrix else k_lane,
        "valu_lane_ops_per_s": vector,
        "valu_issue_frac": None if vector is None else vector / (PEAK_FP32_TFLOPS * 1e12 / 2),
        "obs_read": args.obs_read,
        "seed_trig": args.seed_trig,
        "transcendentals_per_s": None if matrix else 2 * evals / k_lane / (k_ms * 1e-3),
    }


# the vector kernel's sources and the file that resolves its launch shape (waves,
# splits, items), on which the counters depend as much
KERNEL_SOURCES = {
    "standard": ["paper_2105_04006_amd/csrc/lsp_fp32p.hip", "paper_2105_04006_amd/csrc/lsp_common.h",
                 "paper_2105_04006_amd/csrc/lsp_api.hip"],
    "generalized": ["paper_2105_04006_amd/csrc/lsp_gen.hip",
                    "paper_2105_04006_amd/csrc/lsp_common.h",
                    "paper_2105_04006_amd/csrc/lsp_api.hip"],
}
TRAFFIC_FILES = {
    "standard": os.path.join(ROOT, "profiles", "fp32p_single_4096_traffic.json"),
    "generalized": os.path.join(ROOT, "profiles", "gen_fp32p_single_4096_traffic.json"),
    ("standard", "batch_10k"): os.path.join(ROOT, "profiles", "fp32p_batch_10k_traffic.json"),
    ("standard", "lsst_200k"): os.path.join(ROOT, "profiles", "fp32p_lsst_200k_traffic.json"),
}


def log(msg):
    print(msg, file=sys.stderr, flush=True)


def kernel_hash(method="standard"):
    h = hashlib.sha256()
    for rel in KERNEL_SOURCES[method]:
        with open(os.path.join(ROOT, rel), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def measured_traffic(method="standard", workload="single_4096"):
    """HBM bytes per launch from the committed rocprofv3 counter runs, if they
    were taken on the current kernel source and this workload."""
    path = TRAFFIC_FILES.get((method, workload), TRAFFIC_FILES[method])
    try:
        with open(path) as fh:
            rec = json.load(fh)
    except (OSError, ValueError):
        return None
    if rec.get("kernel_hash") != kernel_hash(method) or rec.get("workload_name") != workload:
        return None
    return rec.get("bytes_per_launch")


def cpu_baseline(w, target_evals, threads, method="standard"):
    """The oracle on a bounded sample of the same workload: every m-th bin of
    the object (one object), or every bin of the first objects (a batch)."""
    import oracle

    oracle.default()
    if w.n_obj == 1:
        stride = max(1, int(round(w.evals / target_evals)))
        bins = np.arange(0, w.n_f, stride, dtype=np.int64)
        objs = np.zeros(len(bins), dtype=np.int64)
        what = f"every {stride}th of the {w.n_f} bins ({len(bins)} bins x {w.n_obs} obs"
    else:
        per_obj = w.n_f * np.diff(w.offsets)
        k = max(1, int(np.searchsorted(np.cumsum(per_obj), target_evals)))
        stride = max(1, int(round(per_obj[:k].sum() / target_evals)))
        bins1 = np.arange(0, w.n_f, stride, dtype=np.int64)
        objs = np.repeat(np.arange(k, dtype=np.int64), len(bins1))
        bins = np.tile(bins1, k)
        what = f"every {stride}th bin of the first {k} objects ({len(bins)} (object, bin) pairs"
    t0 = time.perf_counter()
    if method == "generalized":
        vals = oracle.gen_eval_bins(w.offsets, w.t, w.y, w.dy, w.f_min, w.f_max, w.n_f, objs,
                                    bins, threads=threads)
    else:
        vals = oracle.eval_bins(w.offsets, w.t, w.y, w.f_min, w.f_max, w.n_f, objs, bins,
                                threads=threads)
    dt = time.perf_counter() - t0
    n_t = np.diff(w.offsets)
    evals = int(n_t[objs].sum())
    return {"value": evals / dt, "unit": "evals/s", "cores": threads, "kind": "oracle",
            "sample": f"{what}, {evals:.3g} evals) of the same workload, {dt:.2f} s wall"}, \
        (objs, bins, vals)


def order_code(name):
    from paper_2105_04006_amd import lsp
    return {"auto": lsp.ORDER_AUTO, "input": lsp.ORDER_INPUT, "lpt": lsp.ORDER_LPT}[name]


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=None,
                    help="timed steps (default: 20 on the three-form workloads, whose FP32 step "
                         "takes about 1.5 s, 200 on the others)")
    ap.add_argument("--warmup", type=int, default=None,
                    help="untimed warm-up steps (default: 5, or 10 with 200 timed steps)")
    ap.add_argument("--workload", default="lsst_200k",
                    help="lsst_200k (default), learned_100k, asteroids_100k: the three forms "
                         "(fp32 whole grid, learned proposal, fp64) on one batch; single_256, "
                         "single_4096, batch_10k: the FP32 and FP64 forms")
    ap.add_argument("--forms", default="fp32,learned,fp64",
                    help="forms timed on a three-form workload (comma list; fp32 always runs)")
    ap.add_argument("--proposal", default="hybrid", choices=["hybrid", "coarse", "network"],
                    help="learned form: the proposal rule timed with --steps (the others run "
                         "3 steps each for the comparison)")
    ap.add_argument("--train-objects", type=int, default=40000)
    ap.add_argument("--val-objects", type=int, default=20000)
    ap.add_argument("--oracle-objects", type=int, default=2000,
                    help="three-form workloads: the oracle checks a sample of this many "
                         "leading objects")
    ap.add_argument("--cpu-threads", type=int, default=0,
                    help="oracle threads (0: every core of this process's affinity set)")
    ap.add_argument("--no-cpu", action="store_true", help="skip the oracle baseline")
    ap.add_argument("--recurrence", default="auto", choices=["auto", "rotation", "chebyshev"])
    ap.add_argument("--k", type=int, default=0, help="frequencies per lane (0: library default)")
    ap.add_argument("--waves", type=int, default=0)
    ap.add_argument("--t-split", type=int, default=0,
                    help="single object: split of the observation axis (0: library default)")
    ap.add_argument("--wave-split", default="auto", choices=["auto", "off", "on"],
                    help="FP32 form: the waves of a workgroup split the observations")
    ap.add_argument("--schedule", default="auto", choices=["auto", "grid", "persistent"])
    ap.add_argument("--order", default="auto", choices=["auto", "input", "lpt"],
                    help="order of a batch's rows (longest first, or as given)")
    ap.add_argument("--cpu-evals", type=float, default=3e9,
                    help="oracle evaluations in the CPU-baseline sample (about 10-30 s of CPU work)")
    ap.add_argument("--fp64-steps", type=int, default=0,
                    help="timed steps of the FP64 reference form (default: 2 on a three-form "
                         "workload, else steps // 8, >= 3)")
    ap.add_argument("--mode", default="lsp", choices=["lsp", "copy"],
                    help="copy: time a plain device-to-device copy of --copy-bytes bytes "
                         "(calibrates the FETCH_SIZE / WRITE_SIZE counters)")
    ap.add_argument("--copy-bytes", type=float, default=256 * 2**20)
    ap.add_argument("--launch", default="eager", choices=["eager", "graph"],
                    help="graph: each timed FP32 step replays the call captured once as a HIP "
                         "graph (lsp_plan_*)")
    ap.add_argument("--method", default="standard", choices=["standard", "generalized"],
                    help="generalized: the periodogram with per-point errors and a floating "
                         "mean (Section 4.11), on the workload drawn with errors")
    ap.add_argument("--obs-read", default="auto", choices=["auto", "lds", "direct"],
                    help="FP32 form: observations staged in LDS, or read from global memory "
                         "after a staging pass")
    ap.add_argument("--seed-trig", default="auto", choices=["auto", "hw", "lib", "poly"],
                    help="FP32 form: sin/cos of the reduced seed phases by the hardware, the "
                         "math library's sincospif, or Taylor polynomials")
    ap.add_argument("--recovery", action="store_true",
                    help="asteroid-like population (asteroids_1k): derived vs assigned rotation "
                         "periods and the observation-cutoff curve, standard and generalized, "
                         "FP32 and FP64 forms")
    ap.add_argument("--host-return", action="store_true",
                    help="time the whole batch periodogram returned to host memory: one copy of "
                         "the device periodogram into pageable memory against the pinned-staging "
                         "pipeline (lsp_batch_to_host); PCIe-inclusive, not the headline value")
    args = ap.parse_args()
    if args.steps is None:
        args.steps = 20 if args.workload in FORM_WORKLOADS and args.mode == "lsp" else 200
    if args.warmup is None:
        args.warmup = 5 if args.steps <= 20 else 10
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (got --gpus {args.gpus}); the periodogram of "
              "independent objects would shard by object across GPUs, which is not "
              "implemented.", file=sys.stderr)
        sys.exit(2)

    import torch

    if args.mode == "copy":
        n = int(args.copy_bytes) // 4
        a = torch.ones(n, dtype=torch.float32, device="cuda:0")
        b = torch.empty_like(a)
        for _ in range(args.warmup):
            b.copy_(a)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(args.steps):
            b.copy_(a)
        torch.cuda.synchronize()
        dt = (time.perf_counter() - t0) / args.steps
        print(json.dumps({"mode": "copy", "bytes_read": 4 * n, "bytes_written": 4 * n,
                          "ms_per_copy": dt * 1e3, "GB_per_s": 8 * n / dt / 1e9}), flush=True)
        return

    from paper_2105_04006_amd import lsp, synth

    lsp.lib()  # fails loudly if the HIP library is not built
    dev = torch.device("cuda:0")
    if args.workload in FORM_WORKLOADS and not (args.host_return or args.recovery):
        return bench_forms(args, torch, dev)
    if args.host_return:
        return bench_host_return(args, torch, dev)
    if args.recovery:
        return bench_recovery(args, torch, dev)
    gen = args.method == "generalized"
    w = synth.make_workload(args.workload, errors=gen)
    single = w.n_obj == 1
    log(f"[bench] workload {w.name}: n_obj={w.n_obj} n_obs={w.n_obs} n_f={w.n_f} "
        f"evals={w.evals:.3e}")
    t = torch.as_tensor(w.t, device=dev)
    y = torch.as_tensor(w.y, device=dev)
    off = None if single else torch.as_tensor(w.offsets, device=dev)
    kw = dict(offsets=off, pgram=single, peaks=True)
    rec = {"auto": lsp.REC_AUTO, "rotation": lsp.REC_ROTATION,
           "chebyshev": lsp.REC_CHEBYSHEV}[args.recurrence]
    sched = {"auto": lsp.SCHED_AUTO, "grid": lsp.SCHED_GRID,
             "persistent": lsp.SCHED_PERSISTENT}[args.schedule]
    if gen:
        kw.update(method="generalized", dy=torch.as_tensor(w.dy, device=dev))
    obs = {"auto": 0, "lds": lsp.OBS_LDS, "direct": lsp.OBS_DIRECT}[args.obs_read]
    trig = {"auto": 0, "hw": lsp.TRIG_HW, "lib": lsp.TRIG_LIB, "poly": lsp.TRIG_POLY}[args.seed_trig]
    variant = obs == lsp.OBS_DIRECT or trig in (lsp.TRIG_LIB, lsp.TRIG_POLY)
    kv = dict(obs_read=obs, seed_trig=trig) if variant else {}
    order = order_code(args.order)
    wsp = {"auto": lsp.WSPLIT_AUTO, "off": lsp.WSPLIT_OFF, "on": lsp.WSPLIT_ON}[args.wave_split]
    p32 = lsp.Periodogram(t, y, w.f_min, w.f_max, w.n_f, form=lsp.FORM_FP32P, schedule=sched,
                          recurrence=rec, k=args.k, waves=args.waves, order=order,
                          wave_split=wsp, t_split=args.t_split, **kw, **kv)
    p64 = lsp.Periodogram(t, y, w.f_min, w.f_max, w.n_f, form=lsp.FORM_FP64, order=order, **kw)

    def timed(fn, steps):
        torch.cuda.synchronize()
        a = torch.cuda.Event(enable_timing=True)
        b = torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(steps):
            fn()
        b.record()
        torch.cuda.synchronize()
        return a.elapsed_time(b) / steps

    step32 = p32.capture() if args.launch == "graph" else p32
    for _ in range(args.warmup):
        step32()
    p64()
    torch.cuda.synchronize()
    log("[bench] warm-up done")
    ms32 = timed(step32, args.steps)
    log(f"[bench] fp32p {ms32:.4f} ms/step ({args.launch})")
    steps64 = args.fp64_steps if args.fp64_steps > 0 else max(3, args.steps // 8)
    ms64 = timed(p64, steps64)
    log(f"[bench] fp64 {ms64:.4f} ms/step ({steps64} steps)")
    std_cost = None
    if gen:
        # the standard periodogram of the same input, for the cost ratio
        kws = dict(offsets=off, pgram=single, peaks=True)  # standard, default variant
        s32 = lsp.Periodogram(t, y, w.f_min, w.f_max, w.n_f, form=lsp.FORM_FP32P, **kws)
        s64 = lsp.Periodogram(t, y, w.f_min, w.f_max, w.n_f, form=lsp.FORM_FP64, **kws)
        s32()
        s64()
        ms_s32 = timed(s32, args.steps)
        ms_s64 = timed(s64, steps64)
        std_cost = {"fp32_ms_per_step": ms_s32, "fp64_ms_per_step": ms_s64,
                    "generalized_over_standard_fp32": ms32 / ms_s32,
                    "generalized_over_standard_fp64": ms64 / ms_s64}
        log(f"[bench] standard fp32p {ms_s32:.4f} ms, fp64 {ms_s64:.4f} ms; generalized/standard "
            f"{ms32 / ms_s32:.2f}x (fp32), {ms64 / ms_s64:.2f}x (fp64)")

    # dominant kernel's own device time, from events the library records
    # around the main kernel on its launch stream
    pairs = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
             for _ in range(args.steps)]
    for a, b in pairs:
        a.record()
        b.record()
    torch.cuda.synchronize()
    for a, b in pairs:
        lsp.set_stage_events(a.cuda_event, b.cuda_event)
        p32()
    lsp.set_stage_events(None, None)
    torch.cuda.synchronize()
    k_ms = float(np.mean([a.elapsed_time(b) for a, b in pairs]))
    log(f"[bench] fp32p main kernel {k_ms:.4f} ms/launch")

    pk32, pk64 = p32.peaks(), p64.peaks()
    agree = np.abs(pk32["index"] - pk64["index"]) <= 1
    if single:
        d = (p32.pgram.double() - p64.pgram.double()).abs().max().item()
    else:
        d = float(np.max(np.abs(pk32["power"] - pk64["power"])))

    evals = w.evals
    value = evals / (ms32 * 1e-3)
    rec_name = "rotation" if p32.launch()["recurrence"] == lsp.REC_ROTATION else "chebyshev"
    shape = p32.launch()
    k_lane = shape["k_per_lane"]
    out = {
        "metric": METRIC,
        "value": value,
        "unit": "evals/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms32,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": w.name, "n_obj": w.n_obj, "n_t": int(w.n_obs) if single else
                   "U{%d..%d}" % (int(w.n_t.min()), int(w.n_t.max())), "n_obs": int(w.n_obs),
                   "n_f": w.n_f, "f_range_cycles_per_day": [w.f_min, w.f_max],
                   "form": "fp32 sums, fp64 phase reduction", "output": "pgram f32 + peak"
                   if single else "peaks", "launch": args.launch,
                   "method": "generalized (errors 1/dy^2, floating mean)" if gen else "standard"},
        "objects_per_s": w.n_obj / (ms32 * 1e-3),
        "pgram_bytes_per_step": (4 * w.n_f * w.n_obj) if single else 0,
        "pgram_write_GBps": (4 * w.n_f * w.n_obj / (ms32 * 1e-3) / 1e9) if single else 0.0,
        "fp64_reference": {"evals_per_s": evals / (ms64 * 1e-3), "ms_per_step": ms64,
                           "objects_per_s": w.n_obj / (ms64 * 1e-3)},
        "speedup_vs_fp64": ms64 / ms32,
        "peak_bin_agreement": float(agree.mean()),
        "generalized_vs_standard": std_cost,
        "max_abs_dpower_vs_fp64": d,
        "roofline": roofline(args, gen, rec_name, k_lane, evals, k_ms, w.name, variant),
        "cpu_baseline": None,
    }
    if not args.no_cpu:
        threads, aff = host_threads(args.cpu_threads)
        log(f"[bench] oracle baseline on {threads} threads (affinity {aff})")
        out["cpu_baseline"], (objs, bins, ora_vals) = cpu_baseline(w, args.cpu_evals, threads,
                                                                   args.method)
        out["cpu_baseline"]["cpu_model"] = cpu_model()
        out["cpu_baseline"]["affinity_cores"] = aff
        # the FP32 form's power at the same (object, bin) pairs, against the
        # oracle: the bench line states its error against the FP64 oracle
        if single:
            got = p32.pgram[0][torch.as_tensor(bins, device=dev)].double().cpu().numpy()
        else:
            k = int(objs.max()) + 1
            sub = lsp.Periodogram(t, y, w.f_min, w.f_max, w.n_f, offsets=off[:k + 1],
                                  form=lsp.FORM_FP32P, schedule=sched, recurrence=rec, k=args.k,
                                  waves=args.waves, method=kw.get("method", "standard"),
                                  dy=kw.get("dy"), pgram=True, peaks=False, **kv)
            sub()
            flat = torch.as_tensor(objs * w.n_f + bins, device=dev)
            got = sub.pgram.view(-1)[flat].double().cpu().numpy()
        out["oracle_check"] = {"pairs": int(len(bins)),
                               "max_abs_dpower_vs_oracle": float(np.max(np.abs(got - ora_vals))),
                               "form": "fp32 (the timed form)"}
    print(json.dumps(out), flush=True)


CUTOFFS = (0, 25, 50, 75, 100, 150, 200, 300, 400, 550)


def recovery_curve(p_rot_true_h, p_lc_days, n_t, tol_h=0.1):
    """Fraction of objects whose derived rotation period (twice the light-curve
    period at the peak) is within tol_h of the assigned one, overall and for
    every observation cutoff (objects with at least that many points)."""
    derived = 2.0 * 24.0 * np.asarray(p_lc_days, dtype=np.float64)
    ok = np.abs(derived - p_rot_true_h) <= tol_h
    curve = []
    for c in CUTOFFS:
        m = n_t >= c
        curve.append({"cutoff": c, "objects": int(m.sum()),
                      "matched": float(ok[m].mean()) if m.any() else None})
    return float(ok.mean()), curve, ok


def bench_recovery(args, torch, dev):
    """Section 4.2's accuracy study on an asteroid-like population: the peak
    of each object's periodogram on the paper's batch grid (rad/day,
    N_f = 200,000) gives the light-curve period; twice it should match the
    assigned rotation period within 0.1 h.  Timed as whole batches."""
    from paper_2105_04006_amd import lsp, synth

    w = synth.make_workload("asteroids_1k")
    n_t = np.diff(w.offsets)
    log(f"[bench] recovery: {w.name} n_obj={w.n_obj} n_obs={w.n_obs} n_f={w.n_f} "
        f"N_t median {int(np.median(n_t))}")
    off = torch.as_tensor(w.offsets, device=dev)
    t = torch.as_tensor(w.t, device=dev)
    y = torch.as_tensor(w.y, device=dev)
    dy = torch.as_tensor(w.dy, device=dev)
    runs = {}
    for name, form, method in (("standard_fp32", lsp.FORM_FP32P, "standard"),
                               ("standard_fp64", lsp.FORM_FP64, "standard"),
                               ("generalized_fp32", lsp.FORM_FP32P, "generalized"),
                               ("generalized_fp64", lsp.FORM_FP64, "generalized")):
        p = lsp.Periodogram(t, y, w.f_min, w.f_max, w.n_f, offsets=off, unit=lsp.ANGULAR,
                            form=form, method=method, dy=dy if method == "generalized" else None,
                            pgram=False, peaks=True)
        p()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        steps = 3 if form == lsp.FORM_FP32P else 1
        for _ in range(steps):
            p()
        torch.cuda.synchronize()
        ms = (time.perf_counter() - t0) / steps * 1e3
        pk = p.peaks()
        frac, curve, ok = recovery_curve(w.p_rot_hours, pk["period"], n_t)
        runs[name] = {"ms_per_batch": ms, "objects_per_s": w.n_obj / (ms * 1e-3),
                      "matched": frac, "curve": curve, "index": pk["index"]}
        log(f"[bench] {name}: {ms:.2f} ms, matched {frac:.4f}, "
            f"N_t>=50 {curve[2]['matched']:.4f}")
    agree = {
        "standard fp32 vs fp64": float(np.mean(np.abs(runs["standard_fp32"]["index"]
                                                      - runs["standard_fp64"]["index"]) <= 1)),
        "generalized fp32 vs fp64": float(np.mean(np.abs(runs["generalized_fp32"]["index"]
                                                         - runs["generalized_fp64"]["index"])
                                                  <= 1)),
    }
    for r in runs.values():
        del r["index"]
    in_grid = float(np.mean(w.p_rot_hours / 2.0 <= 2 * np.pi / w.f_min * 24.0))
    out = {
        "metric": "recovered rotation periods (within 0.1 h) on an asteroid-like population",
        "value": runs["standard_fp32"]["matched"],
        "unit": "fraction of objects",
        "n_gpus": 1,
        "steps": 3,
        "warmup": 1,
        "ms_per_step": runs["standard_fp32"]["ms_per_batch"],
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": w.name, "n_obj": w.n_obj, "n_obs": int(w.n_obs), "n_f": w.n_f,
                   "grid_rad_per_day": [w.f_min, w.f_max],
                   "n_t": "log-normal, median %d, [%d, %d]" % (int(np.median(n_t)),
                                                                int(n_t.min()), int(n_t.max())),
                   "output": "peaks"},
        "paper_context": "94.9% of ~1,000 synthetic asteroids within 0.1 h; 99% with >= 50 "
                         "observations; 100% for the 45 objects with >= 550 (Section 4.2)",
        "rotation_period_on_grid": in_grid,
        "runs": runs,
        "peak_agreement_within_one_bin": agree,
        "roofline": None,
        "cpu_baseline": None,
    }
    print(json.dumps(out), flush=True)


def bench_host_return(args, torch, dev):
    """Section 3.5: periodograms of a whole batch returned to host memory.

    standard: lsp_batch into a device periodogram, then one device-to-host
    copy into pageable memory (the driver stages it); pipelined: the
    pinned-staging pipeline, chunk by chunk with host copy threads.  Both are end-to-end (kernels + transfer), inputs resident on the
    device, destination pages touched beforehand."""
    from paper_2105_04006_amd import lsp, synth

    gen = args.method == "generalized"
    w = synth.make_workload(args.workload, errors=gen)
    nbytes = 4 * w.n_obj * w.n_f
    log(f"[bench] host return: {w.name} n_obj={w.n_obj} n_f={w.n_f}, {nbytes / 1e9:.2f} GB FP32")
    off = torch.as_tensor(w.offsets, device=dev)
    t = torch.as_tensor(w.t, device=dev)
    y = torch.as_tensor(w.y, device=dev)
    dy = torch.as_tensor(w.dy, device=dev) if gen else None
    method = "generalized" if gen else "standard"
    host_a = np.zeros((w.n_obj, w.n_f), dtype=np.float32)
    host_b = np.zeros((w.n_obj, w.n_f), dtype=np.float32)
    ta = torch.from_numpy(host_a)
    p = lsp.Periodogram(t, y, w.f_min, w.f_max, w.n_f, offsets=off, form=lsp.FORM_FP32P,
                        method=method, dy=dy, pgram=True, peaks=True)
    pipe = lsp.HostPipe()

    def standard():
        p()
        ta.copy_(p.pgram)  # synchronous device-to-pageable copy
        p.peaks()

    def pipelined():
        pipe.batch_to_host(off, t, y, w.f_min, w.f_max, w.n_f, dy=dy, method=method,
                           form=lsp.FORM_FP32P, out=host_b)

    def timed(fn, steps):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(steps):
            fn()
        torch.cuda.synchronize()
        return (time.perf_counter() - t0) / steps * 1e3

    steps = max(1, min(args.steps, 5))
    for _ in range(max(1, args.warmup if args.warmup < 3 else 1)):
        standard()
        pipelined()
    ms_std = timed(standard, steps)
    log(f"[bench] standard (kernels + one copy to pageable memory) {ms_std:.1f} ms")
    ms_pipe = timed(pipelined, steps)
    log(f"[bench] pipelined (pinned staging, copy threads) {ms_pipe:.1f} ms")
    p()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        p()
    torch.cuda.synchronize()
    ms_kern = (time.perf_counter() - t0) / steps * 1e3
    same = bool(np.array_equal(host_a, host_b))
    out = {
        "metric": METRIC + " (periodograms returned to host memory, PCIe-inclusive)",
        "value": w.evals / (ms_pipe * 1e-3),
        "unit": "evals/s",
        "n_gpus": 1,
        "steps": steps,
        "warmup": 1,
        "ms_per_step": ms_pipe,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": w.name, "n_obj": w.n_obj, "n_obs": int(w.n_obs), "n_f": w.n_f,
                   "output": "pgram f32 to host + peaks", "method": method},
        "host_return": {
            "pgram_bytes": nbytes,
            "standard_ms": ms_std,
            "pipelined_ms": ms_pipe,
            "device_only_ms": ms_kern,
            "speedup_pipelined_vs_standard": ms_std / ms_pipe,
            "standard_GBps": nbytes / (ms_std * 1e-3) / 1e9,
            "pipelined_GBps": nbytes / (ms_pipe * 1e-3) / 1e9,
            "identical_results": same,
            "pipe": "library defaults: 1 lane (kernel + copy stream, two chunk buffers), "
                    "16 MiB pinned staging (two halves), 128 MiB chunks, 12 copy threads",
        },
        "roofline": None,
        "cpu_baseline": None,
    }
    pipe.close()
    print(json.dumps(out), flush=True)


FORM_WORKLOADS = ("lsst_200k", "learned_100k", "asteroids_100k")
KIND_NAMES = {0: "sinusoid", 1: "two_harmonic", 2: "noise"}


def cpu_model():
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def host_threads(requested):
    """Threads of the oracle: every core of this process's affinity set, or
    the number requested."""
    aff = len(os.sched_getaffinity(0))
    return (int(requested) if requested > 0 else aff), aff


def oracle_subset(w, n_sub, target_evals, threads, extra_bins, method="standard"):
    """The oracle on a bounded sample of the first n_sub objects: every
    stride-th bin of each (start staggered per object) plus the bins in
    extra_bins (per-object peak indices of the GPU forms, -1 = none).
    Returns the sample, the oracle's values and the cpu_baseline record."""
    import oracle

    oracle.default()
    n_sub = min(n_sub, w.n_obj)
    n_t = np.diff(w.offsets)[:n_sub]
    stride = max(1, int(np.ceil(float(n_t.sum()) * w.n_f / target_evals)))
    objs, bins = [], []
    for o in range(n_sub):
        b = np.arange((o * 7919) % stride, w.n_f, stride, dtype=np.int64)
        ex = np.unique(np.concatenate([e[o:o + 1] for e in extra_bins]))
        ex = ex[(ex >= 0) & (ex < w.n_f)]
        b = np.union1d(b, ex)
        objs.append(np.full(len(b), o, dtype=np.int64))
        bins.append(b)
    objs, bins = np.concatenate(objs), np.concatenate(bins)
    t0 = time.perf_counter()
    if method == "generalized":
        vals = oracle.gen_eval_bins(w.offsets, w.t, w.y, w.dy, w.f_min, w.f_max, w.n_f, objs,
                                    bins, unit=w.unit, threads=threads)
    else:
        vals = oracle.eval_bins(w.offsets, w.t, w.y, w.f_min, w.f_max, w.n_f, objs, bins,
                                unit=w.unit, threads=threads)
    dt = time.perf_counter() - t0
    evals = int(np.diff(w.offsets)[objs].sum())
    rec = {"value": evals / dt, "unit": "evals/s", "cores": threads, "kind": "oracle",
           "sample": f"first {n_sub} objects of the same workload: every {stride}th bin "
                     f"(start staggered per object) plus the GPU forms' peak bins, "
                     f"{len(bins)} (object, bin) pairs, {evals:.3g} evals, {dt:.2f} s wall"}
    return objs, bins, vals, rec


def bin_values(w, tensors, form, index, method="standard", dy=None):
    """Each object's power at one chosen bin (index[o], -1 = none), through
    row mode with one-bin bands."""
    import torch
    from paper_2105_04006_amd import lsp

    off, t, y = tensors
    band = torch.as_tensor(np.where(index >= 0, index, -1).astype(np.int32), device=t.device)
    r = lsp.Rows(off, t, y, w.f_min, w.f_max, w.n_f, None, band, 1, 1, unit=w.unit, form=form,
                 method=method, dy=dy)
    r()
    return r.peaks()["power"]


def bench_forms(args, torch, dev):
    """The three forms on one batch workload (default lsst_200k: 2e5 objects,
    N_t U{20..500}, 60% sinusoids, 30% with a second harmonic, 10% pure
    noise, N_f = 250,000 over [0.5, 24) cycles/day), each returning every
    object's peak, inputs resident in HBM:
      fp32    the FP32 form with FP64 phase reduction on the whole grid (the
              timed headline: its evals/s is the line's value);
      learned features -> network -> top bands -> refine -> fallback (the
              network trained and the thresholds calibrated beforehand, on
              independent objects, outside the timed region);
      fp64    the plain FP64 form on the whole grid (the reference form).
    Peak agreement is judged against the FP64 form on every object; the FP64
    and FP32 forms are checked against the CPU oracle on a sample of the first
    2,000 objects, which also times the oracle (cpu_baseline)."""
    from paper_2105_04006_amd import learned, lsp, synth

    gen = args.method == "generalized"
    method = "generalized" if gen else "standard"
    forms = [f for f in args.forms.split(",") if f]
    name = args.workload

    def make(n_obj=None, seed=None):
        if name.startswith("asteroids"):
            return synth.make_workload(name, n_obj=n_obj, seed=seed)
        return synth.make_workload(name, n_obj=n_obj, seed=seed, errors=gen)

    w = make()
    n_t = np.diff(w.offsets)
    log(f"[bench] workload {w.name}: n_obj={w.n_obj} n_obs={w.n_obs} n_f={w.n_f} "
        f"evals={w.evals:.3e}")
    tt = learned._tensors(w, dev)
    off, t, y = tt
    dy = learned._errors(w, dev, method)
    rec = {"auto": lsp.REC_AUTO, "rotation": lsp.REC_ROTATION,
           "chebyshev": lsp.REC_CHEBYSHEV}[args.recurrence]
    sched = {"auto": lsp.SCHED_AUTO, "grid": lsp.SCHED_GRID,
             "persistent": lsp.SCHED_PERSISTENT}[args.schedule]

    def whole(form, **kw):
        return lsp.Periodogram(t, y, w.f_min, w.f_max, w.n_f, offsets=off, form=form,
                               pgram=False, unit=w.unit, method=method, dy=dy,
                               order=order_code(args.order), **kw)

    def wall(fn, steps):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(steps):
            fn()
        torch.cuda.synchronize()
        return (time.perf_counter() - t0) * 1e3 / steps

    # --- FP32 form, whole grid: the headline ------------------------------
    p32 = whole(lsp.FORM_FP32P, recurrence=rec, schedule=sched, k=args.k, waves=args.waves)
    shape = p32.launch()
    for _ in range(args.warmup):
        p32()
    torch.cuda.synchronize()
    log("[bench] fp32 warm-up done")
    # each timed step also records events around the main kernel on the
    # library's launch stream (the kernel's own device time)
    pairs = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
             for _ in range(args.steps)]
    for a, b in pairs:
        a.record()
        b.record()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for a, b in pairs:
        lsp.set_stage_events(a.cuda_event, b.cuda_event)
        p32()
    torch.cuda.synchronize()
    ms32 = (time.perf_counter() - t0) * 1e3 / args.steps
    lsp.set_stage_events(None, None)
    k_ms = float(np.mean([a.elapsed_time(b) for a, b in pairs]))
    log(f"[bench] fp32 whole grid {ms32:.2f} ms/step, main kernel {k_ms:.2f} ms")
    pk32 = p32.peaks()

    # --- learned form --------------------------------------------------------
    lrn = None
    if "learned" in forms:
        props = ("hybrid", "coarse", "network")
        prop = learned.fit_proposer(
            lambda n, s: make(n, s), dev, n_train=args.train_objects, n_val=args.val_objects,
            seed_train=synth.SEED_BASE + 1000, seed_val=synth.SEED_BASE + 1001,
            method=method, proposals=props, log=lambda m: log("[bench] " + m),
            # 99.93% on 20,000 validation objects keeps the evaluated batch at
            # >= 99.9% despite the sampling spread (about +-0.02%)
            target=0.9993)
        runs = {}
        for pr in props:
            lp = prop.periodogram(off, t, y, w.f_min, w.f_max, unit=w.unit, proposal=pr,
                                  method=method, dy=dy)
            steps = args.steps if pr == args.proposal else max(1, min(3, args.steps))
            for _ in range(max(1, min(args.warmup, 2))):
                lp()
            ms = wall(lp, steps)
            pk = lp.peaks()
            idx = lp.rows.cpu().numpy()  # the bands kept for refinement
            bb = np.where(idx >= 0, np.minimum(prop.geo.band_bins,
                                               w.n_f - idx * prop.geo.band_bins), 0).sum(axis=1)
            fb = lp.objects[:lp.n_fallback].cpu().numpy()
            evaluated = float(np.sum(n_t * bb) + np.sum(n_t[fb]) * w.n_f)
            runs[pr] = {"ms_per_step": ms, "steps": steps, "objects_per_s": w.n_obj / (ms * 1e-3),
                        "whole_grid_equiv_evals_per_s": w.evals / (ms * 1e-3),
                        "fallback_objects": int(lp.n_fallback),
                        "evaluated_fraction": evaluated / float(w.evals),
                        "thresholds": {"mass_min": prop.thresholds[pr][0],
                                       "power_min": prop.thresholds[pr][1],
                                       "alpha": prop.thresholds[pr][3],
                                       "tau": prop.thresholds[pr][4]},
                        "_peaks": pk, "_idx": idx}
            log(f"[bench] learned ({pr}) {ms:.2f} ms/step, {lp.n_fallback} fallbacks, "
                f"evaluated {evaluated / w.evals:.4f} of the grid")
            if pr == args.proposal:
                # stage breakdown of one step (events on the current stream)
                ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
                ev[0].record()
                lp.propose()
                ev[1].record()
                lp.refine()
                ev[2].record()
                learned.select_fallback(lp.peaks_raw, None if pr == "coarse" else lp.mass,
                                        lp.n_obj, lp.mass_min, lp.power_min, lp.objects,
                                        lp.count)
                nfb = int(lp.count.item())
                if nfb:
                    lp.full.set_rows(lp.objects[:nfb])
                    lp.full()
                ev[3].record()
                torch.cuda.synchronize()
                runs[pr]["stages_ms"] = {"features_network_topk": ev[0].elapsed_time(ev[1]),
                                         "refine": ev[1].elapsed_time(ev[2]),
                                         "select_and_fallback": ev[2].elapsed_time(ev[3])}
            del lp
        lrn = (prop, runs)

    # --- plain FP64 form, whole grid ---------------------------------------
    pk64 = None
    ms64 = None
    if "fp64" in forms:
        k_warm = int(np.searchsorted(w.offsets, min(w.n_obs, 20000)))
        k_warm = max(1, min(w.n_obj, k_warm))
        warm = lsp.Periodogram(t, y, w.f_min, w.f_max, w.n_f, offsets=off[:k_warm + 1],
                               form=lsp.FORM_FP64, pgram=False, unit=w.unit, method=method,
                               dy=dy)
        warm()
        p64 = whole(lsp.FORM_FP64)
        steps64 = args.fp64_steps if args.fp64_steps > 0 else 2
        ms64 = wall(p64, steps64)
        log(f"[bench] fp64 whole grid {ms64:.1f} ms/step ({steps64} steps)")
        pk64 = p64.peaks()
        del p64

    # --- agreement, on every object ------------------------------------------
    ref = pk64 if pk64 is not None else pk32
    ref_name = "fp64" if pk64 is not None else "fp32"
    ok = ref["status"] == 0
    kinds = w.kind if w.kind is not None else np.zeros(w.n_obj, np.int32)

    def agreement(pk):
        hit = np.abs(pk["index"] - ref["index"]) <= 1
        d = {"all": float(hit[ok].mean())}
        for kv, kn in KIND_NAMES.items():
            m = ok & (kinds == kv)
            if m.any():
                d[kn] = float(hit[m].mean())
        d["statuses_equal"] = bool(np.array_equal(pk["status"], ref["status"]))
        return d

    form_rec = {}
    f32 = {"ms_per_step": ms32, "steps": args.steps, "objects_per_s": w.n_obj / (ms32 * 1e-3),
           "evals_per_s": w.evals / (ms32 * 1e-3), "main_kernel_ms": k_ms,
           "launch": dict(shape["matrix"], kernels="matrix cores") if shape["matrix"] else
           dict({k: shape[k] for k in ("k_per_lane", "waves_per_wg", "schedule", "recurrence",
                                       "tile_freqs", "tiles_per_item", "n_items")},
                kernels="vector")}
    if pk64 is not None:
        f32["peak_bin_agreement_vs_fp64"] = agreement(pk32)
        # power error at both peak indices (FP32 form against the FP64 form)
        p32_at_64 = bin_values(w, tt, lsp.FORM_FP32P, np.where(ok, ref["index"], -1), method,
                               dy)
        p64_at_32 = bin_values(w, tt, lsp.FORM_FP64, np.where(ok, pk32["index"], -1), method,
                               dy)
        d1 = np.abs(p32_at_64[ok] - ref["power"][ok])
        d2 = np.abs(pk32["power"][ok] - p64_at_32[ok])
        f32["max_abs_dpower_vs_fp64_at_both_peaks"] = float(max(d1.max(), d2.max()))
    form_rec["fp32"] = f32
    if lrn is not None:
        prop, runs = lrn
        band = np.where(ok, ref["index"] // prop.geo.band_bins, -2)
        for pr, r in runs.items():
            pk, idx = r.pop("_peaks"), r.pop("_idx")
            r["peak_bin_agreement_vs_" + ref_name] = agreement(pk)
            r["peak_bin_agreement_vs_fp32"] = float(np.mean(
                np.abs(pk["index"][ok] - pk32["index"][ok]) <= 1))
            r["proposal_covers_peak_band"] = float(np.mean((idx == band[:, None]).any(axis=1)[ok]))
            r["mean_refined_bands"] = float(np.mean((idx >= 0).sum(axis=1)))
            if pk64 is not None:
                p64_at_l = bin_values(w, tt, lsp.FORM_FP64, np.where(ok, pk["index"], -1),
                                      method, dy)
                r["max_abs_dpower_vs_fp64_at_own_peak"] = float(np.max(
                    np.abs(pk["power"][ok] - p64_at_l[ok])))
        form_rec["learned"] = {"default_proposal": args.proposal, "proposals": runs,
                               "train_objects": prop.n_train, "val_objects": prop.n_val,
                               "train_seconds": prop.train_seconds,
                               "train_loss": [prop.history[0], prop.history[-1]],
                               "network": "1088-512-256-64 BF16 MFMA, FP32 accumulation"}
    if ms64 is not None:
        form_rec["fp64"] = {"ms_per_step": ms64, "steps": steps64,
                            "objects_per_s": w.n_obj / (ms64 * 1e-3),
                            "evals_per_s": w.evals / (ms64 * 1e-3)}
        form_rec["fp32"]["speedup_vs_fp64"] = ms64 / ms32
        if lrn is not None:
            for r in lrn[1].values():
                r["speedup_vs_fp64"] = ms64 / r["ms_per_step"]
                r["speedup_vs_fp32_whole_grid"] = ms32 / r["ms_per_step"]

    rec_name = "rotation" if shape["recurrence"] == lsp.REC_ROTATION else "chebyshev"
    k_lane = shape["k_per_lane"]
    out = {
        "metric": METRIC,
        "value": w.evals / (ms32 * 1e-3),
        "unit": "evals/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms32,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": w.name, "n_obj": w.n_obj,
                   "n_t": "U{%d..%d}" % (int(n_t.min()), int(n_t.max()))
                   if not name.startswith("asteroids") else "log-normal",
                   "n_obs": int(w.n_obs), "n_f": w.n_f, "f_range": [w.f_min, w.f_max],
                   "unit": "rad/day" if w.unit == 1 else "cycles/day",
                   "timed_form": "fp32 sums, fp64 phase reduction, whole grid",
                   "output": "peaks", "method": method},
        "objects_per_s": w.n_obj / (ms32 * 1e-3),
        "forms": form_rec,
        "roofline": roofline(args, gen, rec_name, k_lane, w.evals, k_ms, w.name),
        "cpu_baseline": None,
    }
    if not args.no_cpu:
        threads, aff = host_threads(args.cpu_threads)
        log(f"[bench] oracle on {threads} threads (affinity {aff})")
        extra = [ref["index"], pk32["index"]]
        objs, bins, ora, cb = oracle_subset(w, args.oracle_objects, args.cpu_evals, threads,
                                            extra, method)
        cb["cpu_model"] = cpu_model()
        cb["affinity_cores"] = aff
        out["cpu_baseline"] = cb
        k = int(objs.max()) + 1
        chk = {"objects": k, "pairs": int(len(bins))}
        flat = torch.as_tensor(objs * w.n_f + bins, device=dev)
        for fname, form in (("fp32", lsp.FORM_FP32P), ("fp64", lsp.FORM_FP64)):
            if fname == "fp64" and "fp64" not in forms:
                continue
            kw = dict(recurrence=rec, schedule=sched, k=args.k, waves=args.waves) \
                if form == lsp.FORM_FP32P else {}
            sub = lsp.Periodogram(t, y, w.f_min, w.f_max, w.n_f, offsets=off[:k + 1], form=form,
                                  pgram=True, peaks=True, unit=w.unit, method=method, dy=dy,
                                  pgram_dtype=lsp.PGRAM_F64 if form == lsp.FORM_FP64
                                  else lsp.PGRAM_F32, **kw)
            sub()
            got = sub.pgram.view(-1)[flat].double().cpu().numpy()
            spk = sub.peaks()
            full_pk = pk32 if form == lsp.FORM_FP32P else pk64
            same = bool(np.array_equal(spk[:k].tobytes(), full_pk[:k].tobytes()))
            d = np.abs(got - ora)
            rel = d / np.maximum(ora, 1e-3)
            k_w = int(np.nanargmax(rel))
            chk[fname] = {"max_abs_dpower": float(np.nanmax(d)),
                          "max_rel_dpower": float(rel[k_w]),
                          "worst_pair": {"object": int(objs[k_w]), "bin": int(bins[k_w]),
                                         "p_oracle": float(ora[k_w]), "p_gpu": float(got[k_w])},
                          "subset_peaks_equal_full_run": same}
            del sub
        out["oracle_check"] = chk
        log(f"[bench] oracle check {chk}")
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
