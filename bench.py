#!/usr/bin/env python3
"""Benchmark: solve time of Z w = 1 at n = 32768, m = 3 on one MI355X.

One step = one complete weighting solve (tile generation, FP32 MFMA Cholesky,
FP64 GMRES iterative refinement to ||1 - Z w||_inf <= 1e-12, magnitude) of a
seeded Gaussian cloud x ~ N(0, I_3), n = 32768, at the scale
t = 2^(7/8) m^(-2/3) n^(1/4) ~ 11.86 (the Gaussian cutoff law, Appendix C.2),
with the coordinates already resident in HBM.  Two FP64 dense comparators are
timed on the same GPU beside it: FP64 Z + rocSOLVER dpotrf/dpotrs, and FP64 Z +
this library's FP64 MFMA blocked Cholesky and FP64 substitution.  The CPU
oracle is timed on a bounded sample on the host cores.

Prints one JSON line (rank 0).
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

FP32_MFMA_PEAK_TFLOPS = 157.3
# the trailing update takes six BF16 products per FP32 product: dense BF16 peak / 6
SPLIT_MFMA_PEAK_TFLOPS = 2500.0 / 6.0
FP64_MFMA_PEAK_TFLOPS = 78.6
SYRK_SOURCES = [os.path.join(ROOT, "paper_2607_23354_amd", "csrc", f) for f in ("gemm_split.hip", "chol32.hip")]
SYRK_TRAFFIC = os.path.join(ROOT, "profiles", "k_syrk_split_gaussian_n32768_m3_traffic.txt")


def counter_traffic(n):
    """HBM bytes per launch of the trailing-update kernel, from the committed
    FETCH_SIZE + WRITE_SIZE counter summary, or None when there is none for
    this size or the kernel or its launch schedule changed after the counters
    were taken (hash of both sources)."""
    import hashlib
    try:
        kv = {}
        with open(SYRK_TRAFFIC) as f:
            for line in f:
                if ":" in line and not line.startswith((" ", "#", "|")):
                    k, v = line.split(":", 1)
                    kv[k.strip()] = v.strip()
        h = hashlib.sha256()
        for src in SYRK_SOURCES:
            with open(src, "rb") as f:
                h.update(f.read())
        sha = h.hexdigest()
        if kv.get("source_sha256") != sha or int(kv.get("n", -1)) != n:
            return None
        return float(kv["traffic_bytes_per_launch"])
    except (OSError, KeyError, ValueError):
        return None


GOLDEN = os.path.join(ROOT, "tests", "golden", "full_size")
METRIC_SCALES = ("tstar", "tstar_over4", "tstar_over2", "tstar_x2", "t_b")


def per_scale_errors(mag, Xd, ctx, w):
    """relerr_w = |w - w_oracle|_inf / |w_oracle|_inf and relerr_M against the
    oracle's weighting of the metric cloud at t*, t*/4, t*/2, 2 t*, t_b."""
    import numpy as np
    try:
        with open(os.path.join(GOLDEN, "index.json")) as f:
            index = json.load(f)
    except OSError:
        return None
    out = []
    for sc in METRIC_SCALES:
        rec = index.get(f"gauss_n32768_m3_seed0_{sc}")
        if rec is None:
            continue
        wg = np.load(os.path.join(GOLDEN, rec["w_file"]), allow_pickle=False)
        t0 = time.perf_counter()
        r = mag.weighting(Xd, rec["t"], ctx=ctx, out=w, solver="fp32_ir")
        wh = w.cpu().numpy()
        ms = (time.perf_counter() - t0) * 1e3
        out.append({"scale": sc, "t": rec["t"],
                    "relerr_w": float(np.abs(wh - wg).max() / np.abs(wg).max()),
                    "relerr_M": abs(r.info["magnitude"] - rec["M"]) / abs(rec["M"]),
                    "resid_inf_device": r.info["resid_inf"], "outer_iters": r.info["outer_iters"],
                    "gmres_iters": r.info["gmres_iters"], "min_w": r.info["min_w"],
                    "kappa_M_oracle": rec["kappa_M"], "cond_est_oracle": rec["cond_est"],
                    "ms_wall": ms})
        print(f"[bench] scale {sc}: t={rec['t']:.6g} relerr_w={out[-1]['relerr_w']:.2e} "
              f"relerr_M={out[-1]['relerr_M']:.2e}", file=sys.stderr, flush=True)
    return out


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--n", type=int, default=32768)
    ap.add_argument("--m", type=int, default=3)
    ap.add_argument("--seed", type=int, default=0)
    ap.add_argument("--dense-steps", type=int, default=2)
    ap.add_argument("--cpu-sample-n", type=int, default=16384)
    ap.add_argument("--no-scales", action="store_true",
                    help="skip the per-scale comparison with the oracle's expected weightings")
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--no-dense", action="store_true", help="skip both FP64 dense comparators")
    ap.add_argument("--no-rocsolver", action="store_true",
                    help="skip the rocSOLVER FP64 comparator (keep this library's FP64 MFMA one)")
    ap.add_argument("--check-rows", type=int, default=512)
    ap.add_argument("--eig-steps", type=int, default=1,
                    help="timed runs of the extreme-eigenvalue estimator on the same workload (0: skip)")
    ap.add_argument("--zero-steps", type=int, default=3,
                    help="timed solves of the scale-zero weighting of the same cloud (0: skip)")
    ap.add_argument("--copy-calib-mib", type=int, default=0,
                    help="run one plain device copy of this many MiB before the solves, so a "
                         "hardware-counter run can scale FETCH_SIZE / WRITE_SIZE by a kernel "
                         "of known traffic")
    args = ap.parse_args()

    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (got --gpus {args.gpus}); a solve of this size "
              "is one GPU's work and no multi-GPU path is built", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch

    import paper_2607_23354_amd as mag
    import workloads as W
    from paper_2607_23354_amd import _lib

    if not os.path.exists(_lib.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    assert torch.cuda.is_available(), "bench needs a GPU"
    dev = torch.device("cuda:0")
    n, m = args.n, args.m
    X = W.gaussian(n, m, seed=args.seed)
    t = W.gaussian_cutoff_estimate(n, m)
    Xd = torch.from_numpy(X).to(dev)
    w = torch.empty(n, dtype=torch.float64, device=dev)
    ctx = mag.Context(0)

    if args.copy_calib_mib > 0:
        nel = args.copy_calib_mib * (1 << 20) // 4
        src = torch.ones(nel, dtype=torch.float32, device=dev)
        dst = torch.empty_like(src)
        torch.cuda.synchronize()
        dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst

    def step(profile=True, solver="fp32_ir"):
        return mag.weighting(Xd, t, ctx=ctx, out=w, solver=solver, profile=profile)

    print(f"[bench] n={n} m={m} t={t:.6f} warmup={args.warmup} steps={args.steps}", file=sys.stderr, flush=True)
    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    infos = []
    t0 = time.perf_counter()
    for i in range(args.steps):
        infos.append(step().info)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    ms_per_step = (t1 - t0) * 1e3 / args.steps
    print(f"[bench] fp32_ir {ms_per_step:.2f} ms/solve", file=sys.stderr, flush=True)

    # roofline of the dominant kernel (trailing-update MFMA GEMM), from HIP events
    # recorded around every launch on the library's stream during the timed steps
    ms_upd = sum(i["ms_update"] for i in infos)
    fl_upd = sum(i["flop_update"] for i in infos)
    n_upd = sum(i["n_update"] for i in infos)
    achieved = fl_upd / (ms_upd * 1e-3) / 1e12 if ms_upd > 0 else None
    ms_factor = float(np.median([i["ms_factor"] for i in infos]))
    ms_tilegen = float(np.median([i["ms_tilegen"] for i in infos]))
    ms_refine = float(np.median([i["ms_refine"] for i in infos]))
    factor_flops = n ** 3 / 3.0
    last = infos[-1]

    # acceptance on the last result: oracle residual (Dot2) on sampled rows
    import oracle
    wh = w.cpu().numpy()
    rows = np.random.default_rng(123).choice(n, size=min(args.check_rows, n), replace=False)
    r_s = oracle.residual(X, t, wh, rows)
    resid_sampled = float(np.abs(r_s).max())

    dense = None
    if not args.no_dense and not args.no_rocsolver:
        try:
            step(profile=True, solver="fp64_dense")
            torch.cuda.synchronize()
            d0 = time.perf_counter()
            dinfo = None
            for _ in range(args.dense_steps):
                dinfo = step(profile=True, solver="fp64_dense").info
            torch.cuda.synchronize()
            d1 = time.perf_counter()
            dms = (d1 - d0) * 1e3 / args.dense_steps
            w_dense = w.cpu().numpy()
            dense = {
                "ms_per_solve": dms,
                "ms_potrf": dinfo["ms_factor"],
                # the comparator at the FP64 MFMA peak would still need n^3/3 flops there
                "ms_fp64_peak_floor": factor_flops / (FP64_MFMA_PEAK_TFLOPS * 1e12) * 1e3,
                "potrf_frac_fp64_peak": factor_flops / (dinfo["ms_factor"] * 1e-3) / 1e12 / FP64_MFMA_PEAK_TFLOPS,
                "resid_inf_device": dinfo["resid_inf"],
                "resid_inf_sampled_oracle": float(np.abs(oracle.residual(X, t, w_dense, rows)).max()),
                "magnitude": dinfo["magnitude"],
                "relerr_M_vs_fp32_ir": abs(dinfo["magnitude"] - last["magnitude"]) / abs(dinfo["magnitude"]),
            }
            print(f"[bench] fp64_dense {dms:.2f} ms/solve", file=sys.stderr, flush=True)
        except Exception as e:  # report, do not hide
            dense = {"error": repr(e)}

    # this library's FP64 MFMA blocked Cholesky + FP64 substitution on the same
    # cloud: the plain FP64 dense solve on the matrix cores
    chol64 = None
    if not args.no_dense:
        try:
            step(profile=True, solver="fp64_chol")
            torch.cuda.synchronize()
            c0 = time.perf_counter()
            cinfos = []
            for _ in range(args.dense_steps):
                cinfos.append(step(profile=True, solver="fp64_chol").info)
            torch.cuda.synchronize()
            c1 = time.perf_counter()
            cms = (c1 - c0) * 1e3 / args.dense_steps
            ci = cinfos[-1]
            upd_ms = sum(i["ms_update"] for i in cinfos)
            upd_fl = sum(i["flop_update"] for i in cinfos)
            syrk64 = upd_fl / (upd_ms * 1e-3) / 1e12 if upd_ms > 0 else None
            w64 = w.cpu().numpy()
            chol64 = {
                "ms_per_solve": cms,
                "ms_tilegen": ci["ms_tilegen"],
                "ms_factor": ci["ms_factor"],
                "ms_substitution": ci["ms_refine"],
                "factor_frac_fp64_peak": factor_flops / (ci["ms_factor"] * 1e-3) / 1e12 / FP64_MFMA_PEAK_TFLOPS,
                "syrk64_tflops": syrk64,
                "syrk64_frac_fp64_peak": (syrk64 / FP64_MFMA_PEAK_TFLOPS) if syrk64 else None,
                "syrk64_launches": sum(i["n_update"] for i in cinfos) // len(cinfos),
                "resid_inf_device": ci["resid_inf"],
                "resid_inf_sampled_oracle": float(np.abs(oracle.residual(X, t, w64, rows)).max()),
                "magnitude": ci["magnitude"],
                "relerr_M_vs_fp32_ir": abs(ci["magnitude"] - last["magnitude"]) / abs(ci["magnitude"]),
            }
            print(f"[bench] fp64_chol {cms:.2f} ms/solve", file=sys.stderr, flush=True)
        except Exception as e:  # report, do not hide
            chol64 = {"error": repr(e)}

    # error of w and of M = 1^T w against the oracle at every scale of the metric
    # cloud (expected values written by tests/golden/make_full_size.py from the
    # oracle alone; one untimed solve per scale)
    scales = None
    if not args.no_scales and n == 32768 and m == 3 and args.seed == 0:
        scales = per_scale_errors(mag, Xd, ctx, w)

    # the positive-definiteness check of the same workload (Lanczos on Z and Z^{-1});
    # reported beside the metric, never part of it
    eig = None
    if args.eig_steps > 0:
        mag.eig_extremes(Xd, t, ctx=ctx)
        torch.cuda.synchronize()
        e0 = time.perf_counter()
        einfo = None
        for _ in range(args.eig_steps):
            einfo = mag.eig_extremes(Xd, t, ctx=ctx)
        torch.cuda.synchronize()
        e1 = time.perf_counter()
        eig = dict(einfo)
        eig["ms"] = (e1 - e0) * 1e3 / args.eig_steps
        print(f"[bench] eig_extremes {eig['ms']:.2f} ms", file=sys.stderr, flush=True)

    # the weighting at scale zero of the same cloud (d w = 1 through c 1 1^T - d)
    zero = None
    if args.zero_steps > 0:
        wz = torch.empty(n, dtype=torch.float64, device=dev)
        mag.weighting_zero(Xd, ctx=ctx, out=wz)
        torch.cuda.synchronize()
        z0 = time.perf_counter()
        zr = None
        for _ in range(args.zero_steps):
            zr = mag.weighting_zero(Xd, ctx=ctx, out=wz)
        torch.cuda.synchronize()
        z1 = time.perf_counter()
        zrows = rows[:128]
        zres = oracle.dist_residual(X, wz.cpu().numpy() * zr.info["sum_dinv"], zrows)
        zero = {"ms_per_solve": (z1 - z0) * 1e3 / args.zero_steps,
                "outer_iters": zr.info["outer_iters"], "gmres_iters": zr.info["gmres_iters"],
                "c": zr.info["c"], "sum_dinv": zr.info["sum_dinv"], "min_w": zr.info["min_w"],
                "resid_rel_sampled_oracle": float(np.abs(zres).max()), "sampled_rows": int(len(zrows))}
        print(f"[bench] weighting_zero {zero['ms_per_solve']:.2f} ms/solve", file=sys.stderr, flush=True)

    cpu = None
    if not args.no_cpu:
        ns = args.cpu_sample_n
        Xs = W.gaussian(ns, m, seed=args.seed)
        ts = W.gaussian_cutoff_estimate(ns, m)
        c0 = time.perf_counter()
        oracle.weighting(Xs, ts)
        c1 = time.perf_counter()
        sec = c1 - c0
        cpu = {
            "value": (1.0 / sec) * (ns / n) ** 3,
            "unit": "solves/s",
            "cores": oracle.num_threads(),
            "kind": "oracle",
            "sample": (f"oracle FP64 solve (Z build, plain Cholesky, substitution, 3 Dot2 "
                       f"refinement steps) of a Gaussian cloud n={ns}, m={m} at its own t*, "
                       f"{sec:.2f} s, scaled by (n_sample/n)^3 to n={n}"),
        }

    out = {
        "metric": "Zw=1 solve time n=32768 m=3 (FP32+IR vs FP64 dense), rel residual ≤1e-12",
        "value": 1e3 / ms_per_step,
        "unit": "solves/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_per_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "fp32-factor+f64",
        "data": "synthetic",
        "config": {"workload": f"gaussian_n{n}_m{m}_tstar", "n": n, "m": m, "t": t,
                   "seed": args.seed, "solver": "fp32_ir", "parallelism": "single-gpu"},
        "roofline": {
            "bound": "mfma",
            "kernel": ("k_syrk_split (trailing update A22 -= L21 L21^T of two 512-column panels, K = 1024, FP32 operands "
                       "as three BF16 parts, six BF16 MFMA products each; achieved and peak count FP32 products)"),
            "achieved": achieved,
            "peak": SPLIT_MFMA_PEAK_TFLOPS,
            "unit": "TFLOP/s",
            "frac": (achieved / SPLIT_MFMA_PEAK_TFLOPS) if achieved else None,
            "traffic": counter_traffic(n),
            "launches": n_upd,
            "avg_launch_ms": ms_upd / n_upd if n_upd else None,
        },
        "phases_ms": {"tilegen": ms_tilegen, "factor": ms_factor, "refine": ms_refine},
        # against the FP32 matrix peak (above 1 where the split products outrun it)
        "factor_frac_fp32_peak": factor_flops / (ms_factor * 1e-3) / 1e12 / FP32_MFMA_PEAK_TFLOPS,
        "solve": {"outer_iters": last["outer_iters"], "gmres_iters": last["gmres_iters"],
                  "resid_inf_device": last["resid_inf"], "resid_inf_sampled_oracle": resid_sampled,
                  "sampled_rows": int(len(rows)), "magnitude": last["magnitude"],
                  "min_w": last["min_w"], "shifted": last["shifted"]},
        "fp64_dense": dense,
        "speedup_vs_fp64_dense": (dense["ms_per_solve"] / ms_per_step) if dense and "ms_per_solve" in dense else None,
        "fp64_mfma_chol": chol64,
        "speedup_vs_fp64_mfma_chol": (chol64["ms_per_solve"] / ms_per_step) if chol64 and "ms_per_solve" in chol64
        else None,
        "speedup_vs_fp64_peak_floor": (factor_flops / (FP64_MFMA_PEAK_TFLOPS * 1e12) * 1e3) / ms_per_step,
        "per_scale_vs_oracle": scales,
        "eig_extremes": eig,
        "weighting_zero": zero,
        "cpu_baseline": cpu,
        # the paper's own timing of this computation (section "Current scaling"): context on
        # other hardware with another solver, not the target
        "paper_context": {
            "value_s": 60.0,
            "what": "about one minute per cutoff-search iteration (one Zw=1 solve with HSS "
                    "compression and ULV factorisation, plus Lanczos), n about 30000 Gaussian points",
            "hardware": "16-core Apple M4 Max laptop CPU (Docker capped at 16 CPUs)",
            "method": "FP64 HSS + ULV (STRUMPACK), OpenBLAS",
        },
    }
    print(json.dumps(out))


if __name__ == "__main__":
    main()
