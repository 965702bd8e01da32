#!/usr/bin/env python
"""Benchmark: batched ALB generation on one MI355X.

One step = the whole hot path on one batch: a seeded cold start -> LOBPCG to a
residual of 1e-8 Ha on every element -> ALBs (restriction + orthonormalisation).
The headline workload is the uneven batch: 256 elements of the graphene-like slab
with extended grids of 32x32x64, 48x48x64 and 64x64x64 points and 20-80 states,
2 % vacancies, solved in FP64; every timed step must return DG_OK with every
residual <= 1e-8.  Beside it: the mixed-precision path (FP32 stage + FP64
refinement) on the same batch, a step with per-kernel HIP-event timing (the class
table and the roofline of the dominant kernel), a step with all elements in one
stream (kernel durations without overlap between element groups), and the oracle
timed on the host cores on one element of the batch.

Prints one JSON line.  Inputs are resident in HBM before the timed region.
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import sys
import time

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
HBM_PEAK_GBS = 8000.0          # MI355X HBM3E, GB/s
FP64_PEAK_TFLOPS = 78.6        # MI355X FP64 (vector and matrix)
BF16_PEAK_TFLOPS = 2500.0      # MI355X dense BF16 matrix
CLASSES = ("plane", "zcol", "nonlocal", "teter", "gram", "rotate", "rayleigh_ritz", "other")
# kernel symbol of each timing class's main kernel (rocprofv3 names; the Rayleigh-Ritz
# class is k_rr_chol .. k_rr_coef, its label the name of the one kernel they came from)
CLASS_KERNEL = {"plane": "k_plane", "zcol": "k_zcol", "nonlocal": "k_nl_", "teter": "k_plane",
                "gram": "k_gram", "rotate": "k_rotate", "rayleigh_ritz": "k_rr_lds", "other": "k_residual"}
METRIC = "ALB element-solves/s + Hψ GB/s, mixed vs FP64 on one GPU at 1e-8 Ha eigen error"

# HBM bytes per launch from `rocprofv3 --pmc FETCH_SIZE` and `--pmc WRITE_SIZE` runs of
# the instrumented step (profiles/*_hbm_traffic.md), scaled by what the counters read
# for a 1 GiB device copy of the same run.  Valid only for the kernel source and
# workload they were taken on: `traffic` is reported null once any of the sources that
# fix the kernels and the workload's shapes (the kernel file, the context plan with the
# guard rule, the input generators) differs.
PMC_TRAFFIC = {
    # profiles/c4_fp64_hbm_traffic.md: one-stream C4, Gram class (k_gram + k_gram_reduce) per call
    "gram": {"config": "c4/1",
             "source": ["paper_2003_00407_amd/csrc/k_dense.hip", "paper_2003_00407_amd/csrc/runtime.hip",
                        "workloads/__init__.py"],
             "sha256": "2f5df9f2ddb6bb9a94cf05cdf92f435d178ebc822ec53a24835dd3aa046287f7",
             "bytes_per_launch": 210379159044},
}


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=3)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--config", default="c4")
    ap.add_argument("--tol", type=float, default=1e-8)
    ap.add_argument("--mixed-steps", type=int, default=2, help="timed mixed-precision steps (after one warm-up)")
    ap.add_argument("--no-mixed", action="store_true")
    ap.add_argument("--no-instrumented", action="store_true", help="skip the per-kernel timing step")
    ap.add_argument("--no-isolated", action="store_true", help="skip the one-stream step")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--inner-steps", type=int, default=3,
                    help="timed inner-SCF re-solves (V_eff update + warm start); 0 skips the leg")
    ap.add_argument("--budget-s", type=float, default=520.0,
                    help="wall-clock budget: side legs that would end past it are skipped (and said so)")
    ap.add_argument("--method", default="lobpcg", choices=["lobpcg", "chfsi"])
    ap.add_argument("--cheb-degree", type=int, default=16)
    ap.add_argument("--graph-iters", type=int, default=0,
                    help="LOBPCG steps captured per HIP graph replay (0: launch per kernel)")
    ap.add_argument("--no-peak-probe", action="store_true",
                    help="skip the box-measured copy bandwidth and FP64 GEMM rate (context, not the peak used)")
    ap.add_argument("--copy-probe-mib", type=int, default=0,
                    help="copy a buffer of this size once before timing (reference for PMC byte counters)")
    return ap.parse_args()


def log(msg):
    print(f"[bench] {msg}", file=sys.stderr, flush=True)


def one_step(E, x0, kw, tol, tag):
    """One solve + ALBs; a step that does not reach tol everywhere is an error."""
    from paper_2003_00407_amd import dgalb as D
    eig, res, iters, st = E.solve(x0, **kw)
    E.make_alb()
    mr = float(res.max().item())
    if st != D.DG_OK or not (mr <= tol):
        raise SystemExit(f"bench.py: {tag} step ended with status {D.status_string(st)} and max residual "
                         f"{mr:.3e} (tolerance {tol:g})")
    return iters, mr


def run_timed(E, x0, kw, steps, warmup, tol, torch, tag):
    """Warm up, then time `steps` full solves + ALBs with per-kernel timing off."""
    for i in range(warmup):
        one_step(E, x0, kw, tol, tag)
        log(f"{tag}: warm-up step {i + 1}/{warmup} done")
    E.timing(enable=False, reset=True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    iters, mr, worst = None, 0.0, 0.0
    for i in range(steps):
        iters, mr = one_step(E, x0, kw, tol, tag)
        worst = max(worst, mr)
        log(f"{tag}: step {i + 1}/{steps} at {time.perf_counter() - t0:.1f} s")
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    return {"seconds": t1 - t0, "iters": iters, "max_resid": worst}


def run_instrumented(E, x0, kw, tol, torch, tag):
    """One step with HIP events around every launch group: per-class times and work."""
    E.timing(enable=True, reset=True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    iters, mr = one_step(E, x0, kw, tol, tag)
    torch.cuda.synchronize()
    sec = time.perf_counter() - t0
    ms, launches, work = E.timing(enable=False, reset=True)
    return {"seconds": sec, "iters": iters, "ms": ms, "launches": launches, "work": work[:8],
            "hpsi_alg_bytes": work[8], "max_resid": mr}


def kernel_table(r):
    """Per kernel class: total ms, launches, average launch, achieved algorithmic rate."""
    tab = {}
    for i, name in enumerate(CLASSES):
        if r["launches"][i]:
            row = {"ms_total": round(r["ms"][i], 3), "launches": int(r["launches"][i]),
                   "avg_us": round(1000.0 * r["ms"][i] / r["launches"][i], 2)}
            if r["work"][i] > 0 and r["ms"][i] > 0:
                rate = r["work"][i] / (r["ms"][i] / 1000.0)
                if i <= 3:
                    row["GBs"] = round(rate / 1e9, 1)
                else:
                    row["TFLOPs"] = round(rate / 1e12, 2)
            tab[name] = row
    return tab


def source_sha(paths):
    """sha256 of one file, or of the concatenated per-file digests of a list."""
    if isinstance(paths, str):
        with open(os.path.join(HERE, paths), "rb") as f:
            return hashlib.sha256(f.read()).hexdigest()
    h = hashlib.sha256()
    for p in paths:
        h.update(source_sha(p).encode())
    return h.hexdigest()


def roofline_for(r, config, with_traffic=True, mixed=False):
    """Roofline of the dominant kernel class (most GPU time) over a run's kernels."""
    i = int(np.argmax(r["ms"]))
    name = CLASSES[i]
    ms, n, w = r["ms"][i], max(1, r["launches"][i]), r["work"][i]
    avg_s = ms / 1000.0 / n
    if i <= 3:       # HBM-bound passes: algorithmic bytes per launch / duration
        achieved = (w / n) / avg_s / 1e9
        peak, unit, bound = HBM_PEAK_GBS, "GB/s", "hbm"
    elif i <= 5:     # subspace GEMMs on the matrix cores: algorithmic flops per launch / duration
        achieved = (w / n) / avg_s / 1e12
        peak, unit, bound = (BF16_PEAK_TFLOPS if mixed else FP64_PEAK_TFLOPS), "TFLOP/s", "mfma"
    else:            # small dense FP64, one workgroup per element: vector ALU
        achieved = (w / n) / avg_s / 1e12
        peak, unit, bound = FP64_PEAK_TFLOPS, "TFLOP/s", "alu"
    traffic = None
    t = PMC_TRAFFIC.get(name) if with_traffic else None
    if t and t["config"] == config and source_sha(t["source"]) == t["sha256"]:
        traffic = t["bytes_per_launch"]
    return {"kernel": name, "symbol": CLASS_KERNEL[name], "bound": bound, "achieved": round(achieved, 4),
            "peak": peak, "unit": unit, "frac": round(achieved / peak, 5), "traffic": traffic,
            "avg_launch_us": round(avg_s * 1e6, 2), "launches": int(n),
            "work_per_launch": w / n}


def hpsi_rates(r):
    """H*psi GB/s over the three H*psi classes: by the per-state count 2Ns + Ns/J +
    nnz(s+4)/J (algorithmic), and by the passes' own minimal bytes."""
    ms = r["ms"][0] + r["ms"][1] + r["ms"][2]
    if ms <= 0:
        return None, None
    alg = r["hpsi_alg_bytes"] / (ms / 1000.0) / 1e9
    passes = (r["work"][0] + r["work"][1] + r["work"][2]) / (ms / 1000.0) / 1e9
    return round(alg, 1), round(passes, 1)


def cpu_baseline(cfg, tol):
    """The oracle (plain NumPy/SciPy FP64) solving one element of the batch to tol."""
    import workloads as W
    from oracle import alb as oalb
    from oracle import lobpcg as olob
    from oracle.planewave import n_workers
    # the element of median cost N (J + g)^2 (a representative element of the batch)
    cost = [e.npts * (e.n_states + W.guard_count(e.n_states)) ** 2 for e in cfg.elements]
    k = int(np.argsort(cost)[len(cost) // 2])
    el = cfg.elements[k]
    J = el.n_states
    x0 = W.initial_block(el.npts, J + W.guard_count(J), cfg.x0_seed_base + k).T
    t0 = time.perf_counter()
    r = olob.lobpcg(el, x0, J, tol=tol)
    oalb.make_alb(el, r.X, J)
    dt = time.perf_counter() - t0
    return {"value": round(1.0 / dt, 5), "unit": "element-solves/s", "cores": n_workers(), "kind": "oracle",
            "sample": (f"element {k} of {cfg.n_elem} (median cost; grid {'x'.join(map(str, el.n))}, J = {J}): "
                       f"full oracle LOBPCG solve to {tol:g} ({r.iters} iterations, converged={r.converged}) "
                       f"+ ALB SVD in {dt:.1f} s")}


def peak_probe(torch):
    """What this machine delivers to a plain device copy (1 GiB, read + write) and to a
    library FP64 GEMM (torch.matmul, 8192^3, rocBLAS): context for the roofline,
    whose peaks stay the published ones."""
    n = 1 << 27
    a = torch.empty(n, dtype=torch.float64, device="cuda")
    b = torch.empty_like(a)
    b.copy_(a)
    torch.cuda.synchronize()
    reps = 10
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    ev[0].record()
    for _ in range(reps):
        b.copy_(a)
    ev[1].record()
    torch.cuda.synchronize()
    copy_gbs = 2.0 * 8 * n * reps / (ev[0].elapsed_time(ev[1]) / 1000.0) / 1e9
    del a, b
    m = 8192
    x = torch.randn(m, m, dtype=torch.float64, device="cuda")
    y = torch.randn(m, m, dtype=torch.float64, device="cuda")
    z = x @ y
    torch.cuda.synchronize()
    ev[0].record()
    for _ in range(3):
        z = x @ y
    ev[1].record()
    torch.cuda.synchronize()
    tf = 2.0 * m ** 3 * 3 / (ev[0].elapsed_time(ev[1]) / 1000.0) / 1e12
    del x, y, z
    # the library at this path's own GEMM shapes: S^T S and S C for the largest and a
    # middle element of the uneven batch (N, 3K = 262144, 264 and 147456, 165)
    lib = {}
    for N, K in ((262144, 88), (147456, 55)):
        S = torch.randn(3 * K, N, dtype=torch.float64, device="cuda")     # column-major N x 3K
        Cc = torch.randn(K, 3 * K, dtype=torch.float64, device="cuda")
        for tag, fn, fl in (("gram", lambda: S @ S.T, 2.0 * N * 9 * K * K), ("rotation", lambda: Cc @ S, 6.0 * N * K * K)):
            fn()
            torch.cuda.synchronize()
            ev[0].record()
            for _ in range(3):
                fn()
            ev[1].record()
            torch.cuda.synchronize()
            lib[f"{tag}_N{N}_3K{3 * K}_TFLOPs"] = round(fl * 3 / (ev[0].elapsed_time(ev[1]) / 1000.0) / 1e12, 2)
        del S, Cc
    torch.cuda.empty_cache()
    return {"copy_GBs": round(copy_gbs, 1), "dgemm_TFLOPs": round(tf, 2), "library_at_path_shapes": lib,
            "how": ("1 GiB device copy x10 (2 x bytes per copy); torch.matmul FP64 8192^3 x3 and at the "
                    "path's Gram (S^T S, dense count) and rotation (S C) shapes x3; HIP events")}


def smooth_field(el, seed, amp):
    """Smooth seeded potential change on Q_k: one cosine per axis with random phases."""
    rng = np.random.default_rng(seed)
    ph = rng.uniform(0, 2 * np.pi, 3)
    ax = [np.cos(2 * np.pi * np.arange(n) / n + p) for n, p in zip(el.n, ph)]
    return amp * (ax[2][:, None, None] * ax[1][None, :, None] * ax[0][None, None, :]).ravel()


def run_inner_scf(E, els, D, torch, kw, tol, steps):
    """Inner SCF as in the paper's flowchart: V_eff changes by a decaying correction
    (0.05 Ha, then x0.3 per step), and each step re-solves warm-started from the last
    vectors and regenerates the ALBs.  The potentials are uploaded before the timed
    region; the original V_eff is restored afterwards."""
    base = np.concatenate([el.v_eff for el in els])
    delta = np.concatenate([smooth_field(el, 900 + k, 0.05) for k, el in enumerate(els)])
    vs = [torch.tensor(base + (0.3 ** s) * delta, dtype=torch.float64, device="cuda") for s in range(steps)]
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    its = []
    for s in range(steps):
        E.set_potential(vs[s])
        eig, res, it, st = E.solve(None, warm_start=True, **kw)
        E.make_alb()
        mr = float(res.max().item())
        if st != D.DG_OK or not (mr <= tol):
            raise SystemExit(f"bench.py: inner-SCF step {s} ended with status {D.status_string(st)} and max "
                             f"residual {mr:.3e}")
        its.append(float(np.mean(it)))
        log(f"inner SCF: step {s + 1}/{steps}, mean iterations {its[-1]:.1f}")
    torch.cuda.synchronize()
    sec = time.perf_counter() - t0
    E.set_potential(torch.tensor(base, dtype=torch.float64, device="cuda"))
    torch.cuda.synchronize()
    return sec, its


def make_x0(cfg, E, D, torch):
    if cfg.name == "c4":
        # 2.3e9 starting values: drawn on the device from a seeded generator
        gen = torch.Generator(device="cuda").manual_seed(cfg.x0_seed_base)
        return torch.randn(int(E.offsets(D.DG_OFF_X0)[-1]), dtype=torch.float64, device="cuda", generator=gen)
    return torch.tensor(D.pack_initial(cfg.elements, cfg.x0_seed_base), dtype=torch.float64, device="cuda")


def main():
    args = parse()
    if args.gpus != 1:
        print(f"bench.py: the benchmark runs on one GPU only (--gpus {args.gpus} requested); "
              "the element batch would shard across GPUs by whole elements with no communication, "
              "which is not measured here.", file=sys.stderr)
        sys.exit(2)
    t_start = time.perf_counter()
    import torch
    import workloads as W
    from paper_2003_00407_amd import dgalb as D
    if not torch.cuda.is_available():
        print("bench.py needs a GPU", file=sys.stderr)
        sys.exit(1)
    cfg = W.make_config(args.config)
    els = cfg.elements
    E = D.Elements(els)
    x0 = make_x0(cfg, E, D, torch)
    if args.copy_probe_mib > 0:
        buf = torch.empty(args.copy_probe_mib << 20, dtype=torch.uint8, device="cuda")
        buf2 = torch.empty_like(buf)
        buf2.copy_(buf)
        del buf, buf2
    torch.cuda.synchronize()
    n = len(els)
    grids = sorted({e.n for e in els})
    js = [e.n_states for e in els]
    log(f"config={cfg.name} elements={n} grids={grids} J={min(js)}..{max(js)} "
        f"(setup {time.perf_counter() - t_start:.1f} s)")
    meth = D.DG_LOBPCG if args.method == "lobpcg" else D.DG_CHFSI
    kw64 = dict(precision=D.DG_FP64, tol=args.tol, graph_iters=args.graph_iters, method=meth,
                cheb_degree=args.cheb_degree)
    r64 = run_timed(E, x0, kw64, args.steps, args.warmup, args.tol, torch, "fp64")
    step_s = r64["seconds"] / args.steps
    log(f"fp64: {r64['seconds']:.3f} s for {args.steps} steps")
    groups = int(os.environ.get("DG_STREAMS", "0")) or max(1, min(4, n // 4))
    out = {
        "metric": METRIC,
        "value": round(n * args.steps / r64["seconds"], 4),
        "unit": "element-solves/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(1000.0 * step_s, 3),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64",
        "data": "synthetic",
        "config": {"workload": cfg.name + ": " + cfg.description, "n_elem": n,
                   "grids": [list(g) for g in grids], "states": [min(js), max(js)], "tol": args.tol,
                   "method": args.method, "precision": "fp64", "graph_iters": args.graph_iters,
                   "element_groups": groups},
        "iters_fp64": {"min": int(np.min(r64["iters"])), "max": int(np.max(r64["iters"])),
                       "mean": round(float(np.mean(r64["iters"])), 2)},
        "max_resid_fp64": r64["max_resid"],
        "timing_note": "value: per-kernel event timing off; kernel tables from separate instrumented steps",
    }
    skipped = []

    # the one-stream step (the headline roofline) and the oracle timing run last and
    # must fit: every earlier side leg leaves time for them
    reserve = (0.0 if args.no_isolated else 2.5 * step_s + 15.0) + (0.0 if args.no_cpu_baseline else 60.0)

    def have_time(est_s, keep=reserve):
        return time.perf_counter() - t_start + est_s + keep <= args.budget_s

    if not args.no_mixed:
        kwmx = dict(kw64, precision=D.DG_MIXED)
        if have_time((args.mixed_steps + 1) * step_s * 1.1):
            rmx = run_timed(E, x0, kwmx, args.mixed_steps, 1, args.tol, torch, "mixed")
            log(f"mixed: {rmx['seconds']:.3f} s for {args.mixed_steps} steps")
            mx_step = rmx["seconds"] / args.mixed_steps
            out["mixed"] = {"value": round(n / mx_step, 4), "steps": args.mixed_steps, "warmup": 1,
                            "ms_per_step": round(1000.0 * mx_step, 3),
                            "speedup_vs_fp64": round(step_s / mx_step, 3),
                            "iters": {"min": int(np.min(rmx["iters"])), "max": int(np.max(rmx["iters"])),
                                      "mean": round(float(np.mean(rmx["iters"])), 2)},
                            "max_resid": rmx["max_resid"]}
        else:
            skipped.append("mixed")
    if args.inner_steps > 0:
        if have_time(args.inner_steps * step_s + 10.0):
            sec, its = run_inner_scf(E, els, D, torch, kw64, args.tol, args.inner_steps)
            out["inner_scf_fp64"] = {"value": round(n * args.inner_steps / sec, 4), "unit": "element-solves/s",
                                     "steps": args.inner_steps, "ms_per_step": round(1000.0 * sec / args.inner_steps, 3),
                                     "iters_mean_per_step": [round(x, 2) for x in its],
                                     "cold_iters_mean": out["iters_fp64"]["mean"],
                                     "dv": "smooth seeded correction, 0.05 Ha x 0.3^step"}
        else:
            skipped.append("inner_scf")

    if not args.no_instrumented and have_time(step_s * 1.3):
        ri = run_instrumented(E, x0, kw64, args.tol, torch, "fp64 instrumented")
        log(f"fp64 instrumented step: {ri['seconds']:.3f} s")
        alg, passes = hpsi_rates(ri)
        out["hpsi_GBs_fp64"] = alg
        out["hpsi_pass_GBs_fp64"] = passes
        # with element groups on their own streams, kernels of different groups overlap
        # and every event-timed duration includes the others' share of the GPU: this
        # table shows where the time goes, the roofline is taken from the one-stream step
        out["kernels_fp64"] = kernel_table(ri)
        out["kernels_fp64_note"] = "element groups on 4 streams: durations include overlap with other groups"
        out["roofline"] = roofline_for(ri, cfg.name, with_traffic=False)
        out["roofline"]["measured"] = "instrumented FP64 step, element groups sharing the GPU (overlapped)"
        if "mixed" in out and have_time(step_s * 1.2):
            rim = run_instrumented(E, x0, dict(kw64, precision=D.DG_MIXED), args.tol, torch, "mixed instrumented")
            alg, passes = hpsi_rates(rim)
            out["mixed"]["hpsi_GBs"] = alg
            out["mixed"]["kernels"] = kernel_table(rim)
    elif not args.no_instrumented:
        skipped.append("instrumented")
    if not args.no_isolated:
        if have_time(step_s * 2.5, keep=0.0 if args.no_cpu_baseline else 60.0):
            # all elements in one stream: kernel durations without overlap between groups
            del E
            torch.cuda.empty_cache()
            E1 = D.Elements(els, n_streams=1)
            one_step(E1, x0, kw64, args.tol, "one-stream warm-up")
            r1 = run_instrumented(E1, x0, kw64, args.tol, torch, "one-stream")
            log(f"one stream: {r1['seconds']:.3f} s")
            alg, passes = hpsi_rates(r1)
            out["one_stream_fp64"] = {"value": round(n / r1["seconds"], 4), "hpsi_GBs": alg,
                                      "hpsi_pass_GBs": passes, "kernels": kernel_table(r1)}
            # the headline roofline: kernels one at a time, durations not shared
            out["roofline"] = roofline_for(r1, cfg.name + "/1")
            out["roofline"]["measured"] = ("instrumented FP64 step, all elements in one stream (HIP events "
                                           "on that stream around each launch group)")
            del E1
        else:
            skipped.append("one_stream")
    if not args.no_peak_probe:
        out["box_measured"] = peak_probe(torch)
        log(f"peak probe: {out['box_measured']}")
    if not args.no_cpu_baseline:
        log("timing the oracle on the host")
        out["cpu_baseline"] = cpu_baseline(cfg, args.tol)
    if skipped:
        out["skipped_for_time"] = skipped
    log(f"total {time.perf_counter() - t_start:.1f} s")
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
