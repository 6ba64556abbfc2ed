"""Benchmark: time-to-solution of the shell multigrid solve on one MI355X.

One step = one whole solve of H u = b from u = 0 to relative residual 1e-8
(FP32 V-cycles inside the FP64 refinement loop; the workload's cycle, V(2,4)
on the 1024x768x70 shell) on the 1024x768x70 shell (55M unknowns), with b
and alpha already resident in HBM. The plain FP64 multigrid solve of the same
system is timed beside it, and the finest level's post-smoothing sweeps of
every V-cycle in the timed region are bracketed by HIP events on the solver's
stream to give the dominant kernel's achieved bandwidth against the HBM
roofline.

    python bench.py [--steps K] [--warmup W] [--gpus 1] [--workload NAME]
                    [--no-cpu-baseline] [--no-fp64] [--no-accuracy]

After the timed solves, the oracle solves the same system on the host from
u = 0 to the same tolerance (timed: cpu_baseline) and on to relres 1e-12;
that solution is the reference for the forward errors of the GPU solves, and
a sweep of tighter tolerances gives the time to a forward error of 1e-8.
On workloads too large for the oracle (over 1e8 cells) the reference is the
FP64 GPU solve to relres 1e-13, its residual recomputed on the host by the
oracle's operator.

Prints one JSON line on stdout; progress goes to stderr.
"""
from __future__ import annotations

import argparse
import json
import os
import statistics
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "time-to-1e-8 solve (s) + HBM GB/s, FP32+refine vs FP64 MG, 1024x768x70"
HBM_PEAK_GBPS = 8000.0


def log(msg):
    print(f"[bench] {msg}", file=sys.stderr, flush=True)


def kernel_roofline(stats_list, cls):
    """Achieved algorithmic GB/s of one kernel class over the timed solves."""
    ms = sum(s.kernels[cls]["fine_ms"] for s in stats_list)
    nb = sum(s.kernels[cls]["fine_bytes"] for s in stats_list)
    launches = sum(s.kernels[cls]["fine_launches"] for s in stats_list)
    if launches == 0 or ms <= 0:
        return None
    avg_ms = ms / launches
    bytes_per_launch = nb / launches
    gbps = bytes_per_launch / (avg_ms * 1e-3) / 1e9
    return {"kernel": cls, "launches": launches, "avg_ms": avg_ms,
            "bytes_per_launch": bytes_per_launch, "GBps": gbps}


def file_sha256(paths):
    import hashlib
    h = hashlib.sha256()
    for p in paths:
        with open(os.path.join(ROOT, p), "rb") as f:
            h.update(p.encode() + b"\0" + f.read())
    return h.hexdigest()


def split_note(cls, bytes_per_launch, n):
    """The library reports a launch that does two sweeps from zero (12 bytes per
    cell) as a third of its time and bytes for the first sweep and two for the
    second; nothing times the first sweep by itself."""
    if cls == "smooth0" and bytes_per_launch < 6 * n:
        return "a third of the launches of two sweeps from zero, not timed apart"
    return None


def measured_traffic(workload, cls):
    """HBM bytes per launch of the dominant kernel from the committed counter
    summary (rocprofv3 FETCH_SIZE / WRITE_SIZE, scaled by a plain copy), or
    None when no summary covers this workload and kernel class or when the
    kernel's sources have changed since the counters were taken."""
    path = os.path.join(ROOT, "profiles", f"traffic_{cls}_{workload}.json")
    if not os.path.exists(path):
        return None, "no counter summary for this kernel and workload"
    with open(path) as f:
        rec = json.load(f)
    try:
        now = file_sha256(rec["sources"])
    except OSError as e:
        return None, f"source missing: {e}"
    if now != rec["sources_sha256"]:
        return None, "kernel sources changed since the counters were taken"
    return rec["bytes_per_launch"], rec["kernel"]


def _oracle_setup(shell, smooth, threshold):
    import shellgen
    import oracle
    a, b = shellgen.alpha(shell), shellgen.rhs(shell)
    L = oracle.build_hierarchy(shell, a, threshold=threshold)
    opt = oracle.Options(nu_pre=shell.nu_pre, nu_post=shell.nu_post)
    opt.smooth_lo, opt.smooth_hi = smooth if smooth else (0.0, 0.0)
    return L, b, opt


def oracle_reference(shell, smooth, threshold, tol, tol_ref=1e-12, extra_iters=4):
    """The oracle, untuned, on the host: its whole solve of the workload
    from u = 0 to the bench tolerance, timed (wall clock, and the process's
    CPU time, whose ratio is the number of cores it kept busy), then
    continued from that iterate to relres tol_ref: the reference solution
    the GPU solves' forward errors are measured against."""
    import numpy as np
    import oracle
    t0 = time.perf_counter()
    L, b, opt = _oracle_setup(shell, smooth, threshold)
    t_setup = time.perf_counter() - t0
    w0, c0 = time.perf_counter(), time.process_time()
    u, st = oracle.solve(L, b, opt, tol=tol)
    wall, cpu = time.perf_counter() - w0, time.process_time() - c0
    cores = max(1, round(cpu / wall)) if wall > 0 else 1
    log(f"cpu oracle: setup {t_setup:.1f}s, solve to {tol:g} in {wall:.1f}s "
        f"({st['iters']} iterations, relres {st['relres']:.2e}, cpu/wall {cpu / wall:.2f})")
    t1 = time.perf_counter()
    uref, st2 = oracle.solve(L, b, opt, tol=tol_ref, u0=u)
    # a few more cycles: the residual stalls near FP64 rounding from here
    # on, the iterate still converges, and the reference must be well ahead
    # of the GPU solves it is compared with (which run the same cycle)
    uref, st3 = oracle.solve(L, b, opt, u0=uref, fixed_iters=extra_iters)
    log(f"cpu oracle: continued to relres {st2['relres']:.2e} "
        f"(+{st2['iters']} iterations), then {extra_iters} more (relres {st3['relres']:.2e}), "
        f"{time.perf_counter() - t1:.1f}s")
    base = {"value": wall, "unit": "s", "cores": cores,
            "host_cores": len(os.sched_getaffinity(0)), "kind": "oracle",
            "sample": (f"the whole solve of {shell.name} by the numpy FP64 oracle from u = 0 to "
                       f"relres {tol:g} (V({shell.nu_pre},{shell.nu_post}), {st['iters']} "
                       f"iterations, relres {st['relres']:.2e}); setup {t_setup:.1f} s not "
                       f"included; cores = its CPU time over wall time"),
            "iters": st["iters"], "relres": st["relres"], "setup_s": t_setup}
    ref = {"kind": "oracle", "relres": st3["relres"],
           "iters": st["iters"] + st2["iters"] + st3["iters"]}
    return uref, base, ref


def gpu_reference(S64, shell, b, threshold, tol_ref=1e-13):
    """Where the oracle's solve does not fit a bench run: the FP64 GPU solve
    to relres tol_ref, with its residual recomputed on the host by the
    oracle's operator (an independent FP64 check that it solves H u = b)."""
    import numpy as np
    import torch
    import shellgen
    import oracle
    u = torch.zeros_like(b)
    _, st = S64.solve(b, tol=tol_ref, out=u)
    torch.cuda.synchronize()
    L = oracle.build_hierarchy(shell, shellgen.alpha(shell), levels=1, threshold=threshold)
    uh, bh = u.cpu().numpy(), b.cpu().numpy()
    rel = float(np.linalg.norm(bh - oracle.apply(L[0], uh)) / np.linalg.norm(bh))
    log(f"reference: FP64 GPU solve to {tol_ref:g} ({st.iters} iterations); "
        f"oracle residual {rel:.2e}")
    return u, {"kind": "FP64 GPU solve, residual checked by the oracle", "tol": tol_ref,
               "iters": st.iters, "relres_oracle": rel}


def fwd_err(u, uref):
    return float((u - uref).norm() / uref.norm())


def oracle_solve(shell, tol, smooth, threshold, u_gpu):
    """Small workloads (up to a million cells): the oracle's whole solve on
    the host, beside the GPU's. Reports its iterations, contraction factors,
    relative residual and time, the time of a sparse direct solve (scipy
    splu of the assembled operator), and the GPU solution's relative
    difference from the oracle's."""
    import numpy as np
    import scipy.sparse.linalg as spla
    import shellgen
    import oracle
    L, b, opt = _oracle_setup(shell, smooth, threshold)
    t0 = time.perf_counter()
    u, st = oracle.solve(L, b, opt, tol=tol)
    t_solve = time.perf_counter() - t0
    t0 = time.perf_counter()
    lu = spla.splu(oracle.assemble(L[0]).tocsc())
    ud = lu.solve(b.ravel())
    t_splu = time.perf_counter() - t0
    rho = oracle.convergence_factors(st["res_hist"])
    diff = float(np.linalg.norm(u_gpu - u) / np.linalg.norm(u))
    log(f"oracle solve: {st['iters']} iterations, relres {st['relres']:.2e}, {t_solve:.2f}s; "
        f"splu {t_splu:.2f}s; GPU vs oracle {diff:.2e}")
    return {"iters": st["iters"], "relres": st["relres"], "seconds": t_solve, "cores": 1,
            "factors": [float(x) for x in rho], "splu_seconds": t_splu,
            "splu_vs_oracle": float(np.linalg.norm(ud - u.ravel()) / np.linalg.norm(ud)),
            "gpu_vs_oracle": diff}


def adjoint_run(S, sh, tol, steps=5):
    """The adjoint solve lambda = H^-T w (w ~ N(0,1), seeded) with the
    transposed V-cycle in the same refinement loop, from lambda = 0: median
    time over `steps` solves after one untimed one."""
    import torch
    import shellgen
    w = torch.from_numpy(shellgen.weights(sh)).to("cuda:0")
    S.solve_adjoint(w, tol=tol)
    torch.cuda.synchronize()
    ts = []
    for _ in range(steps):
        t1 = time.perf_counter()
        _, st = S.solve_adjoint(w, tol=tol)
        torch.cuda.synchronize()
        ts.append(time.perf_counter() - t1)
    ms = statistics.median(ts) * 1e3
    log(f"adjoint: {steps} solves, median {ms:.2f} ms, iters {st.iters}, relres {st.relres:.2e}")
    return {"ms": ms, "iters": st.iters, "relres": st.relres,
            "ms_per_iteration": ms / max(st.iters, 1),
            "what": "mg_solve_adjoint of w ~ N(0,1) to the same tolerance: transposed "
                    "V-cycles inside the FP64 refinement loop, from lambda = 0"}


def timestep_run(S, sh, alpha0, b0, steps, tol):
    """Steps 1..steps of shellgen.timestep: per step, the coefficient update
    (masses, pivots, coarsest matrix) and the solve warm-started from the
    previous step's solution, each timed with a device synchronisation. The
    inputs are resident in HBM before the first step."""
    import torch
    import shellgen
    seq = [tuple(torch.from_numpy(x).to(b0.device) for x in shellgen.timestep(sh, t))
           for t in range(1, steps + 1)]
    S.update_alpha(alpha0)
    u = torch.zeros_like(b0)
    _, st0 = S.solve(b0, tol=tol, out=u)
    torch.cuda.synchronize()
    upd, sol, iters = [], [], []
    for a_t, b_t in seq:
        t0 = time.perf_counter()
        S.update_alpha(a_t)
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        _, st = S.solve(b_t, tol=tol, u0=u, out=u)
        torch.cuda.synchronize()
        t2 = time.perf_counter()
        upd.append(t1 - t0)
        sol.append(t2 - t1)
        iters.append(st.iters)
    ucold = torch.zeros_like(b0)
    _, stc = S.solve(seq[-1][1], tol=tol, out=ucold)
    S.update_alpha(alpha0)
    log(f"timesteps: {steps} steps, update {statistics.mean(upd)*1e3:.2f} ms, warm solve "
        f"{statistics.mean(sol)*1e3:.2f} ms, iters {iters} (cold {stc.iters})")
    return {"steps": steps, "drift": 0.02, "tol": tol,
            "ms_per_step": (sum(upd) + sum(sol)) / steps * 1e3,
            "update_ms": statistics.mean(upd) * 1e3, "solve_ms": statistics.mean(sol) * 1e3,
            "iters": iters, "first_step_cold_iters": st0.iters,
            "last_step_cold_iters": stc.iters}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--workload", default="shell1024x768x70")
    ap.add_argument("--tol", type=float, default=1e-8)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-fp64", action="store_true")
    ap.add_argument("--copy-probe", action="store_true",
                    help="first run a plain 1 GiB device copy (counter calibration)")
    ap.add_argument("--smooth-interval", default=None, metavar="LO,HI",
                    help="per-sweep damping factors from the Chebyshev nodes of [LO, HI] "
                         "(default: the workload's interval, 1/3,2 unless it names "
                         "another); 'none': every sweep uses omega 0.8")
    ap.add_argument("--levels", type=int, default=0,
                    help="hierarchy depth: 0 = automatic (default), n = at most n levels "
                         "(the paper's shallow hierarchy is 4)")
    ap.add_argument("--precision", choices=["mixed", "fp64", "fp32"], default="mixed",
                    help="the timed solve: FP32 V-cycle inside FP64 refinement (default), "
                         "or everything in FP32 (its residual stalls near 1e-4 relative: "
                         "use --tol above that)")
    ap.add_argument("--semi-threshold", type=float, default=2.0,
                    help="latitude rows merge only where both rows' anisotropy is at most "
                         "this (default 2, the library default)")
    ap.add_argument("--no-accuracy", action="store_true",
                    help="skip the forward errors against a reference solution and the "
                         "tolerance sweep")
    ap.add_argument("--no-adjoint", action="store_true",
                    help="skip the timing of the adjoint solve (outside the timed region)")
    ap.add_argument("--timesteps", type=int, default=0, metavar="K",
                    help="also time K steps of a slowly varying sequence (alpha and b drift "
                         "by 2 %% per step): coefficient update plus a solve warm-started "
                         "from the previous step's solution")
    args = ap.parse_args()
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py measures one GPU only: the solver runs on a single MI355X "
              "(no multi-GPU path is built); run with --gpus 1", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch
    import shellgen
    from paper_2307_04528_amd import Solver

    sh = shellgen.workload(args.workload)
    if args.smooth_interval is None:
        smooth = tuple(sh.smooth)
    elif args.smooth_interval == "none":
        smooth = None
    else:
        smooth = tuple(float(v) for v in args.smooth_interval.split(","))
    dev = torch.device("cuda:0")
    log(f"workload {sh.name}: {sh.nlon}x{sh.nlat}x{sh.nlev} = {sh.n} unknowns")
    alpha = torch.from_numpy(shellgen.alpha(sh)).to(dev)
    b = torch.from_numpy(shellgen.rhs(sh)).to(dev)
    torch.cuda.synchronize()
    if args.copy_probe:
        # a plain device copy of known size (1 GiB read + 1 GiB written), the
        # reference that scales hardware byte counters to bytes
        src = torch.empty(1 << 27, dtype=torch.float64, device=dev).fill_(1.0)
        dst = torch.empty_like(src)
        for _ in range(3):
            dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst
        log("copy probe: 3 copies of 1 GiB")

    t0 = time.perf_counter()
    # The timed solves carry one pair of HIP events per V-cycle, around the
    # finest level's post-smoothing sweeps (the dominant kernel, nu_post
    # launches in a row; profile mode 3): every event pair between two
    # kernels idles the GPU for a few microseconds. One more, untimed, solve
    # with every finest-level launch timed gives the per-kernel breakdown.
    S = Solver.from_shell(sh, alpha, nu_pre=sh.nu_pre, nu_post=sh.nu_post,
                          precision=args.precision, profile=3, smooth_interval=smooth,
                          levels=args.levels, semi_threshold=args.semi_threshold)
    torch.cuda.synchronize()
    t_setup = time.perf_counter() - t0
    log(f"setup {t_setup * 1e3:.1f} ms")
    u = torch.empty_like(b)

    def run(solver, steps, warmup, label):
        for _ in range(warmup):
            solver.solve(b, tol=args.tol, out=u)
        torch.cuda.synchronize()
        times, stats = [], []
        t_all = time.perf_counter()
        for _ in range(steps):
            t1 = time.perf_counter()
            _, st = solver.solve(b, tol=args.tol, out=u)
            torch.cuda.synchronize()
            times.append(time.perf_counter() - t1)
            stats.append(st)
        torch.cuda.synchronize()
        total = time.perf_counter() - t_all
        log(f"{label}: {steps} solves in {total:.3f}s, median {statistics.median(times)*1e3:.2f} ms, "
            f"iters {stats[-1].iters}, relres {stats[-1].relres:.2e}")
        return times, stats, total

    times, stats, total = run(S, args.steps, args.warmup, args.precision)
    u_mixed = u.clone()
    mean_s = total / args.steps
    st = stats[-1]

    out = {
        "metric": METRIC, "value": mean_s, "unit": "s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": mean_s * 1e3,
        "higher_is_better": False, "scaling": "weak", "vs_baseline": None,
        "dtype": {"mixed": "f32+f64", "fp64": "f64", "fp32": "f32"}[args.precision],
        "data": "synthetic",
        "config": {"workload": sh.name, "grid": [sh.nlon, sh.nlat, sh.nlev],
                   "unknowns": sh.n, "cycle": f"V({sh.nu_pre},{sh.nu_post})",
                   "tol": args.tol, "levels": st.levels, "iters": st.iters,
                   "hierarchy": "automatic" if args.levels == 0 else f"at most {args.levels} levels",
                   "precision": {"mixed": "FP32 V-cycle inside FP64 refinement",
                                 "fp64": "FP64 throughout",
                                 "fp32": "FP32 throughout"}[args.precision],
                   "smoothing": (f"Chebyshev factors on [{smooth[0]:g}, {smooth[1]:g}]"
                                 if smooth else "omega 0.8 every sweep"),
                   "semi_threshold": args.semi_threshold,
                   "coarse_sweeps": S.option("coarse_sweeps"), "omega": S.option("omega")},
        "median_s": statistics.median(times),
        "relres": st.relres,
        "setup_s": t_setup,
        "alg_GBps": st.alg_bytes / statistics.median(times) / 1e9,
        # the paper's own figures (other hardware, the operational model's
        # matrices): context beside this run, not a baseline of it
        "paper_context": {
            "solver_vs_bicgstab": "about 2x (abstract, section 1); 1.40-1.64x solver time "
                                  "in Table 1",
            "forecast_speedup": "10-15% (abstract); 8-16% total runtime in Table 1",
            "hardware": "CPU cluster, 4608, 9216 and 11520 cores (Table 1); no machine "
                        "named",
            "workload": "ENDGame 2560x1920x70, 75 h global forecast (Table 1)"},
    }
    S.set_options(profile=1)
    _, st_all = S.solve(b, tol=args.tol, out=u)
    torch.cuda.synchronize()
    S.set_options(profile=3)
    kern = {c: kernel_roofline([st_all], c) for c in st_all.kernels}
    kern = {c: v for c, v in kern.items() if v}
    dom = max(kern, key=lambda c: kern[c]["avg_ms"] * kern[c]["launches"])
    # the dominant kernel's figures from the timed solves when it is the
    # class they timed (the sweep), else from the breakdown solve
    k = kernel_roofline(stats, dom) or kern[dom]
    traffic, traffic_note = measured_traffic(sh.name, dom)
    if traffic is not None and dom == "smooth":
        # counted at 16 B per cell and launch; a launch may be two sweeps here
        traffic = round(traffic * k["bytes_per_launch"] / (16 * sh.n))
    out["roofline"] = {"bound": "hbm", "kernel_class": dom, "achieved": k["GBps"],
                       "peak": HBM_PEAK_GBPS, "unit": "GB/s",
                       "frac": k["GBps"] / HBM_PEAK_GBPS, "traffic": traffic,
                       "traffic_source": traffic_note,
                       "avg_launch_ms": k["avg_ms"], "bytes_per_launch": k["bytes_per_launch"],
                       "launches": k["launches"]}
    out["fine_level_kernels"] = {c: {"GBps": v["GBps"], "avg_ms": v["avg_ms"],
                                     "launches": v["launches"]} for c, v in kern.items()}
    for c, v in kern.items():
        note = split_note(c, v["bytes_per_launch"], sh.n)
        if note:
            out["fine_level_kernels"][c]["note"] = note

    S64 = None
    if not args.no_fp64:
        S64 = Solver.from_shell(sh, alpha, nu_pre=sh.nu_pre, nu_post=sh.nu_post,
                                precision="fp64", profile=3, smooth_interval=smooth,
                                levels=args.levels, semi_threshold=args.semi_threshold)
        times64, stats64, total64 = run(S64, args.steps, args.warmup, "fp64")
        u_fp64 = u.clone()
        out["fp64_solve_s"] = total64 / args.steps
        out["fp64_iters"] = stats64[-1].iters
        out["speedup_vs_fp64"] = (total64 / args.steps) / mean_s
        out["mixed_vs_fp64_rel_diff"] = fwd_err(u_mixed, u_fp64)

    if not args.no_adjoint:
        out["adjoint"] = adjoint_run(S, sh, args.tol)
        out["adjoint"]["forward_ms_per_iteration"] = mean_s * 1e3 / max(st.iters, 1)
    if args.timesteps > 0:
        out["timestep"] = timestep_run(S, sh, alpha, b, args.timesteps, args.tol)

    # Accuracy: the forward error ||u - u_ref|| / ||u_ref|| of the timed
    # solves against a reference solution of H u = b, and the loosest
    # tolerance at which the timed solve's forward error is at most 1e-8.
    uref = None
    use_oracle = not args.no_cpu_baseline and sh.n <= 100_000_000
    if use_oracle:
        uref_np, base, ref = oracle_reference(sh, smooth, args.semi_threshold, args.tol)
        out["cpu_baseline"] = base
        uref = torch.from_numpy(uref_np).to(dev)
        del uref_np
    elif not args.no_accuracy:
        S_ref = S64 or Solver.from_shell(sh, alpha, nu_pre=sh.nu_pre, nu_post=sh.nu_post,
                                         precision="fp64", smooth_interval=smooth,
                                         levels=args.levels,
                                         semi_threshold=args.semi_threshold)
        uref, ref = gpu_reference(S_ref, sh, b, args.semi_threshold)
    if uref is not None:
        acc = {"reference": ref, "fwd_err": fwd_err(u_mixed, uref)}
        if S64 is not None:
            acc["fwd_err_fp64"] = fwd_err(u_fp64, uref)
        if not args.no_accuracy:
            sweep = []
            for tol in (1e-9, 1e-10, 1e-11, 1e-12):
                ts = []
                for _ in range(3):
                    t1 = time.perf_counter()
                    _, st_t = S.solve(b, tol=tol, out=u)
                    torch.cuda.synchronize()
                    ts.append(time.perf_counter() - t1)
                sweep.append({"tol": tol, "ms": statistics.median(ts) * 1e3,
                              "iters": st_t.iters, "relres": st_t.relres,
                              "fwd_err": fwd_err(u, uref)})
            acc["tol_sweep"] = sweep
            ok = [r for r in sweep if r["fwd_err"] <= 1e-8]
            acc["to_fwd_err_1e-8"] = ok[0] if ok else None
            log("forward errors: timed " + f"{acc['fwd_err']:.2e}" + "; " + ", ".join(
                f"tol {r['tol']:g}: {r['ms']:.2f} ms, {r['iters']} it, {r['fwd_err']:.2e}"
                for r in sweep))
        out["accuracy"] = acc
        del uref
    if S64 is not None:
        S64.close()

    if use_oracle and sh.n <= 1_000_000:
        out["oracle_solve"] = oracle_solve(sh, args.tol, smooth, args.semi_threshold,
                                           u_mixed.cpu().numpy())
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
