"""Benchmark: EXX pair Poisson solves/s and EXX evaluation time on one MI355X.

A step is one full exx_eval (pair list, pair densities, moments, boundary
values, CG solves, E_xx, D_xx and sigma_xx) over every pair of a water-like
workload, with the orbitals already resident in HBM.  The default workload is
the 512-molecule set, the largest that one GPU holds (cubic 47.0 bohr cell,
240^3 grid, 2048 orbitals as FP32 grid arrays (113 GB), R_pair 10, R_PE 6,
R_ME 9 bohr, l_max 8, 19-point stencil, CG tol 1e-10), timed in FP64 and in
mixed precision; the mixed figure is the headline value.  Prints one JSON line.

  python bench.py [--gpus 1] [--steps K] [--warmup W] [--precision both|fp64|mixed]
                  [--workload water512|water64|water128|water256|hex64|tri64]
                  [--time-budget S]

The wall-clock budget (default 420 s from the start of the process) caps the
warm-up and timed evaluations: after the first warm-up evaluation (which runs
the CG autotuner) the remaining warm-ups and the timed steps are cut to what
fits, at least one timed step per precision.  The JSON line reports the
warm-ups and timed steps actually run (`steps`, `warmup`) beside the ones
asked for.

water256 runs as the MD-like repeated-call case: per-orbital sphere radii (9
classes), a fixed pair capacity, one eager warm-up call (which runs the CG
autotuner), the call recorded into a HIP graph, then K replays; before each
replay every centre moves 0.02 bohr and the orbitals are regenerated on the
device in the same buffers (not timed).  Each replay is timed with HIP events.
By default each replay's CG starts from the pair's solution of the previous
replay (--no-warm-start: from zero).

Every evaluation's statistics are checked: a pair whose CG did not converge
(iteration cap, breakdown or non-finite norm) makes the run print the failing
pairs and the CG variant of each sphere class to stderr and exit with status 3.

The roofline entry is for the dominant kernel, the persistent CG solve:
algorithmic bytes (8 N_PE b per pair per iteration, 6 in a fused quad sweep) over
the summed device time of its launches in the timed region, from HIP events
that the library records on its stream (eager calls only).  moments_roofline
gives the moment contraction's matrix-core rate.  The CPU baseline is the FP64
oracle on a bounded sample of the same workload, on the host's cores: every
pair among the orbitals nearest one orbital (the oracle reads only those
orbitals, copied back from the device).
"""
from __future__ import annotations

import argparse
import hashlib
import json
import math
import os
import statistics
import sys
import time

T_START = time.perf_counter()
ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0
MFMA_PEAK_TFLOPS = {"fp64": 78.6, "mixed": 2500.0}   # dense FP64 and BF16 matrix peaks
METRIC = "EXX pair Poisson solves/s + EXX eval time, mixed vs FP64 at 1e-6 tol"
TRAFFIC_FILE = os.path.join(ROOT, "profiles", "solve_traffic.json")
# sources of the CG kernel, its launch shape and its data layout: the stored
# counter traffic is used only while these are unchanged
KERNEL_SOURCES = ["paper_2011_07209_amd/csrc/solve_impl.h", "paper_2011_07209_amd/csrc/solve.hip",
                  "paper_2011_07209_amd/csrc/solve_n1.hip", "paper_2011_07209_amd/csrc/solve_n2.hip",
                  "paper_2011_07209_amd/csrc/solve_n3.hip", "paper_2011_07209_amd/csrc/exx_internal.h",
                  "paper_2011_07209_amd/csrc/plan_geometry.cpp", "paper_2011_07209_amd/csrc/pcg_impl.h",
                  "paper_2011_07209_amd/csrc/pcg_cols.h"]
MOLECULES = {"tiny16": 4, "water64": 64, "water128": 128, "water256": 256, "water512": 512, "hex64": 64,
             "tri64": 64}   # molecule-equivalents (4 orbitals each)
D_CHECK_ROWS = 16   # orbitals whose D the mixed/FP64 comparison uses
CPU_SAMPLE_ORBITALS = 32
DTYPE = {"fp64": "f64", "mixed": "f32+f64 (FP32 CG, FP64 dots and reliable updates; split-bf16 MFMA moments)"}


class CgFailure(RuntimeError):
    """A pair's CG did not converge in an evaluation."""


def kernel_hash() -> str:
    h = hashlib.sha256()
    for f in KERNEL_SOURCES:
        with open(os.path.join(ROOT, f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def stored_traffic(workload: str, precision: str, threads: int, depth: int, layout: int):
    """HBM bytes per solve launch from the committed counter runs, or None when
    the kernels changed since they were taken or the run used another CG
    variant (workgroup size, load depth, column or quad layout) than the one
    measured."""
    try:
        with open(TRAFFIC_FILE) as f:
            d = json.load(f)
    except (OSError, ValueError):
        return None
    e = d.get(f"{workload}/{precision}")
    if not e or e.get("kernel_hash") != kernel_hash():
        return None
    args = [a.strip() for a in e.get("kernel", "").split("<", 1)[-1].rstrip(">").split(",")]
    if len(args) < 7 or args[2] != str(threads) or args[3] != str(depth):
        return None
    if (args[6] == "true") != (layout == 2):
        return None
    return e.get("hbm_bytes_per_launch")


def plan_steps(now, deadline, t_eval, asked, minimum=1):
    """Evaluations of about t_eval seconds that fit between now and deadline,
    at most `asked`, at least `minimum`."""
    if t_eval <= 0:
        return max(minimum, asked)
    fit = int((deadline - now) / t_eval)
    return max(minimum, min(asked, fit))


def describe(cfg) -> str:
    grid = "x".join(str(n) for n in cfg.grid)
    cell = "x".join(f"{x:g}" for x in cfg.cell)
    if cfg.general:
        import numpy as np
        h = cfg.h
        ang = [math.degrees(math.acos(np.dot(h[:, i], h[:, j]) / np.linalg.norm(h[:, i]) / np.linalg.norm(h[:, j])))
               for i, j in ((1, 2), (0, 2), (0, 1))]
        cell += " (angles " + "/".join(f"{x:.0f}" for x in ang) + " deg, NK Laplacian)"
    radii = (f"R_PE {cfg.R_orb_range[0]:g}-{cfg.R_orb_range[1]:g} per orbital ({cfg.R_PE_classes[2]} classes)"
             if cfg.R_PE_classes else f"R_PE {cfg.R_PE:g}")
    kind = (f"water-like {MOLECULES[cfg.key]}-molecule set, {cfg.lattice} lattice" if cfg.lattice else
            "Gaussian-times-polynomial orbitals at uniform random centres")
    return (f"{cfg.key}: {kind}, cell {cell} bohr, "
            f"{grid} grid, {cfg.n_orb} orbitals ({cfg.orb_dtype}), R_pair {cfg.R_pair:g}, {radii}, "
            f"R_ME {cfg.R_ME:g}, l_max {cfg.l_max}, n {cfg.stencil_n}, CG tol {cfg.cg_tol:g}")


def cpu_model() -> str:
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def nearest_orbitals(cfg, centres, i0, k):
    """The k orbitals nearest orbital i0 (minimum image), i0 first."""
    import numpy as np
    h = cfg.h
    s = (centres - centres[i0]) @ np.linalg.inv(h).T
    s -= np.round(s)
    d = s @ h.T
    return [int(x) for x in np.argsort((d * d).sum(1), kind="stable")[:k]]


def cpu_baseline(cfg, orbs, orb_t, n_pairs_total):
    """The FP64 oracle on every pair among the CPU_SAMPLE_ORBITALS orbitals
    nearest orbital 0: a compact cluster whose pairs have the workload's sphere
    sizes and stencil, so its pair rate stands for the whole set's.  The oracle
    reads those orbitals only, copied back from the device (the values the GPU
    path read)."""
    import torch
    import oracle
    threads = int(os.environ.get("OMP_NUM_THREADS", "0")) or os.cpu_count() or 1
    idx = nearest_orbitals(cfg, orbs.centres, 0, min(CPU_SAMPLE_ORBITALS, cfg.n_orb))
    phi = orb_t[idx].to(torch.float64).cpu().numpy()
    R_sub = orbs.R_orb[idx] if cfg.R_PE_classes is not None else None
    P = oracle.make_params(cfg.h, cfg.grid, cfg.R_pair, cfg.R_PE, cfg.R_ME, cfg.l_max, cfg.stencil_n, cfg.cg_tol,
                           R_PE_classes=cfg.R_PE_classes, n_threads=threads)
    t0 = time.perf_counter()
    r = oracle.evaluate(P, phi, orbs.centres[idx], R_sub, want_D=True)
    dt = time.perf_counter() - t0
    n = len(r["pairs"])
    rate = n / dt
    return {"value": rate, "unit": "pair solves/s", "cores": threads, "kind": "oracle",
            "sample": f"all {n} pairs among the {len(idx)} orbitals nearest orbital 0 (full E/D/sigma per pair), "
                      f"{dt:.1f} s",
            "cpu_model": cpu_model(), "sample_s": dt, "sample_pairs": n,
            "extrapolated_eval_s": n_pairs_total / rate}


def _plan(exx, cfg, precision, **kw):
    opt = dict(stencil_n=cfg.stencil_n, cg_tol=cfg.cg_tol,
               precision=exx.EXX_PREC_MIXED if precision == "mixed" else exx.EXX_PREC_FP64,
               workspace_gb=24.0 if cfg.key == "water512" else 48.0)
    if cfg.R_PE_classes is not None:
        opt.update(R_PE_min=cfg.R_PE_classes[0], R_PE_step=cfg.R_PE_classes[1], R_PE_nclass=cfg.R_PE_classes[2])
    opt.update(kw)
    return exx.Plan(cfg.h, cfg.grid, cfg.R_pair, cfg.R_PE, cfg.R_ME, cfg.l_max, **opt)


def variants(st):
    """The CG variant of each sphere class, for the record and for failures."""
    out = []
    for t, d, l, p, dl in zip(st["class_threads"], st["class_depth"], st["class_layout"], st["class_pairs"],
                              st["class_refine_delta"]):
        v = {"threads": t, "depth": d, "layout": "quads" if l == 2 else "columns", "pairs": p}
        if dl > 0:
            v["refine_delta"] = dl
        out.append(v)
    return out


def checked_stats(exx, plan, tag):
    """Statistics of the last evaluation; a pair whose CG did not converge
    raises CgFailure after its pairs and the class variants went to stderr."""
    st = plan.stats(allow_noconv=True)
    if st["cg_restarts"]:
        print(f"[bench] {tag}: {st['cg_restarts']} CG restarts from the last FP64 solution", file=sys.stderr,
              flush=True)
    if st["n_unconverged"] == 0:
        return st
    pr = plan.pair_results()
    bad = [k for k in range(len(pr["exit"])) if pr["exit"][k] != exx.EXX_CG_CONVERGED]
    print(f"[bench] {tag}: {st['n_unconverged']} of {st['n_pairs']} pairs did not converge (cap {st['n_cg_cap']}, "
          f"breakdown {st['n_cg_breakdown']}, non-finite {st['n_cg_nonfinite']}); CG variant per class: "
          f"{variants(st)}", file=sys.stderr, flush=True)
    for k in bad[:32]:
        print(f"[bench]   pair ({pr['ij'][k][0]},{pr['ij'][k][1]}) exit {exx.CG_EXIT_NAMES.get(int(pr['exit'][k]))} "
              f"iterations {pr['iters'][k]} rel_res {pr['rel_res'][k]:.3e} updates {pr['updates'][k]} "
              f"restarts {pr['restarts'][k]}", file=sys.stderr, flush=True)
    raise CgFailure(f"{tag}: {st['n_unconverged']} pairs did not converge")


def run_precision(exx, torch, synth, cfg, orbs, bufs, precision, steps, warmup, graph, deadline, warm=False,
                  cmp_step=None):
    """Times up to `steps` evaluations (after up to `warmup`) in one precision,
    cut to what fits before `deadline` (perf_counter seconds); returns the
    measurement and the outputs of the last evaluation (of trajectory step
    `cmp_step` in graph mode when given, so that two precisions are compared
    at the same centres)."""
    orb_t, cen_t, R_t, D = bufs
    dev = orb_t.device
    E = torch.zeros(1, dtype=torch.float64, device=dev)
    S = torch.zeros(9, dtype=torch.float64, device=dev)
    kw = {"autotune": 1 if warmup > 0 else 0}
    if graph:
        probe = _plan(exx, cfg, precision)
        n0 = probe.count_pairs(cen_t, R_t)
        probe.close()
        kw["max_pairs"] = int(math.ceil(1.05 * n0)) + 64   # displacements change the pair list a little
        kw["warm_start"] = 1 if warm else 0
    plan = _plan(exx, cfg, precision, **kw)
    geo = plan.geometry()
    n_warm_max = max(warmup, 1 if graph else 0)
    n_warm, t_eval = 0, 0.0
    restarts = 0
    while n_warm < n_warm_max:
        t0 = time.perf_counter()
        plan.eval(orb_t, cen_t, E, D, S, R_t)
        torch.cuda.synchronize()
        st = checked_stats(exx, plan, f"{cfg.key} {precision} warmup {n_warm + 1}")
        restarts += st["cg_restarts"]
        t_eval = time.perf_counter() - t0
        n_warm += 1
        print(f"[bench] {cfg.key} {precision} warmup {n_warm}/{n_warm_max} {t_eval:.1f} s E={E.item():.10f} "
              f"variants {variants(st)}", file=sys.stderr, flush=True)
        # further warm-ups only while every timed step asked for still fits after them
        if time.perf_counter() + (steps + 1) * t_eval > deadline:
            break
    zero = {"solve_launches": 0, "solve_ms_total": 0.0, "cg_alg_bytes_total": 0.0}
    s0 = plan.stats(allow_noconv=True) if n_warm > 0 else zero
    n_steps = plan_steps(time.perf_counter(), deadline, t_eval, steps)
    step_ms, step_pairs, step_iters, step_warm = [], [], [], []
    s_last = None
    snap = None
    if graph:
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        g = torch.cuda.CUDAGraph()
        with torch.cuda.stream(side):
            plan.set_stream(side)
            with torch.cuda.graph(g, stream=side):
                plan.eval(orb_t, cen_t, E, D, S, R_t)
        torch.cuda.current_stream().wait_stream(side)
        plan.set_stream(torch.cuda.current_stream())
        ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        traj = orbs
        for k in range(n_steps):
            traj = synth.displace(cfg, traj, k + 1)
            synth.fill_orbitals_device(cfg, traj, dev, out=orb_t)
            cen_t.copy_(torch.from_numpy(traj.centres).to(dev))
            torch.cuda.synchronize()
            ev0.record()
            g.replay()
            ev1.record()
            torch.cuda.synchronize()
            st = checked_stats(exx, plan, f"{cfg.key} {precision} replay {k + 1}")
            restarts += st["cg_restarts"]
            step_ms.append(ev0.elapsed_time(ev1))
            step_pairs.append(st["n_pairs"])
            step_iters.append(st["cg_iter_sum"] / max(1, st["n_pairs"]))
            step_warm.append(st["warm_pairs"])
            s_last = st
            if k + 1 == (cmp_step or n_steps):
                snap = (k + 1, E.item(), S.cpu().numpy().reshape(3, 3, order="F"), D[:D_CHECK_ROWS].double().cpu())
            print(f"[bench] {cfg.key} {precision} replay {k + 1}/{n_steps}: {step_ms[-1]:.1f} ms, {st['n_pairs']} pairs "
                  f"({st['warm_pairs']} warm-started), mean iterations {step_iters[-1]:.1f}, E={E.item():.10f}",
                  file=sys.stderr, flush=True)
        del g
        ms = sum(step_ms) / len(step_ms)
        value = sum(step_pairs) / (sum(step_ms) / 1000.0)
        cg = None   # replays record no per-kernel events
    else:
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(n_steps):
            plan.eval(orb_t, cen_t, E, D, S, R_t)
            st = checked_stats(exx, plan, f"{cfg.key} {precision} step {len(step_ms) + 1}")   # waits for the eval
            restarts += st["cg_restarts"]
            step_ms.append(st["eval_ms"])
            step_pairs.append(st["n_pairs"])
            step_iters.append(st["cg_iter_sum"] / max(1, st["n_pairs"]))
            s_last = st
            print(f"[bench] {cfg.key} {precision} step {len(step_ms)}/{n_steps}: {st['eval_ms']:.1f} ms on the device",
                  file=sys.stderr, flush=True)
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        ms = (t1 - t0) * 1000.0 / n_steps
        value = s_last["n_pairs"] / (ms / 1000.0)
        launches = s_last["solve_launches"] - s0["solve_launches"]
        solve_ms = s_last["solve_ms_total"] - s0["solve_ms_total"]
        alg = s_last["cg_alg_bytes_total"] - s0["cg_alg_bytes_total"]
        achieved = (alg / max(launches, 1)) / (solve_ms / max(launches, 1) / 1000.0) / 1e9 if solve_ms > 0 else 0.0
        # (every class of the workloads runs the preconditioned CG: their tolerance, iteration cap and spheres allow it)
        cg = {"bound": "hbm", "kernel": "k_pcg_mixed" if precision == "mixed" else "k_pcg",
              "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": achieved / HBM_PEAK_GBS,
              "traffic": stored_traffic(cfg.key, precision, s_last["solve_threads"], s_last["solve_depth"],
                                        s_last["cg_layout"]),
              "alg_bytes_per_launch": alg / max(launches, 1),
              "launch_ms": solve_ms / max(launches, 1)}
    print(f"[bench] {cfg.key} {precision} timed {n_steps} steps: {ms:.1f} ms/step E={E.item():.10f}", file=sys.stderr,
          flush=True)
    moments = None
    if s_last["moment_ms"] > 0:
        # moment contraction of the last evaluation: executed MFMA flops (padded
        # rows and points, three products in the mixed path) and the algorithmic
        # 2 N_lm N_PE per pair, over the device time of its launches
        mom_s = s_last["moment_ms"] / 1000.0
        mfma = s_last["moment_mfma_flops"] / mom_s / 1e12
        alg_tf = s_last["moment_flops"] / mom_s / 1e12
        peak = MFMA_PEAK_TFLOPS[precision]
        moments = {"bound": "mfma", "kernel": "k_moments_bf16" if precision == "mixed" else "k_moments_f64",
                   "achieved": mfma, "peak": peak, "unit": "TFLOP/s", "frac": mfma / peak,
                   "algorithmic_tflops": alg_tf, "algorithmic_frac": alg_tf / peak,
                   "density_read_gbs": 8.0 * s_last["moment_flops"] / (2.0 * (cfg.l_max + 1) ** 2) / mom_s / 1e9,
                   "launch_ms": s_last["moment_ms"]}
    plan.close()
    n_pairs = s_last["n_pairs"]
    out = {
        "value": value, "ms_per_step": ms, "n_pairs": n_pairs, "n_pe": geo["n_pe"],
        "steps": n_steps, "warmup": n_warm,
        "eval_ms_median": statistics.median(step_ms), "eval_ms_steps": step_ms,
        "cg_iters_mean_steps": step_iters, "warm_pairs_steps": step_warm,
        "cg_iters_mean": s_last["cg_iter_sum"] / max(1, n_pairs), "cg_iters_max": s_last["cg_iter_max"],
        "updates_max": s_last["refine_passes_max"], "max_rel_residual": s_last["max_rel_residual"],
        "cg_restarts": restarts,
        "solve_variant": {"threads": s_last["solve_threads"], "depth": s_last["solve_depth"],
                          "layout": "quads" if s_last["cg_layout"] == 2 else "columns", "tune_ms": s_last["tune_ms"],
                          "per_class": variants(s_last)},
        "t_pairlist_ms": s_last["t_pairlist_ms"], "t_reduce_ms": s_last["t_reduce_ms"],
        "roofline": cg, "moments_roofline": moments,
        "E": E.item(), "sigma": S.cpu().numpy().reshape(3, 3, order="F"),
        "D_rows": D[:D_CHECK_ROWS].double().cpu(),
    }
    if graph:   # the outputs of the compared trajectory step (None: this run did not reach it)
        out["compared_step"] = snap[0] if snap else None
        if snap:
            out["E"], out["sigma"], out["D_rows"] = snap[1], snap[2], snap[3]
    return out


def main(argv=None):
    ap = argparse.ArgumentParser(description=__doc__, formatter_class=argparse.RawDescriptionHelpFormatter)
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=None, help="timed steps asked for (default 5; 10 replays for "
                                                            "water256), cut to the time budget")
    ap.add_argument("--warmup", type=int, default=1, help="warm-up evaluations asked for, cut to the time budget")
    ap.add_argument("--workload", choices=sorted(MOLECULES), default="water512")
    ap.add_argument("--precision", choices=["both", "fp64", "mixed"], default="both",
                    help="both: time the FP64 and the mixed path, report the mixed one as the value")
    ap.add_argument("--time-budget", type=float, default=420.0,
                    help="wall-clock seconds from the start of the process that the run aims to stay within")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-warm-start", action="store_true",
                    help="water256: start every replay's CG from zero instead of the previous solution")
    ap.add_argument("--copy-probe-gib", type=float, default=0.0,
                    help="after the timed steps, copy this many GiB device-to-device (counter calibration)")
    args = ap.parse_args(argv)

    if args.gpus != 1:
        print(f"bench.py runs on one GPU only; --gpus {args.gpus} is not supported (the library has no multi-GPU "
              f"pair sharding)", file=sys.stderr)
        return 2

    import numpy as np
    import torch

    from paper_2011_07209_amd import exx, synth

    if not torch.cuda.is_available():
        print("bench.py needs a GPU", file=sys.stderr)
        return 1
    dev = torch.device("cuda:0")
    cfg = synth.CONFIGS[args.workload]
    graph = cfg.key == "water256"
    steps = args.steps if args.steps is not None else (10 if graph else 5)
    orbs = synth.make_orbitals(cfg)
    t0 = time.perf_counter()
    orb_t = synth.fill_orbitals_device(cfg, orbs, dev)
    cen_t = torch.from_numpy(orbs.centres).to(dev)
    R_t = torch.from_numpy(orbs.R_orb).to(dev) if cfg.R_PE_classes is not None else None
    D = torch.empty_like(orb_t)
    torch.cuda.synchronize()
    print(f"[bench] {cfg.key}: {orb_t.numel() * orb_t.element_size() / 1e9:.1f} GB of orbitals generated on the "
          f"device in {time.perf_counter() - t0:.1f} s", file=sys.stderr, flush=True)

    # the pair count for the extrapolation of the CPU baseline
    probe = _plan(exx, cfg, "fp64")
    n_pairs_total = probe.count_pairs(cen_t, R_t)
    probe.close()
    cpu = None
    if not args.no_cpu_baseline:
        cpu = cpu_baseline(cfg, orbs, orb_t, n_pairs_total)
        print(f"[bench] cpu baseline: {cpu['value']:.1f} pair solves/s on {cpu['cores']} threads ({cpu['sample']})",
              file=sys.stderr, flush=True)

    precs = ["fp64", "mixed"] if args.precision == "both" else [args.precision]
    res = {}
    deadline_all = T_START + args.time_budget
    try:
        for k, p in enumerate(precs):
            if graph:   # every precision replays the same trajectory from the same start
                synth.fill_orbitals_device(cfg, orbs, dev, out=orb_t)
                cen_t.copy_(torch.from_numpy(orbs.centres).to(dev))
            # the FP64 phase takes half of what is left; the mixed phase the rest
            now = time.perf_counter()
            deadline = now + (deadline_all - now) * (0.5 if k + 1 < len(precs) else 1.0)
            # graph mode: compare the precisions at the trajectory step the first one ended on
            cmp = res[precs[0]]["steps"] if graph and k > 0 else None
            res[p] = run_precision(exx, torch, synth, cfg, orbs, (orb_t, cen_t, R_t, D), p, steps, args.warmup,
                                   graph, deadline, warm=graph and not args.no_warm_start, cmp_step=cmp)
    except CgFailure as e:
        print(f"[bench] FAILED: {e}", file=sys.stderr, flush=True)
        return 3
    main_p = "mixed" if "mixed" in res else "fp64"
    r = res[main_p]

    accuracy = None
    if "fp64" in res and "mixed" in res and (not graph or res["mixed"].get("compared_step")):
        a, b = res["mixed"], res["fp64"]
        n_mol = MOLECULES[cfg.key]
        dd = (a["D_rows"] - b["D_rows"]).abs().reshape(D_CHECK_ROWS, -1)
        accuracy = {
            "vs": "FP64 GPU path (itself parity-tested against the FP64 oracle)",
            "dE_Ha_per_molecule": abs(a["E"] - b["E"]) / n_mol,
            "sigma_rel_1norm": float(np.abs(a["sigma"] - b["sigma"]).sum() / np.abs(b["sigma"]).sum()),
            "D_rel_1norm": float(dd.sum().item() / b["D_rows"].abs().sum().item()),
            "D_max_abs_rel": float((dd.max(1).values / b["D_rows"].abs().reshape(D_CHECK_ROWS, -1).max(1).values)
                                   .max().item()),
            "D_rows_compared": D_CHECK_ROWS,
            "targets": {"dE_Ha_per_molecule": 1e-6, "sigma_rel_1norm": 1e-6},
        }
        if graph:
            accuracy["trajectory_step"] = a["compared_step"]

    if args.copy_probe_gib > 0:
        nbytes = int(args.copy_probe_gib * (1 << 30))
        del D
        a = torch.empty(nbytes // 8, dtype=torch.float64, device=dev).fill_(1.0)
        b = torch.empty_like(a)
        b.copy_(a)
        torch.cuda.synchronize()
        del a, b

    def summary(x):
        return {k: x[k] for k in ("value", "ms_per_step", "steps", "warmup", "eval_ms_median", "eval_ms_steps",
                                  "cg_iters_mean_steps", "warm_pairs_steps", "cg_iters_mean", "cg_iters_max",
                                  "updates_max", "max_rel_residual", "cg_restarts", "solve_variant", "t_pairlist_ms",
                                  "t_reduce_ms", "roofline", "moments_roofline")}

    out = {
        "metric": METRIC,
        "value": r["value"],
        "unit": "pair solves/s",
        "n_gpus": 1,
        "steps": r["steps"],
        "warmup": r["warmup"],
        "ms_per_step": r["ms_per_step"],
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": DTYPE[main_p],
        "data": "synthetic",
        "config": {
            "workload": describe(cfg),
            "precision": main_p,
            "n_pairs": r["n_pairs"],
            "n_pe": r["n_pe"],
            "exx_eval_s": r["ms_per_step"] / 1000.0,
            "timing": ("mean of event-timed graph replays over displaced centres (orbital regeneration not timed)"
                       if graph else "host clock around the timed exx_eval calls"),
            "warm_start": bool(graph and not args.no_warm_start),
            "E_xx": r["E"],
            "steps_asked": steps,
            "warmup_asked": args.warmup,
            "time_budget_s": args.time_budget,
            "wall_s": time.perf_counter() - T_START,
        },
        "roofline": r["roofline"],
        "moments_roofline": r["moments_roofline"],
        "cpu_baseline": cpu,
        "by_precision": {p: summary(x) for p, x in res.items()},
        "mixed_accuracy": accuracy,
    }
    if "fp64" in res and "mixed" in res:
        out["mixed_speedup_vs_fp64"] = res["mixed"]["value"] / res["fp64"]["value"]
    print(json.dumps(out), flush=True)
    return 0


if __name__ == "__main__":
    sys.exit(main())
