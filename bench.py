"""Benchmark: converged kappa_eff solves/s (and cell*dir*MFP DoF/s) of the
aMFP-BTE hot path on one MI355X, FP32-sweep form and FP64 form, at 1e-4
relative kappa error, on the 128x128 porous-cell workload.

A step is one converged kappa_eff computation through the C ABI: the Fourier
first guess, then source-iteration passes (batched (m,l) solves + reductions)
until the estimated kappa error meets the target.  Inputs (mesh tables,
material weights, sigma) are resident on the device before the timed region
starts.  The same JSON line also carries the 3D membrane (64x64x16, 288
directions x 30 MFPs) and the 64-geometry batch, each at the same error
target, the Fourier-only batch, and one synthetic mode table solved by the
aMFP interpolation and by the mode-resolved iteration (skip them with
--no-extras).
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

METRIC = ("converged κ_eff solves/s and cell·dir·MFP DoF/s, FP32 vs FP64, "
          "at 1e-4 rel err")
# MI355X published peaks: HBM3E 8 TB/s; vector FP32 78.6 TFLOP/s without
# packed FP32 (this build switches packed FP32 off; 157.3 with it), FP64 78.6
PEAK = {"hbm_gbs": 8000.0, "fp32_vector_tflops": 78.6, "fp64_vector_tflops": 78.6}
# Algorithmic HBM bytes of one upwind sweep of one system, per solid cell: the
# apply-equivalent of Eq. (iter2)'s left side reads x once and writes y once
# (2 words of the compute type); the per-cell tables are shared by all systems.
WORDS_PER_CELL_SWEEP = 2
# algorithmic flops of one upwind sweep per solid cell: the triangular update
# x = (b + c_x x_up,x + c_y x_up,y [+ c_z x_up,z]) / d  (2 or 3 FMA + 1 divide
# counted as 3)
FLOPS_PER_CELL_SWEEP = {2: 5, 3: 6}
# Operating points (the GPU tests check each against the oracle).  Plain
# Algorithm 1: the error-estimate stop rule at half the 1e-4 target.  Mixed
# ("_aa"): Anderson depth 8 on (T_L, T_w), relative change and estimated
# iterate error both <= 5e-5.  Both: a forcing term of 0.3 on the per-pass wrap
# solve, the wrap correction lagged into the next pass, and a Fourier first
# guess to 1e-3 (plain) or 3e-3 (mixed): its error is far below the
# BTE-Fourier difference the passes remove (the fastest settings measured).
_COMMON = dict(inner_rtol=0.3, lag_wrap=1, passes_per_graph=4, max_outer=5000)
OP = {
    "fp32": dict(precision=1, outer_tol=5e-5, stop_rule=1, inner_tol=1e-5, fourier_tol=1e-3, **_COMMON),
    "fp64": dict(precision=0, outer_tol=5e-5, stop_rule=1, inner_tol=1e-8, fourier_tol=1e-3, **_COMMON),
    "fp32_aa": dict(precision=1, outer_tol=5e-5, stop_rule=0, accel=8, inner_tol=1e-5, fourier_tol=3e-3,
                    **_COMMON),
    "fp64_aa": dict(precision=0, outer_tol=5e-5, stop_rule=0, accel=8, inner_tol=1e-8, fourier_tol=3e-3,
                    **_COMMON),
}
HEADLINE = "fp32_aa"
FORMS = ("fp32_aa", "fp64_aa", "fp32", "fp64")
REF = dict(precision=0, outer_tol=1e-10, stop_rule=0, accel=8, inner_tol=1e-12, fourier_tol=1e-11,
           passes_per_graph=8, max_outer=20000)
# HBM traffic of the FP32 pass kernel on the 128x128 workload at the headline
# operating point, per launch (rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE over one
# solve, each scaled by the same counter on a plain 256 MiB copy); valid only
# for the kernel source it was taken on.
TRAFFIC = {"kernels_sha256": "71a32952867f9f08b5fb6629e1aeb9e158356e62e952d6877406c39bdba15542",
           "fetch_bytes": 27270122, "write_bytes": 88096960}


def parse():
    p = argparse.ArgumentParser()
    p.add_argument("--gpus", type=int, default=1)
    p.add_argument("--steps", type=int, default=10)
    p.add_argument("--warmup", type=int, default=2)
    p.add_argument("--no-cpu", action="store_true", help="skip the CPU oracle baseline")
    p.add_argument("--no-extras", action="store_true", help="skip the 3D and batch workloads")
    p.add_argument("--cpu-seconds", type=float, default=20.0)
    p.add_argument("--workload", default="cfg2", choices=["cfg1", "cfg2", "cfg4", "cfg5", "umesh"],
                   help="umesh: only with --profile (the unstructured-mesh leg)")
    p.add_argument("--profile", action="store_true",
                   help="only run --steps solves of --workload at the headline operating point "
                        "with direct launches (for rocprofv3 counter runs) and exit")
    p.add_argument("--copy-probe", type=int, default=0,
                   help="only run a plain device copy of this many bytes (scales rocprofv3 "
                        "FETCH_SIZE / WRITE_SIZE) and exit")
    return p.parse_args()


def kernels_sha():
    """Of the structured path's device sources, in name order."""
    src = os.path.join(ROOT, "paper_2106_02764_amd", "csrc")
    h = hashlib.sha256()
    for name in sorted(os.listdir(src)):
        if name.endswith((".hip", ".h")) and not name.startswith("u"):
            with open(os.path.join(src, name), "rb") as f:
                h.update(f.read())
    return h.hexdigest()


def copy_probe(nbytes):
    import torch
    x = torch.ones(nbytes // 4, dtype=torch.float32, device="cuda")
    y = torch.empty_like(x)
    for _ in range(3):
        y.copy_(x)
    torch.cuda.synchronize()
    print(json.dumps({"copy_probe_bytes": nbytes, "launches": 3}), flush=True)


def make_workload(name):
    from inputs import gen
    return {"cfg1": gen.config1, "cfg2": gen.config2, "cfg4": gen.config4, "cfg5": gen.config5}[name]()


def describe(name, w):
    if name == "cfg2":
        return ("128x128 periodic cell, centred circular pore r=%.3f nm (seeded), L=100 nm, "
                "48 directions x 30 MFPs (1 nm..100 um), lognormal kernel, 1e-4 rel kappa error"
                % (w.meta["pore_radius"] * 1e9))
    if name == "cfg5":
        return ("3D membrane 64x64x16, L=200 nm, t=50 nm, cylindrical through-pore r=0.3 L, "
                "diffuse top/bottom, 288 directions x 30 MFPs, 1e-4 rel kappa error")
    return name


def run_solves(solver, opts, steps, warmup):
    """Timed solves; returns wall time and the summed solver statistics."""
    import torch
    for _ in range(warmup):
        solver.solve(opts, want_T_L=False)
    torch.cuda.synchronize()
    acc = {"sweep_ms": 0.0, "reduce_ms": 0.0, "fourier_ms": 0.0, "sweep_launches": 0,
           "outer_iters": 0, "sweeps": 0, "inner_iters": 0}
    t0 = time.perf_counter()
    for _ in range(steps):
        out = solver.solve(opts, want_T_L=False)
        for k in acc:
            acc[k] += out[k]
    torch.cuda.synchronize()
    acc["seconds"] = time.perf_counter() - t0
    acc["kappa"] = out["kappa"]
    acc["status"] = out["status"]
    return acc


def leg(P, solver, w, name, steps, warmup, kref, kor):
    """Throughput leg (pass kernels replayed as HIP graphs), then the same
    solves with HIP events around every launch on the library's stream
    (direct launches) for the per-kernel durations."""
    o = solver.opts(**OP[name])
    # launch shape (systems per workgroup) from the tuner, outside the timing
    choice = P.autotune.tune(solver, o)
    P.autotune.apply(o, choice)
    r = run_solves(solver, o, steps, warmup)
    ot = P.autotune.apply(solver.opts(**OP[name], timing=1), choice)
    rt = run_solves(solver, ot, steps, 0)
    out = {"solves_per_s": steps / r["seconds"], "ms_per_solve": 1e3 * r["seconds"] / steps,
           "dof_per_s": w.dof * steps / r["seconds"], "kappa": r["kappa"], "status": r["status"],
           "passes_per_solve": r["outer_iters"] / steps, "sweeps_per_system_pass":
           r["sweeps"] / max(r["outer_iters"] * w.n_systems, 1),
           "kappa_rel_err_vs_fp64_ref": abs(r["kappa"] - kref) / abs(kref),
           "opts": OP[name], "launch_shape": {"waves_by_class": choice["waves_by_class"],
                                             "dispatch": choice["dispatch"]},
           "timed_leg": {"solves_per_s": steps / rt["seconds"], "sweep_ms": rt["sweep_ms"],
                         "reduce_ms": rt["reduce_ms"], "fourier_ms": rt["fourier_ms"],
                         "sweep_launches": rt["sweep_launches"], "sweeps": rt["sweeps"]}}
    if kor is not None:
        out["kappa_rel_err_vs_oracle"] = abs(r["kappa"] - kor) / kor
    return out


def roofline(w, tl, kernel, tsize=4):
    """HBM roofline of the pass kernel: algorithmic bytes per launch (sweeps
    in that launch x solid cells x 2 words of the compute type) over its
    average launch duration (HIP events on the library's stream); beside it
    the same launch against the vector ALU peak."""
    launches = max(tl["sweep_launches"], 1)
    sweeps_per_launch = tl["sweeps"] / launches
    avg_ms = tl["sweep_ms"] / launches
    bytes_ = sweeps_per_launch * w.n_solid * WORDS_PER_CELL_SWEEP * tsize
    achieved = bytes_ / (avg_ms * 1e-3) / 1e9 if avg_ms > 0 else 0.0
    flops = sweeps_per_launch * w.n_solid * FLOPS_PER_CELL_SWEEP[w.ndim]
    tflops = flops / (avg_ms * 1e-3) / 1e12 if avg_ms > 0 else 0.0
    alu_peak = PEAK["fp32_vector_tflops"] if tsize == 4 else PEAK["fp64_vector_tflops"]
    return {"bound": "hbm", "achieved": achieved, "peak": PEAK["hbm_gbs"], "unit": "GB/s",
            "frac": achieved / PEAK["hbm_gbs"], "traffic": None, "kernel": kernel,
            "avg_launch_ms": avg_ms, "sweeps_per_launch": sweeps_per_launch,
            "algorithmic_bytes_per_launch": bytes_,
            "alu_view": {"achieved_tflops": tflops, "peak_tflops": alu_peak, "frac": tflops / alu_peak}}


def single(P, name, steps, warmup):
    w = make_workload(name)
    solver = P.Solver.from_workload(w)
    ref = solver.solve(solver.opts(**REF), want_T_L=False)        # untimed
    kref = ref["kappa"]
    golden = None
    gpath = os.path.join(ROOT, "tests", "golden", f"{name}_oracle.json")
    if os.path.exists(gpath):
        golden = json.load(open(gpath))
    kor = golden["kappa_cc"] if golden else None
    res = {n: leg(P, solver, w, n, steps, warmup, kref, kor) for n in FORMS}
    return w, kref, kor, res


def batch(P, steps, warmup):
    """64 geometries of uneven size in one launch per pass: geometry solves/s."""
    import torch
    from inputs import gen
    geoms = gen.config3()
    solvers = [P.Solver.from_workload(w) for w in geoms]
    dof = sum(w.dof for w in geoms)
    ref, _ = P.solve_batch(solvers, P.default_opts(**REF))
    out = {"workload": "64 periodic 2D geometries (48^2..256^2, 1-4 circular pores, L 50-500 nm), "
                       "48 directions x 30 MFPs, all in one launch per pass",
           "dof": dof, "solid_cells": sum(w.n_solid for w in geoms)}
    for name in FORMS:
        o = P.default_opts(**OP[name])
        choice = P.autotune.tune(solvers, o)
        P.autotune.apply(o, choice)
        for _ in range(warmup):
            P.solve_batch(solvers, o)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(steps):
            k, st = P.solve_batch(solvers, o)
        torch.cuda.synchronize()
        dt = (time.perf_counter() - t0) / steps
        ot = P.default_opts(**OP[name], timing=1)
        P.autotune.apply(ot, choice)
        _, stt = P.solve_batch(solvers, ot)
        out[name] = {"geometry_solves_per_s": len(geoms) / dt, "ms_per_batch": 1e3 * dt,
                     "dof_per_s": dof / dt,
                     "max_kappa_rel_err_vs_fp64_ref": max(abs(x - y) / y for x, y in zip(k, ref)),
                     "launch_shape": {"waves_by_class": choice["waves_by_class"],
                                      "dispatch": choice["dispatch"]},
                     "max_passes": max(x["outer_iters"] for x in st),
                     "mean_passes": sum(x["outer_iters"] for x in st) / len(st),
                     "status_ok": sum(1 for x in st if x["status"] == 0),
                     "timed_leg": {"sweep_ms": stt[0]["sweep_ms"], "reduce_ms": stt[0]["reduce_ms"],
                                   "fourier_ms": stt[0]["fourier_ms"],
                                   "sweep_launches": stt[0]["sweep_launches"]}}
    return out


def cpu_share():
    """Host cores this process may use: the affinity set, at most 16 (the
    host-core share of one GPU on the GPU machine)."""
    aff = len(os.sched_getaffinity(0))
    return max(1, min(aff, 16)), aff, os.cpu_count()


def cpu_baseline_measure(w, seconds):
    """Time the FP64 oracle on the same workload before the GPU is touched:
    every (m, l) system factored once (SuperLU, reused as in the paper) and a
    few source-iteration passes, with the directions spread over the host
    cores (one worker process per core).  Bounded by `seconds` of passes."""
    from oracle.parallel import source_iteration_parallel
    cores, aff, ncpu = cpu_share()
    t0 = time.perf_counter()
    r = source_iteration_parallel(w, n_workers=cores, n_passes=3, time_limit=seconds)
    total = time.perf_counter() - t0
    return {"cores": cores, "affinity": aff, "cpu_count": ncpu, "t_factor": r["t_factor"],
            "pass_s": float(r["pass_times"].mean()), "passes_run": int(r["passes"]), "wall_s": total}


def cpu_baseline_value(m, passes, dof):
    per_solve = m["t_factor"] + passes * m["pass_s"]
    return {"value": 1.0 / per_solve, "unit": "solves/s", "cores": m["cores"], "kind": "oracle",
            "sample": (f"full workload, all systems factored ({m['t_factor']:.1f}s) + "
                       f"{m['passes_run']} passes ({m['pass_s']:.3f}s each) on {m['cores']} worker "
                       f"processes (affinity set {m['affinity']} cores, os.cpu_count() "
                       f"{m['cpu_count']}); extrapolated to the {passes} passes the FP64 form needs "
                       f"for the same error target (Fourier guess and setup not counted)"),
            "dof_per_s": dof / per_solve, "seconds_per_solve_estimate": per_solve,
            "cpu_count": m["cpu_count"], "affinity_cores": m["affinity"]}


def cpu_cfg1_one_core():
    """The 32x32 cell (plain method, FP64, 1e-8 relative change), the serial
    oracle on one core: one full converged solve, Fourier guess included."""
    from inputs import gen
    from oracle.bte import Problem, source_iteration
    w = gen.config1()
    t0 = time.perf_counter()
    r = source_iteration(Problem(w), tol=1e-8)
    dt = time.perf_counter() - t0
    return {"solves_per_s": 1.0 / dt, "seconds": dt, "passes": int(r["passes"]), "cores": 1,
            "kappa": r["kappa_cc"], "kind": "oracle (serial, SuperLU per system)"}


def cfg1_leg(P, steps, warmup):
    """The 32x32 cell as specified: plain Algorithm 1 in FP64 to a 1e-8
    relative change of kappa."""
    from inputs import gen
    w = gen.config1()
    s = P.Solver.from_workload(w)
    o = s.opts(precision=0, outer_tol=1e-8, stop_rule=0, accel=0, inner_tol=1e-12, fourier_tol=1e-10,
               passes_per_graph=8, max_outer=20000)
    r = run_solves(s, o, steps, warmup)
    return {"workload": "32x32 cell, centred square pore (25%), 24 directions x 10 MFPs, FP64, "
                        "Algorithm 1 to 1e-8 relative change", "dof": w.dof,
            "solves_per_s": steps / r["seconds"], "ms_per_solve": 1e3 * r["seconds"] / steps,
            "passes_per_solve": r["outer_iters"] / steps, "kappa": r["kappa"]}


def adjoint_leg(P, name, steps, warmup):
    """d kappa / d sigma by the transposed source iteration (Eq. (iter2)
    transposed): adjoint-only gradients/s after one kept forward solve, FP64
    and FP32 forms at the headline operating points, each gradient's error
    against a tight FP64 adjoint on the same inputs."""
    import numpy as np
    import torch
    w = make_workload(name)
    s = P.Solver.from_workload(w)
    ref_o = s.opts(**dict(REF, keep_state=1))
    s.solve(ref_o, sigma=w.sigma, want_T_L=False)
    gref, _ = s.adjoint(ref_o)
    gref = gref.cpu().numpy()
    out = {"workload": name, "cells": w.n_cells}
    for form in ("fp64_aa", "fp32_aa"):
        o = s.opts(**dict(OP[form], keep_state=1))
        fw = s.solve(o, sigma=w.sigma, want_T_L=False)
        for _ in range(warmup):
            s.adjoint(o)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(steps):
            g, st = s.adjoint(o)
        torch.cuda.synchronize()
        dt = (time.perf_counter() - t0) / steps
        g = g.cpu().numpy()
        out[form] = {"gradients_per_s": 1.0 / dt, "ms_per_gradient": 1e3 * dt,
                     "adjoint_passes": st["outer_iters"], "forward_passes": fw["outer_iters"],
                     "max_rel_err_vs_fp64_ref": float(np.max(np.abs(g - gref)) / np.max(np.abs(gref))),
                     "sum_rel_err_vs_fp64_ref": float(abs(g.sum() - gref.sum()) / abs(gref.sum()))}
    return out


def apply_leg(P, name="cfg5", launches=20):
    """The matrix-free upwind apply (Eq. (iter2) left-hand side) over every
    system of a workload at once: y = (sigma + Lambda_m A_l) x for all (m, l),
    x and y system-major over all cells.  HBM roofline: algorithmic bytes =
    one read of x and one write of y per solid DoF (2 x sizeof(T)); the
    arrays themselves also hold the pore cells (written 0)."""
    import torch
    w = make_workload(name)
    s = P.Solver.from_workload(w)
    ns, nc = w.n_systems, w.n_cells
    ids = torch.arange(ns, dtype=torch.int32, device=s.device)
    out = {"workload": describe(name, w), "systems": ns, "cells": nc, "solid_cells": w.n_solid}
    for prec, tag in ((1, "fp32"), (0, "fp64")):
        dt = torch.float32 if prec else torch.float64
        gen_ = torch.Generator(device=s.device).manual_seed(7)
        x = torch.randn(ns * nc, dtype=dt, device=s.device, generator=gen_)
        y = torch.empty_like(x)
        stream = torch.cuda.current_stream()
        for _ in range(3):
            P.obte.obte_upwind_apply(s.mesh, prec, 0, None, ids, x, y, stream=stream)
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record(stream)
        for _ in range(launches):
            P.obte.obte_upwind_apply(s.mesh, prec, 0, None, ids, x, y, stream=stream)
        e1.record(stream)
        torch.cuda.synchronize()
        ms = e0.elapsed_time(e1) / launches
        tsz = 4 if prec else 8
        alg = 2 * tsz * ns * w.n_solid
        arr = 2 * tsz * ns * nc
        out[tag] = {"avg_launch_ms": ms, "algorithmic_bytes_per_launch": alg,
                    "roofline": {"bound": "hbm", "achieved": alg / ms / 1e6, "peak": PEAK["hbm_gbs"],
                                 "unit": "GB/s", "frac": alg / ms / 1e6 / PEAK["hbm_gbs"]},
                    "array_bytes_GBs": arr / ms / 1e6}
        del x, y
        torch.cuda.empty_cache()
    return out


def unstructured_leg(P, steps=3):
    """Algorithm 1 on an unstructured triangle mesh (the paper meshes its
    cells with unstructured polygons): a 100 nm cell with a centred pore
    (r = 30 nm), 64 x 64 node lattice displaced by 0.3 h, two triangles per
    quadrilateral; 48 directions x 30 MFPs; FP64; the non-orthogonal
    heat-conduction first guess, then passes to a 1e-6 relative change
    (forcing term 0.3 on the periodic-face solves)."""
    import torch
    from inputs import gen
    nm = 1e-9
    w = gen.unstructured_2d(64, 64, amp=0.3, tri=True, seed=7, L=100 * nm,
                            pores=[((50 * nm, 50 * nm), 30 * nm)], n_dir=48, n_mfp=30, mfp_hi=100e-6)
    s = P.UMeshSolver.from_workload(w)
    o = s.opts(outer_tol=1e-6, max_outer=3000, inner_tol=1e-8, inner_rtol=0.3, max_inner=100, fourier_tol=1e-8)
    r = s.solve(o)                      # warm-up
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        r = s.solve(o)
    torch.cuda.synchronize()
    dt = (time.perf_counter() - t0) / steps
    t1 = time.perf_counter()
    f = s.fourier(tol=1e-8)
    torch.cuda.synchronize()
    return {"workload": f"unstructured triangles ({len(w.cells)} cells, {s.n_solid} solid, {s.n_faces} faces, "
                        f"{s.n_walls} wall faces), centred pore r=30 nm in a 100 nm cell, 48 directions x 30 MFPs, "
                        "FP64, Algorithm 1 to a 1e-6 relative change",
            "solves_per_s": 1.0 / dt, "ms_per_solve": 1e3 * dt, "passes": r["outer_iters"],
            "bicgstab_iters_per_system_pass": r["inner_iters"] / max(r["outer_iters"] * s.n_systems, 1),
            "ms_per_pass": 1e3 * dt / max(r["outer_iters"], 1), "kappa": r["kappa"], "kappa_face": r["kappa_face"],
            "kappa_fourier": r["kappa_fourier"], "status": r["status"],
            "fourier_ms": 1e3 * (time.perf_counter() - t1), "fourier_outer_iters": f["outer_iters"],
            "levels_per_direction_max": max(s.levels())}


def adjoint_3d(P):
    """One adjoint pass of the 3D membrane at sigma = 1 (FP32 form, headline
    operating point) after its kept forward solve."""
    import torch
    w = make_workload("cfg5")
    s = P.Solver.from_workload(w)
    o = s.opts(**dict(OP[HEADLINE], keep_state=1))
    fw = s.solve(o, want_T_L=False)
    s.adjoint(o)                      # warm-up (graph capture)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    g, st = s.adjoint(o)
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    return {"workload": describe("cfg5", w) + ", d kappa / d sigma at sigma = 1 (FP32 form)",
            "ms_per_gradient": 1e3 * dt, "adjoint_passes": st["outer_iters"],
            "forward_passes": fw["outer_iters"], "p_T_lambda_vs_kappa":
            abs(st["kappa"] - fw["kappa"]) / abs(fw["kappa"])}


def fourier_batch(P, steps, warmup):
    """The Fourier-only workload (only_fourier) over the 64 geometries:
    geometry solves/s of the batched FP64 CG."""
    import torch
    from inputs import gen
    geoms = gen.config3()
    solvers = [P.Solver.from_workload(w) for w in geoms]
    ref, _ = P.solve_batch(solvers, P.default_opts(only_fourier=1, fourier_tol=1e-12))
    o = P.default_opts(only_fourier=1, fourier_tol=1e-8)
    for _ in range(warmup):
        P.solve_batch(solvers, o)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        k, st = P.solve_batch(solvers, o)
    torch.cuda.synchronize()
    dt = (time.perf_counter() - t0) / steps
    return {"workload": "Fourier first guess only (FP64 CG to 1e-8) over the 64 geometries",
            "geometry_solves_per_s": len(geoms) / dt, "ms_per_batch": 1e3 * dt,
            "cells": sum(w.n_cells for w in geoms),
            "max_cg_iters": max(x["fourier_iters"] for x in st),
            "max_kappa_rel_err_vs_1e-12": max(abs(x - y) / y for x, y in zip(k, ref))}


def modes_compare(P, n_modes, steps, warmup):
    """One synthetic mode table (3D modes, in-plane part, mirrored pairs) on
    the 128x128 cell: interpolated onto the 48 x 30 grid (aMFP) against one
    system per mode (the mode-resolved iteration), both at the mixed FP32
    operating point."""
    import dataclasses
    from inputs import gen
    w = gen.with_modes(gen.config2(), n_modes, 29, dim3=True)
    out = {"workload": f"128x128 cell, {n_modes} synthetic 3D modes (in-plane part), "
                       "aMFP on 48 directions x 30 MFPs vs one system per mode",
           "n_modes": n_modes}
    for label, wk in (("amfp", w), ("mode_resolved", dataclasses.replace(w, modes_exact=True))):
        s = P.Solver.from_workload(wk)
        kref = s.solve(s.opts(**REF), want_T_L=False)["kappa"]
        r = run_solves(s, s.opts(**OP[HEADLINE]), steps, warmup)
        out[label] = {"systems": s.n_systems, "solves_per_s": steps / r["seconds"],
                      "ms_per_solve": 1e3 * r["seconds"] / steps, "kappa": r["kappa"],
                      "kappa_ref_fp64": kref, "passes_per_solve": r["outer_iters"] / steps,
                      "kappa_rel_err_vs_fp64_ref": abs(r["kappa"] - kref) / abs(kref)}
    out["speedup_amfp"] = out["mode_resolved"]["ms_per_solve"] / out["amfp"]["ms_per_solve"]
    out["kappa_amfp_vs_mode_resolved"] = (out["amfp"]["kappa_ref_fp64"] /
                                          out["mode_resolved"]["kappa_ref_fp64"])
    return out


def main():
    a = parse()
    if a.copy_probe:
        copy_probe(a.copy_probe)
        return
    if a.gpus != 1:
        print(json.dumps({"error": "this build runs on one GPU; --gpus must be 1 "
                                   "(multi-GPU sharding is design-only)"}))
        sys.exit(2)
    if a.profile and a.workload == "umesh":
        import paper_2106_02764_amd as P
        print(json.dumps({"profile": "umesh", **unstructured_leg(P, steps=a.steps)}), flush=True)
        return
    if a.workload == "umesh":
        print(json.dumps({"error": "--workload umesh runs only with --profile"}))
        sys.exit(2)
    if a.profile:
        import paper_2106_02764_amd as P
        w = make_workload(a.workload)
        s = P.Solver.from_workload(w)
        # the bench's launch shape: read from the tuner's cache when a bench
        # run wrote it (else tuned here, and those launches show up in a
        # trace too)
        choice = P.autotune.lookup(s, s.opts(**OP[HEADLINE])) or P.autotune.tune(s, s.opts(**OP[HEADLINE]))
        o = P.autotune.apply(s.opts(**OP[HEADLINE], timing=1), choice)
        r = run_solves(s, o, a.steps, 0)
        print(json.dumps({"profile": a.workload, "kernels_sha256": kernels_sha(),
                          "launch_shape": choice["waves_by_class"], "shape_from_cache": choice["from_cache"],
                          **r}), flush=True)
        return
    w0 = make_workload(a.workload)
    cpu = None if a.no_cpu else cpu_baseline_measure(w0, a.cpu_seconds)
    cpu1 = None if a.no_cpu else cpu_cfg1_one_core()
    import paper_2106_02764_amd as P

    w, kref, kor, res = single(P, a.workload, a.steps, a.warmup)
    main_r = res[HEADLINE]
    roof = roofline(w, main_r["timed_leg"], "k_sweep_pass<float>", tsize=4)
    sha = kernels_sha()
    if TRAFFIC["kernels_sha256"] == sha and a.workload == "cfg2":
        roof["traffic"] = TRAFFIC["fetch_bytes"] + TRAFFIC["write_bytes"]
        roof["traffic_fetch_bytes"] = TRAFFIC["fetch_bytes"]
        roof["traffic_write_bytes"] = TRAFFIC["write_bytes"]
    line = {
        "metric": METRIC, "value": main_r["solves_per_s"], "unit": "solves/s", "n_gpus": 1,
        "steps": a.steps, "warmup": a.warmup, "ms_per_step": main_r["ms_per_solve"],
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": describe(a.workload, w), "solid_cells": w.n_solid,
                   "systems": w.n_systems, "dof": w.dof},
        "dof_per_s": main_r["dof_per_s"],
        "kappa": main_r["kappa"], "kappa_ref_fp64": kref, "kappa_oracle": kor,
        "headline_form": HEADLINE, **res,
        "roofline": roof,
        "kernels_sha256": sha,
    }
    if cpu is not None:
        line["cpu_baseline"] = cpu_baseline_value(cpu, int(round(res["fp64"]["passes_per_solve"])), w.dof)
        line["cpu_baseline"]["cfg1_one_core"] = cpu1
    line["extra_cfg1_fp64"] = cfg1_leg(P, max(a.steps, 3), a.warmup)
    line["extra_adjoint_cfg4"] = adjoint_leg(P, "cfg4", max(2, min(a.steps, 5)), 1)
    if not a.no_extras:
        steps_x, warm_x = max(1, min(a.steps, 2)), 1
        line["extra_adjoint_3d"] = adjoint_3d(P)
        line["extra_upwind_apply"] = apply_leg(P)
        line["extra_unstructured"] = unstructured_leg(P)
        w5, kref5, kor5, res5 = single(P, "cfg5", steps_x, warm_x)
        line["extra_3d_membrane"] = {"workload": describe("cfg5", w5), "dof": w5.dof,
                                     "kappa_ref_fp64": kref5, **res5,
                                     "roofline": roofline(w5, res5[HEADLINE]["timed_leg"],
                                                          "k_sweep_pass3<float>", tsize=4)}
        line["extra_batch_64"] = batch(P, steps_x, warm_x)
        line["extra_fourier_batch_64"] = fourier_batch(P, max(a.steps, 3), warm_x)
        line["extra_modes_128"] = modes_compare(P, 11520, steps_x, warm_x)
    print(json.dumps(line), flush=True)


if __name__ == "__main__":
    main()
