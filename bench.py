"""Benchmark: fine-step cell-updates/s of one optimisation cycle on one MI355X.

A step is one warm one-shot cycle (Alg. 3 lines 9-12): pt_parareal_forward
(modified Parareal primal pass), pt_parareal_adjoint (reversed Parareal adjoint
pass) and pt_sensitivities, one Parareal iteration, with the previous cycle's
solution as the guess. The workload is the 256 x 256 FP64 problem (512
backward-Euler steps in 32 slices, SIMP k(rho) = 1e-3 + rho^3 (1 - 1e-3),
seeded rho = 0.3 + U(-0.1, 0.1), q = 1, Jacobi-PCG to relative residual
1e-10); the guess for the timed cycles comes from one untimed cold cycle on
the same design. Work per cycle = N_e * N_t cell updates.

Prints one JSON line. `roofline` reports the lane engine (the kernel that runs
each whole pass, one launch per pass) against HBM peak: `achieved` is the
algorithmic byte model -- per node and CG iteration 12 words, plus 4 words per
node and fine step in the primal pass and 7 in the adjoint pass (FP64), with
the pass's measured CG iteration counts -- per launch over the mean launch
time; `traffic` is the launch's measured HBM bytes (rocprofv3 FETCH_SIZE and
WRITE_SIZE, calibrated on a plain copy), null when the engine sources changed
since, and `measured_hbm_frac` the bandwidth those bytes mean. `cpu_baseline`
times the FP64 oracle on a warm cycle of the same workload, in one thread and
slice-parallel over worker processes.
"""
from __future__ import annotations

import argparse
import json
import os
import subprocess
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0
WORKLOAD = "plain_fp64_256"

# HBM bytes per engine launch of this workload, from rocprofv3 FETCH_SIZE and
# WRITE_SIZE runs (each scaled by what the counter reads for a 1 GiB device
# copy: x2.0 and x1.0), averaged over the forward and adjoint launches of a warm
# cycle; valid only for the engine sources with this hash (see profiles/).
TRAFFIC = {"sources_sha1": "ff262c266d1ecd0336206d5fd24022c2291b10a2",
           "bytes_per_launch": 0.5 * (13.81e9 + 18.41e9)}


def traffic_per_launch():
    """Measured HBM bytes of one engine launch, or None once the engine sources
    differ from those the counters were taken on."""
    return TRAFFIC["bytes_per_launch"] if sources_sha1() == TRAFFIC["sources_sha1"] else None


# The sources k_engine is built from: its kernel, its layouts and the host
# planner that shapes its launch. The coarse-mesh and filter kernels are not
# among them.
ENGINE_SOURCES = ("pt_engine.hip", "pt_resident.hip", "pt_gmg.hip", "pt_cm_lane.hip", "pt_internal.h", "pt_host.hip",
                  "pt_plan.h")


def sources_sha1() -> str:
    import hashlib
    h = hashlib.sha1()
    for f in ENGINE_SOURCES:
        with open(os.path.join(ROOT, "paper_2411_19030_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-precision-compare", action="store_true",
                    help="skip the FP32+refine vs FP64 comparison at equal objective accuracy")
    ap.add_argument("--no-plt", action="store_true",
                    help="skip the PLT (Sec. 7), cheaper-coarse-propagator and sequential-method "
                         "cycles on the workload")
    ap.add_argument("--no-batch", action="store_true",
                    help="skip the 64-design batch (batched FP32+refine vs plain FP64)")
    ap.add_argument("--workload", default=WORKLOAD,
                    choices=[WORKLOAD, "batch_fp32_64", "large_2048", "large_law_512",
                             "paper_100", "one_shot_chain", "plt_fp64_256", "cmesh_fp64_256",
                             "diff_fp64_512"],
                    help="the headline workload (default), or one of the other workloads "
                         "measured on its own")
    ap.add_argument("--cpu-sample-only", type=int, default=0, metavar="WORKERS",
                    help=argparse.SUPPRESS)
    ap.add_argument("--copy-calibration", action="store_true",
                    help="run only a plain device copy of 1 GiB (counter calibration)")
    ap.add_argument("--lane-trace", action="store_true",
                    help="with the headline workload or cmesh_fp64_256: print the lane trace "
                         "of a warm cycle per pass (rounds, CG iterations and times per lane "
                         "kind; per-round phase times on the headline) instead of the bench line")
    ap.add_argument("--autotune", action="store_true",
                    help="with --workload batch_fp32_64: run pt_autotune_batched on the batch "
                         "(FP32+refine) and print the shape it picks")
    return ap.parse_args()


def copy_calibration():
    """A plain device-to-device copy of exactly 1 GiB, three times: the HBM
    byte counters of this kernel calibrate FETCH_SIZE / WRITE_SIZE."""
    import torch
    n = (1 << 30) // 8
    a = torch.ones(n, dtype=torch.float64, device="cuda:0")
    b = torch.empty_like(a)
    for _ in range(3):
        b.copy_(a)
    torch.cuda.synchronize()
    print(json.dumps({"copy_bytes_read": n * 8, "copy_bytes_written": n * 8, "repeats": 3}))


def _cpu_model() -> str:
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def _oracle_problem(w):
    import oracle as O
    return O.Problem(nx=w["nx"], ny=w["ny"], n_steps=w["n_steps"], n_slices=w["n_slices"],
                     p=w["p"], k0=w["k0"], kmin=w["kmin"], pk=w["pk"], c0=w["c0"],
                     cmin=w["cmin"], pc=w["pc"], q=w["q"], t_final=w["t_final"], bc=w["bc"])


# slice-parallel oracle workers (fork start): the discretisation with its
# factors, and the forward's S and Theta for the adjoint, are inherited
_POOL_STATE = {}


def _f_pri_task(item):
    import oracle as O
    n, T, th = item
    return O.F_pri(_POOL_STATE["d"], T, th, n)


def _f_adj_task(item):
    import oracle as O
    n, lam, g = item
    return O.F_adj(_POOL_STATE["d"], _POOL_STATE["S"], _POOL_STATE["Theta"], lam, g, n)


def cpu_sample(workers: int) -> dict:
    """The FP64 oracle on the benchmark workload, the GPU's unit of work: one
    warm one-iteration cycle (forward + adjoint + sensitivities) restarting
    from the oracle's own cold cycle (untimed).
    workers == 1: every step in this process (mode i, sequential).
    workers > 1: the paper's structure (Sec. 4.3, Sec. 5.2): a pool of worker
    processes runs the fine propagators of all slices, this process the
    coarse sweeps (mode ii, slice-parallel). Factorisations happen before
    the timed cycle in both modes (they belong to the design, not the cycle)."""
    import multiprocessing as mp

    import numpy as np

    import oracle as O
    from workloads import workload, workload_density
    w = workload(WORKLOAD)
    P = _oracle_problem(w)
    d = O.Discretisation(P, workload_density(WORKLOAD))
    d._factor(P.dt)
    d._factor(P.dtau)
    cold_f = O.parareal_forward(d, 1)
    cold_a = O.parareal_adjoint(d, cold_f["S"], cold_f["Theta"], 1)
    gT, gth, gl = cold_f["uT"], cold_f["utheta"], cold_a["lam"]
    del cold_f, cold_a
    _POOL_STATE["d"] = d
    ctx = mp.get_context("fork")
    t0 = time.perf_counter()
    if workers <= 1:
        fw = O.parareal_forward(d, 1, gT, gth)
        ad = O.parareal_adjoint(d, fw["S"], fw["Theta"], 1, gl)
    else:
        with ctx.Pool(workers) as pool:
            fw = O.parareal_forward(d, 1, gT, gth,
                                    fmap=lambda items: pool.map(_f_pri_task, items))
        _POOL_STATE["S"], _POOL_STATE["Theta"] = fw["S"], fw["Theta"]
        with ctx.Pool(workers) as pool:
            ad = O.parareal_adjoint(d, fw["S"], fw["Theta"], 1, gl,
                                    fmap=lambda items: pool.map(_f_adj_task, items))
    t = time.perf_counter() - t0
    cells = w["nx"] * w["ny"] * w["n_steps"]
    return dict(seconds=t, cells=cells, workers=workers, Theta=fw["Theta"],
                grad_norm=float(np.linalg.norm(ad["grad"])))


def cpu_baseline() -> dict:
    """Oracle cell-updates/s on this host: mode (i) one thread, and mode (ii)
    min(N_tau, 16, cores) worker processes, each a fresh child with BLAS
    pinned to one thread per process."""
    from workloads import workload
    env = dict(os.environ)
    for k in ("OMP_NUM_THREADS", "OPENBLAS_NUM_THREADS", "MKL_NUM_THREADS"):
        env[k] = "1"
    cores = os.cpu_count() or 1
    pool = max(1, min(workload(WORKLOAD)["n_slices"], 16, cores))

    def child(workers):
        out = subprocess.run([sys.executable, os.path.abspath(__file__), "--cpu-sample-only",
                              str(workers)], capture_output=True, text=True, env=env,
                             timeout=900)
        if out.returncode != 0:
            raise RuntimeError(out.stderr[-2000:])
        return json.loads(out.stdout.strip().splitlines()[-1])

    seq = child(1)
    par = child(pool)
    host = f"{_cpu_model()}, {cores} logical CPUs"
    return {"value": seq["cells"] / seq["seconds"], "unit": "cell-updates/s", "cores": 1,
            "kind": "oracle",
            "sample": (f"one warm one-iteration cycle (forward + adjoint + sensitivities) of the "
                       f"{WORKLOAD} workload by the FP64 oracle (sparse LU per step) in one "
                       f"thread, restarting from the oracle's cold cycle: {seq['seconds']:.1f} s "
                       f"for {seq['cells']} cell updates; host {host}"),
            "host": host,
            "slice_parallel": {"value": par["cells"] / par["seconds"], "cores": pool,
                               "seconds": par["seconds"],
                               "sample": (f"the same warm cycle with the fine propagators of "
                                          f"all slices on {pool} worker processes and the "
                                          f"coarse sweeps in the master (the paper's "
                                          f"structure)")}}


def precision_compare(prob, rho, gT, gth, gl, accuracy=1e-6, repeats=3) -> dict:
    """FP32 inner CG with FP64 refinement against plain FP64 at equal objective
    accuracy. For each precision the loosest CG tolerance of a fixed ladder whose
    warm-cycle Theta stays within `accuracy` (relative) of a FP64 cycle solved to
    rtol 1e-13 is chosen, then that cycle is timed (median of `repeats`). The
    FP64 rtol-1e-13 path matches the oracle to 1e-10 in the parity tests."""
    import dataclasses

    import torch

    from paper_2411_19030_amd.cycle import Cycle
    stream = torch.cuda.current_stream()

    def cycle_for(precision, rtol):
        return Cycle(dataclasses.replace(prob, precision=precision, cg_rtol=rtol), rho.device)

    def timed(cyc):
        ts = []
        for _ in range(repeats):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record(stream)
            cyc.run(rho, gT, gth, gl)
            e1.record(stream)
            torch.cuda.synchronize()
            ts.append(e0.elapsed_time(e1))
        return sorted(ts)[len(ts) // 2]

    ref = cycle_for(0, 1e-13)
    ref.run(rho, gT, gth, gl)
    torch.cuda.synchronize()
    th_ref = float(ref.Theta)
    g_ref = ref.grad.clone()
    out = {"accuracy": accuracy, "reference": "fp64 warm cycle at cg_rtol 1e-13"}
    for name, prec in (("fp64", 0), ("fp32_refine", 1)):
        best = None
        for rtol in (1e-5, 1e-6, 1e-7, 1e-8, 1e-9):
            cyc = cycle_for(prec, rtol)
            cyc.run(rho, gT, gth, gl)
            torch.cuda.synchronize()
            err = abs(float(cyc.Theta) - th_ref) / abs(th_ref)
            if err <= accuracy:
                gerr = float(torch.linalg.norm(cyc.grad - g_ref) / torch.linalg.norm(g_ref))
                best = {"cg_rtol": rtol, "ms_per_cycle": timed(cyc), "Theta_rel_err": err,
                        "grad_rel_err": gerr, "status": cyc.status()["status"]}
                break
        out[name] = best
    if out["fp64"] and out["fp32_refine"]:
        out["speedup_fp32_refine_over_fp64"] = (out["fp64"]["ms_per_cycle"]
                                                / out["fp32_refine"]["ms_per_cycle"])
    return out


def plt_compare(prob, rho, parareal_ms, parareal_theta, repeats=5,
                precisions=(("fp64", 0, None), ("fp32_refine", 1, 1e-7))) -> dict:
    """Zero coarse propagators (the PLT form of Sec. 7) on the same workload.

    Each PLT cycle carries information one slice further, so the PLT cycles
    first run N_tau times on the fixed design, each restarting from the last.
    The guesses are then the converged states, the steady state of a one-shot
    run. The warm cycles from those guesses are timed (median of `repeats`):
    FP64 at the workload's CG tolerance, and FP32 with FP64 refinement at
    1e-7 (objective within 1e-6 of FP64). The converged Theta is the
    sequential method's Theta to the CG tolerance, so it also measures the
    objective error of the one-iteration Parareal estimate."""
    import dataclasses

    import torch

    from paper_2411_19030_amd.cycle import Cycle
    stream = torch.cuda.current_stream()
    Nn, Nt = prob.n_nodes, prob.n_steps
    out = {"guess": f"converged ({prob.n_slices} PLT cycles on the design)"}
    th_ref = None
    for name, prec, rtol in precisions:
        rtol = prob.cg_rtol if rtol is None else rtol
        cyc = Cycle(dataclasses.replace(prob, propagator=1, precision=prec, cg_rtol=rtol),
                    rho.device)
        cyc.run(rho)
        for _ in range(prob.n_slices):
            cyc.run(rho, cyc.uT.clone(), None, cyc.lam.clone())
        torch.cuda.synchronize()
        gT, gl = cyc.uT.clone(), cyc.lam.clone()
        ts, tf = [], []
        for _ in range(repeats):
            ev = [torch.cuda.Event(enable_timing=True) for _ in range(3)]
            ev[0].record(stream)
            cyc.forward(rho, gT)
            ev[1].record(stream)
            st_f = cyc.status()
            ev2 = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            ev2[0].record(stream)
            cyc.adjoint(rho, gl)
            cyc.sensitivities(rho)
            ev2[1].record(stream)
            torch.cuda.synchronize()
            tf.append((ev[0].elapsed_time(ev[1]), ev2[0].elapsed_time(ev2[1])))
            ts.append(tf[-1][0] + tf[-1][1])
        st = cyc.status()
        k = sorted(range(repeats), key=lambda i: ts[i])[repeats // 2]
        t_fwd, t_adj = tf[k]
        it_f = st_f["cg_iters_fine"]
        it_a = st["cg_iters_fine"]   # counters restart with each pass
        w = 8.0
        bytes_f = w * Nn * (12 * it_f + 4 * Nt)
        bytes_a = w * Nn * (12 * it_a + 7 * Nt)
        ach = (bytes_f + bytes_a) / ((t_fwd + t_adj) * 1e-3) / 1e9
        th = float(cyc.Theta)
        th_ref = th if th_ref is None else th_ref
        out[name] = {"cg_rtol": rtol, "ms_per_cycle": ts[k],
                     "phase_ms": {"forward": t_fwd, "adjoint+sens": t_adj},
                     "cell_updates_per_s": prob.n_elem * Nt / (ts[k] * 1e-3),
                     "speedup_over_parareal_fp64": (parareal_ms / ts[k]
                                                    if parareal_ms is not None else None),
                     "Theta": th, "Theta_rel_err_vs_fp64": abs(th - th_ref) / th_ref,
                     "status": st["status"],
                     "roofline_fp64_bytes": {"achieved": ach, "frac": ach / HBM_PEAK_GBS}}
        if name == "fp64" and parareal_theta is not None:
            out["parareal_one_shot_Theta_rel_err"] = abs(parareal_theta - th) / th
        del cyc
    return out


def coarse_compare(prob, rho, ref_ms, ref_theta, ref_grad, nus=(10, 20), repeats=3) -> dict:
    """A cheaper coarse propagator on the same workload and protocol: every
    coarse step is exactly nu Jacobi-PCG iterations from its input state
    (coarse_iters = nu) instead of a solve to cg_rtol. The cold cycle gives the
    guesses, then warm cycles are timed (median of `repeats`). Theta and the
    gradient are compared with the exact-G one-shot cycle of the headline."""
    import dataclasses

    import torch

    from paper_2411_19030_amd.cycle import Cycle
    stream = torch.cuda.current_stream()
    out = {}
    for nu in nus:
        cyc = Cycle(dataclasses.replace(prob, coarse_iters=nu), rho.device)
        cyc.run(rho)
        torch.cuda.synchronize()
        g = (cyc.uT.clone(), cyc.utheta.clone(), cyc.lam.clone())
        ts = []
        for _ in range(repeats):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record(stream)
            cyc.run(rho, *g)
            e1.record(stream)
            torch.cuda.synchronize()
            ts.append(e0.elapsed_time(e1))
        ms = sorted(ts)[len(ts) // 2]
        th = float(cyc.Theta)
        out[f"nu_{nu}"] = {
            "ms_per_cycle": ms, "speedup_over_exact_G": ref_ms / ms,
            "Theta_rel_diff_vs_exact_G": abs(th - ref_theta) / ref_theta,
            "grad_rel_diff_vs_exact_G": float(torch.linalg.norm(cyc.grad - ref_grad) /
                                              torch.linalg.norm(ref_grad)),
            "status": cyc.status()["status"]}
        del cyc
    return out


def coarse_mesh_compare(prob, rho, ref_ms=None, ref_theta=None, ref_grad=None,
                        repeats=3) -> dict:
    """The coarse propagators on the nx/2 x ny/2 mesh (propagator
    PT_COARSE_MESH, Sec. 7.3) on the same workload and protocol as the
    headline: the cold cycle gives the guesses, warm cycles are timed (median
    of `repeats`), and Theta and the gradient are compared with the exact-G
    one-shot cycle when it is given."""
    import dataclasses

    import torch

    from paper_2411_19030_amd._pt import PT_COARSE_MESH
    from paper_2411_19030_amd.cycle import Cycle
    stream = torch.cuda.current_stream()
    cyc = Cycle(dataclasses.replace(prob, propagator=PT_COARSE_MESH), rho.device)
    cyc.run(rho)
    torch.cuda.synchronize()
    g = (cyc.uT.clone(), cyc.utheta.clone(), cyc.lam.clone())
    ts = []
    for _ in range(repeats):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record(stream)
        cyc.run(rho, *g)
        e1.record(stream)
        torch.cuda.synchronize()
        ts.append(e0.elapsed_time(e1))
    ms = sorted(ts)[len(ts) // 2]
    th = float(cyc.Theta)
    st = cyc.status()
    out = {"ms_per_cycle": ms, "Theta": th,
           "adjoint_coarse_cg_iterations": st["cg_iters_coarse"],
           "adjoint_coarse_solves": st["solves_coarse"], "status": st["status"]}
    if ref_ms is not None:
        out.update({"speedup_over_exact_G": ref_ms / ms,
                    "Theta_rel_diff_vs_exact_G": abs(th - ref_theta) / ref_theta,
                    "grad_rel_diff_vs_exact_G": float(torch.linalg.norm(cyc.grad - ref_grad) /
                                                      torch.linalg.norm(ref_grad))})
    del cyc
    return out


def sequential_reference(prob, rho, repeats=3) -> dict:
    """The reference method of Sec. 5.2 on the GPU: one slice (N_tau = 1), where
    one iteration is the sequential time stepping exactly (every step is a
    fine step from the previous state). The paper measures both one-shot
    methods as speedups over this reference."""
    import dataclasses

    import torch

    from paper_2411_19030_amd.cycle import Cycle
    stream = torch.cuda.current_stream()
    cyc = Cycle(dataclasses.replace(prob, n_slices=1), rho.device)
    cyc.run(rho)
    torch.cuda.synchronize()
    # with a guess no cold coarse lane runs beside the single fine lane; with
    # one slice the guess does not enter the result
    g = (cyc.uT.clone(), cyc.utheta.clone(), cyc.lam.clone())
    ts = []
    for _ in range(repeats):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record(stream)
        cyc.run(rho, *g)
        e1.record(stream)
        torch.cuda.synchronize()
        ts.append(e0.elapsed_time(e1))
    ms = sorted(ts)[len(ts) // 2]
    return {"ms_per_cycle": ms, "Theta": float(cyc.Theta), "status": cyc.status()["status"]}


def centre_trace(base, rho, Ntau=10) -> dict:
    """The temperature at the domain centre over t (Fig. 3, Sec. 4.3): the
    sequential method (one slice), and one cold Parareal iteration with N_tau
    slices as vanilla Parareal returns it (the corrected coarse points u_n only)
    and as the modified Parareal does (every fine state: the corrected coarse
    points and, between them, the fine propagators' states F(u^0)). Errors are
    against the sequential temperatures; the modified form's coarse points are
    the vanilla ones (the same corrected states)."""
    import dataclasses

    import numpy as np

    from paper_2411_19030_amd.cycle import Cycle
    dev = rho.device
    W = base.nx + 1
    node = (base.ny // 2) * W + base.nx // 2
    Nt = base.n_steps
    M = Nt // Ntau
    seq = Cycle(dataclasses.replace(base, n_slices=1, iterations=1), dev)
    seq.forward(rho)
    par = Cycle(dataclasses.replace(base, n_slices=Ntau, iterations=1), dev)
    par.forward(rho)
    ts = np.concatenate([[0.0], seq.S[:, node].cpu().numpy()])
    tm = np.concatenate([[0.0], par.S[:, node].cpu().numpy()])
    tv = par.uT[:, node].cpu().numpy()
    coarse = np.arange(Ntau + 1) * M
    fine = np.setdiff1d(np.arange(Nt + 1), coarse)
    peak = float(np.max(np.abs(ts)))
    st = [seq.status()["status"], par.status()["status"]]
    del seq, par
    r6 = lambda a: [float(f"{x:.6g}") for x in a]
    return {"figure": "Fig. 3 (Sec. 4.3)", "node": [base.nx // 2, base.ny // 2],
            "n_slices": Ntau, "iterations": 1, "guess": "cold (coarse sweep)",
            "t_sequential_and_modified": r6(np.arange(Nt + 1) / Nt),
            "t_vanilla": r6(coarse / Nt),
            "sequential": r6(ts), "modified": r6(tm), "vanilla": r6(tv),
            "max_err_vanilla_coarse_points": float(np.max(np.abs(tv - ts[coarse]))) / peak,
            "max_err_modified_intermediate_points": float(np.max(np.abs(tm[fine] - ts[fine])))
            / peak,
            "errors_relative_to": "max |T_seq| at the node",
            "vanilla_equals_modified_at_coarse_points": bool(np.array_equal(tv, tm[coarse])),
            "status": st}


def paper_sweep(slices=(5, 10, 20, 30), max_iters=8, repeats=1) -> dict:
    """The paper's preliminary experiment (Sec. 5.2-5.3) on its test case: for
    N_tau in {5, 10, 20, 30} and 1..8 Parareal iterations, cold guesses from the
    coarse propagators, the objective error |Theta_par - Theta_seq| / Theta_seq
    and the sensitivity error ||grad_par - grad_seq||_2 / ||grad_seq||_2 against
    the sequential method (one slice), and the speedup of the cycle over it.
    The same rows with zero coarse propagators (Sec. 7, guesses u^0 = 0) follow.
    All solves to relative residual 1e-12 in FP64."""
    import dataclasses

    import torch

    from paper_2411_19030_amd import Problem
    from paper_2411_19030_amd.cycle import Cycle
    from workloads import workload, workload_density
    w = workload("paper_100")
    base = Problem(nx=w["nx"], ny=w["ny"], n_steps=w["n_steps"], n_slices=1, pnorm=w["p"],
                   k0=w["k0"], kmin=w["kmin"], pk=w["pk"], c0=w["c0"], cmin=w["cmin"],
                   pc=w["pc"], q=w["q"], t_final=w["t_final"], bc=w["bc"], iterations=1,
                   cg_rtol=w["rtol"], max_iter=50000)
    dev = torch.device("cuda:0")
    rho = torch.tensor(workload_density("paper_100"), dtype=torch.float64, device=dev)
    stream = torch.cuda.current_stream()

    def timed(cyc, guess=()):
        cyc.run(rho, *guess)
        torch.cuda.synchronize()
        ts = []
        for _ in range(repeats):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record(stream)
            cyc.run(rho, *guess)
            e1.record(stream)
            torch.cuda.synchronize()
            ts.append(e0.elapsed_time(e1))
        return sorted(ts)[len(ts) // 2]

    seq = Cycle(base, dev)
    seq.run(rho)
    torch.cuda.synchronize()
    g = (seq.uT.clone(), seq.utheta.clone(), seq.lam.clone())
    t_seq = timed(seq, g)
    th_seq = float(seq.Theta)
    gr_seq = seq.grad.clone()
    out = {"workload": "paper_100", "design": "seeded branched conductor (density_branches)",
           "cg_rtol": base.cg_rtol, "sequential": {"ms_per_cycle": t_seq, "Theta": th_seq},
           "columns": ["propagator", "n_slices", "iterations", "objective_error",
                       "sensitivity_error", "ms_per_cycle", "speedup", "status"],
           "rows": []}
    del seq
    out["fig3_centre_trace"] = centre_trace(base, rho)
    for prop in (0, 1):
        for Ntau in slices:
            for it in range(1, max_iters + 1):
                if prop == 1 and it > Ntau:
                    break   # exact from N_tau iterations on
                cyc = Cycle(dataclasses.replace(base, n_slices=Ntau, iterations=it,
                                                propagator=prop), dev)
                ms = timed(cyc)
                e_obj = abs(float(cyc.Theta) - th_seq) / th_seq
                e_sen = float(torch.linalg.norm(cyc.grad - gr_seq) / torch.linalg.norm(gr_seq))
                out["rows"].append(["parareal" if prop == 0 else "plt", Ntau, it, e_obj, e_sen,
                                    ms, t_seq / ms, cyc.status()["status"]])
                print("paper_100", out["rows"][-1], file=sys.stderr, flush=True)
                del cyc
    return out


def one_shot_chain(n_cycles=30, Ntau=30) -> dict:
    """Alg. 3 over a seeded design schedule on the paper's test case.

    The designs chi_i come from `design_schedule`. It starts from the branched
    design and takes smooth seeded steps that shrink by 0.9 per cycle; this
    stands in for the optimiser's iterates, so all methods see the same designs.
    Each passes the filter and projection of Sec. 6.1 (r = 0.03, beta = 32,
    eta = 0.5). Per cycle the sequential method (one slice) gives Theta and
    dTheta/dchi. One-shot Parareal and one-shot PLT (N_tau slices, one
    iteration) restart from their own previous cycle; their first cycle is
    exact (N_tau iterations), as Alg. 3 starts with a sequential cycle. One-shot
    Parareal with the cheaper coarse propagators (coarse steps of 60 CG
    iterations; coarse steps on the 50 x 50 mesh) runs beside them.
    Reported per cycle: the objective and sensitivity errors of both one-shot
    estimates and the cycle times (forward, backward and the filter)."""
    import dataclasses

    import numpy as np
    import torch

    from paper_2411_19030_amd import Problem
    from paper_2411_19030_amd.autograd import OneShotParareal
    from paper_2411_19030_amd.cycle import Cycle
    from paper_2411_19030_amd.design import DesignFilter
    from workloads import density_branches, design_schedule, workload
    w = workload("paper_100")
    nx, ny = w["nx"], w["ny"]
    base = Problem(nx=nx, ny=ny, n_steps=w["n_steps"], n_slices=Ntau, pnorm=w["p"], k0=w["k0"],
                   kmin=w["kmin"], pk=w["pk"], c0=w["c0"], cmin=w["cmin"], pc=w["pc"], q=w["q"],
                   t_final=w["t_final"], bc=w["bc"], iterations=1, cg_rtol=w["rtol"],
                   max_iter=50000)
    dev = torch.device("cuda:0")
    flt = DesignFilter(nx, ny, 0.03, 32.0, 0.5)
    designs = design_schedule(nx, ny, 6, n_cycles, start=density_branches(nx, ny, w["seed"]))
    seq = OneShotParareal(dataclasses.replace(base, n_slices=1), dev, warm=False)
    methods = {"parareal": OneShotParareal(base, dev, warm=True),
               "parareal_coarse60": OneShotParareal(dataclasses.replace(base, coarse_iters=60),
                                                    dev, warm=True),
               "parareal_coarse_mesh": OneShotParareal(dataclasses.replace(base, propagator=2),
                                                       dev, warm=True),
               "plt": OneShotParareal(dataclasses.replace(base, propagator=1), dev, warm=True)}
    stream = torch.cuda.current_stream()

    def run(obj, chi):
        x = torch.tensor(chi, device=dev, requires_grad=True)
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record(stream)
        th = obj(flt(x))
        th.backward()
        e1.record(stream)
        torch.cuda.synchronize()
        return float(th), x.grad.clone(), e0.elapsed_time(e1)

    rows = []
    for i, chi in enumerate(designs):
        th_s, g_s, t_s = run(seq, chi)
        row = {"cycle": i, "Theta_seq": th_s, "ms_seq": t_s}
        for name, obj in methods.items():
            if i == 0:
                # the exact first cycle: N_tau iterations, its outputs are the guesses
                ex = Cycle(dataclasses.replace(obj.prob, iterations=Ntau), dev)
                rho = flt(torch.tensor(chi, device=dev))
                ex.run(rho)
                obj.guess_T, obj.guess_theta = ex.uT.clone(), ex.utheta.clone()
                obj.guess_lambda = ex.lam.clone()
                torch.cuda.synchronize()
                del ex
                continue
            th, g, t = run(obj, chi)
            row[name] = {"objective_error": abs(th - th_s) / th_s,
                         "sensitivity_error": float(torch.linalg.norm(g - g_s) /
                                                    torch.linalg.norm(g_s)),
                         "ms": t, "speedup": t_s / t}
        rows.append(row)
        print("one_shot_chain", json.dumps(row), file=sys.stderr, flush=True)
    summary = {}
    for name in methods:
        r = [x[name] for x in rows[1:]]
        summary[name] = {
            "max_objective_error": max(x["objective_error"] for x in r),
            "max_sensitivity_error": max(x["sensitivity_error"] for x in r),
            "median_sensitivity_error": float(np.median([x["sensitivity_error"] for x in r])),
            "mean_speedup": float(np.mean([x["speedup"] for x in r]))}
    return {"workload": "paper_100", "n_slices": Ntau, "cycles": n_cycles,
            "filter": {"r_fil": 0.03, "beta": 32.0, "eta": 0.5},
            "schedule": "design_schedule(seed 6) from density_branches, step 0.08, decay 0.9",
            "summary": summary, "rows": rows}


# Worker shape of the 64-design batch: None, the built-in plan (groups of a size for
# each class of designs, resident lanes). The best shape of one kind of groups for all
# designs that pt_autotune_batched found (4 fine and 8 sweep workgroups, 8 sweep groups,
# streaming) takes 3.77 s per warm cycle, the built-in plan 1.65.
BATCH_TUNING = None


def batch_autotune(rtol=1e-7) -> dict:
    """pt_autotune_batched on the 64-design batch (FP32+refine): the shape it
    picks, its warm-cycle time and the built-in shape's, and oracle-free checks
    that the tuned shape ran cleanly."""
    import torch

    from paper_2411_19030_amd import Problem
    from paper_2411_19030_amd.batched import BatchedCycle
    from workloads import batch_designs

    dev = torch.device("cuda:0")
    ds = batch_designs()
    rhos = [torch.tensor(d["rho"], device=dev) for d in ds]
    probs = [Problem(nx=d["nx"], ny=d["ny"], n_steps=d["n_steps"], n_slices=d["n_slices"],
                     pnorm=8, cg_rtol=rtol, max_iter=20000, precision=1) for d in ds]
    cyc = BatchedCycle(probs, dev)
    t0 = time.perf_counter()
    best, ms, ms0 = cyc.autotune(rhos, progress=lambda shape, v: print(
        "autotune", shape, f"{v:.1f} ms", file=sys.stderr, flush=True))
    return {"workload": "batch_fp32_64", "tuned": best, "tuned_ms": ms, "default_ms": ms0,
            "tuner_s": time.perf_counter() - t0}


def batch_compare(rtol=1e-7, ref_rtol=1e-12, accuracy=1e-6, replays=5) -> dict:
    """The 64-design workload (sides 64..512, 16..64 slices of 16 steps, seeded
    densities): one cycle of every design. Forms, each timed on a warm cycle
    after a cold one:
    * batched FP32 + FP64 refinement in the built-in shape: all designs in one
      launch per pass; timed eagerly and as the replay of the warm cycle
      captured in a HIP graph (median of `replays`; each replay is the next
      warm cycle, from the guesses the previous one saved);
    * plain FP64: one design after another through the single-design calls;
    * reference: batched FP64 at cg_rtol 1e-12 (the accuracy yardstick).
    The objective accuracy of a form is max over designs of |Theta - Theta_ref| /
    Theta_ref on the (first, eager) warm cycle."""
    import torch

    from paper_2411_19030_amd import Problem
    from paper_2411_19030_amd.batched import BatchedCycle
    from paper_2411_19030_amd.cycle import Cycle
    from workloads import batch_designs

    dev = torch.device("cuda:0")
    ds = batch_designs()
    rhos = [torch.tensor(d["rho"], device=dev) for d in ds]
    cells = sum(d["nx"] * d["ny"] * d["n_steps"] for d in ds)

    def probs(prec, tol):
        return [Problem(nx=d["nx"], ny=d["ny"], n_steps=d["n_steps"], n_slices=d["n_slices"],
                        pnorm=8, cg_rtol=tol, max_iter=20000, precision=prec) for d in ds]

    def timed(fn):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        fn()
        torch.cuda.synchronize()
        return time.perf_counter() - t0

    def batched(prec, tol, tuning, graph=False):
        cyc = BatchedCycle(probs(prec, tol), dev)
        cyc.tuning = tuning
        cyc.run(rhos, warm=False)
        t = timed(lambda: cyc.run(rhos, warm=True))
        th = cyc.Theta.cpu().numpy().copy()
        st = [s_["status"] for s_ in cyc.status()]
        tg = None
        if graph:
            s = torch.cuda.Stream()
            g = torch.cuda.CUDAGraph()
            torch.cuda.synchronize()
            with torch.cuda.graph(g, stream=s):
                cyc.run(rhos, warm=True)
            g.replay()
            torch.cuda.synchronize()
            ts = sorted(timed(g.replay) for _ in range(replays))
            tg = ts[len(ts) // 2]
            st += [s_["status"] for s_ in cyc.status()]
            del g
        del cyc
        torch.cuda.empty_cache()
        return t, th, st, tg

    t_ref, th_ref, st_ref, _ = batched(0, ref_rtol, BATCH_TUNING)
    print(f"batch: fp64 reference {t_ref:.2f} s", file=sys.stderr, flush=True)
    t32, th32, st32, t32g = batched(1, rtol, BATCH_TUNING, graph=True)
    print(f"batch: fp32+refine {t32:.2f} s, graph replay {t32g:.2f} s", file=sys.stderr,
          flush=True)
    th64 = []
    t64 = 0.0
    st64 = []
    for k, d in enumerate(ds):
        cyc = Cycle(probs(0, rtol)[k], dev)
        cyc.run(rhos[k])
        gT, gth, gl = cyc.uT.clone(), cyc.utheta.clone(), cyc.lam.clone()
        t64 += timed(lambda: cyc.run(rhos[k], gT, gth, gl))
        th64.append(float(cyc.Theta))
        st64.append(cyc.status()["status"])
        del cyc
        if k % 16 == 15:
            print(f"batch: plain fp64 designs 1..{k + 1}", file=sys.stderr, flush=True)
    import numpy as np
    th64 = np.array(th64)
    err32 = float(np.max(np.abs(th32 - th_ref) / th_ref))
    err64 = float(np.max(np.abs(th64 - th_ref) / th_ref))
    return {
        "workload": "batch_fp32_64",
        "designs": len(ds),
        "cells_per_cycle": cells,
        "accuracy_target": accuracy,
        "fp32_refine_batched": {"cg_rtol": rtol, "s_per_cycle": t32,
                                "cell_updates_per_s": cells / t32, "max_Theta_rel_err": err32,
                                "tuning": BATCH_TUNING,
                                "tuning_source": "built-in (pt_batch_default_tuning)",
                                "graph_replay_s_per_cycle": t32g,
                                "graph_replay_cell_updates_per_s": cells / t32g,
                                "status_ok": all(v == 0 for v in st32)},
        "fp64_plain_per_design": {"cg_rtol": rtol, "s_per_cycle": t64,
                                  "cell_updates_per_s": cells / t64, "max_Theta_rel_err": err64,
                                  "status_ok": all(v == 0 for v in st64)},
        "reference": {"form": "fp64 batched", "cg_rtol": ref_rtol, "s_per_cycle": t_ref,
                      "status_ok": all(v == 0 for v in st_ref)},
        "speedup_batched_fp32_refine_over_plain_fp64": t64 / t32,
        "speedup_graph_replay_over_plain_fp64": t64 / t32g,
        "both_meet_accuracy": err32 <= accuracy and err64 <= accuracy,
    }


def lane_trace(prob, rho, timers: bool) -> list:
    """Lane trace of a warm cycle (guesses from the cold cycle), one record per
    pass: per lane kind the lanes, group rounds, CG iterations, summed lane
    time and time per round, with `timers` the per-round phase times (work,
    barrier, partial sums) and the flag waits; the sweep's start and step
    times; every fine lane's start and end. Times in microseconds from the
    first lane's start (the 100 MHz device clock)."""
    import dataclasses

    import numpy as np
    import torch

    from paper_2411_19030_amd._pt import pt_query_trace
    from paper_2411_19030_amd.cycle import Cycle
    if timers:
        prob = dataclasses.replace(prob, tuning=dict(phase_timers=1))
    cyc = Cycle(prob, rho.device)
    cyc.run(rho)
    torch.cuda.synchronize()
    g = (cyc.uT.clone(), cyc.utheta.clone(), cyc.lam.clone())
    cyc.run(rho, *g)
    torch.cuda.synchronize()
    out = []
    for name, fn in (("forward", lambda: cyc.forward(rho, g[0], g[1])),
                     ("adjoint", lambda: cyc.adjoint(rho, g[2]))):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        fn()
        e1.record()
        torch.cuda.synchronize()
        tr = pt_query_trace(prob, cyc.ws)
        kinds = {}
        for r in tr:
            k = kinds.setdefault(r["kind"], dict(lanes=0, nwg=[], rounds=0, iters=0,
                                                 lane_us=0.0, work=0.0, barrier=0.0,
                                                 partial_sums=0.0, flag_wait_us=0.0,
                                                 last_end_us=0.0))
            end = r["step_end_us"][-1] if r["step_end_us"] else r["start_us"]
            k["lanes"] += 1
            if r["nwg"] not in k["nwg"]:
                k["nwg"] = sorted(k["nwg"] + [r["nwg"]])
            k["rounds"] += r["rounds"]
            k["iters"] += r["iters"]
            k["lane_us"] += end - r["start_us"]
            k["work"] += r["work_us"]
            k["barrier"] += r["barrier_us"]
            k["partial_sums"] += r["reduce_us"]
            k["flag_wait_us"] += r["flag_us"]
            k["last_end_us"] = max(k["last_end_us"], end)
        for k in kinds.values():
            n = max(k["rounds"], 1)
            k["us_per_round"] = round(k["lane_us"] / n, 2)
            if timers:
                k["per_round_us"] = {q: round(k[q] / n, 2) for q in ("work", "barrier",
                                                                      "partial_sums")}
            for q in ("work", "barrier", "partial_sums"):
                del k[q]
            if not timers:
                del k["flag_wait_us"]
            for q in ("lane_us", "last_end_us", "flag_wait_us"):
                if q in k:
                    k[q] = round(k[q])
        rec = {"pass": name, "launch_ms": round(e0.elapsed_time(e1), 2), "kinds": kinds}
        sw = [r for r in tr if "SWEEP" in r["kind"]]
        if sw:
            st = np.diff([sw[0]["start_us"]] + sw[0]["step_end_us"])
            rec["sweep_start_us"] = round(sw[0]["start_us"])
            rec["sweep_step_us"] = [round(float(x)) for x in st]
        rec["fine_lanes_us"] = {str(r["slice"]): [round(r["start_us"]),
                                                  round(r["step_end_us"][-1])]
                                for r in sorted(tr, key=lambda r: r["start_us"])
                                if r["kind"] in ("F_PRI", "F_ADJ") and r["step_end_us"]}
        out.append(rec)
    return out


def plain_run(name: str, steps: int, warmup: int) -> dict:
    """A store-all FP64 Jacobi workload other than the headline (diff_fp64_512:
    512 x 512, 1024 steps in 64 slices): one cold cycle,
    `warmup` untimed and `steps` timed warm cycles from its guesses, each timed
    with HIP events on the stream (forward, then adjoint + sensitivities)."""
    import torch

    from paper_2411_19030_amd import Problem
    from paper_2411_19030_amd.cycle import Cycle
    from workloads import workload, workload_density

    w = workload(name)
    dev = torch.device("cuda:0")
    prob = Problem(nx=w["nx"], ny=w["ny"], n_steps=w["n_steps"], n_slices=w["n_slices"],
                   pnorm=w["p"], cg_rtol=w["rtol"], max_iter=20000)
    cyc = Cycle(prob, dev)
    rho = torch.tensor(workload_density(name), dtype=torch.float64, device=dev)
    cyc.run(rho)
    torch.cuda.synchronize()
    gT, gth, gl = cyc.uT.clone(), cyc.utheta.clone(), cyc.lam.clone()
    stream = torch.cuda.current_stream()
    times = []
    for i in range(warmup + steps):
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(3)]
        ev[0].record(stream)
        cyc.forward(rho, gT, gth)
        ev[1].record(stream)
        cyc.adjoint(rho, gl)
        cyc.sensitivities(rho)
        ev[2].record(stream)
        torch.cuda.synchronize()
        if i >= warmup:
            times.append((ev[0].elapsed_time(ev[1]), ev[1].elapsed_time(ev[2])))
    st = cyc.status()
    cells = prob.n_elem * prob.n_steps
    ms = sum(a + b for a, b in times) / len(times)
    return {"metric": "fine-step cell-updates/s (fwd+adjoint+sens per cycle)",
            "value": cells / (ms * 1e-3), "unit": "cell-updates/s", "n_gpus": 1,
            "steps": steps, "warmup": warmup, "ms_per_step": ms, "higher_is_better": True,
            "dtype": "f64", "data": "synthetic",
            "config": {"workload": name, "nx": prob.nx, "ny": prob.ny, "n_steps": prob.n_steps,
                       "n_slices": prob.n_slices, "cg_rtol": prob.cg_rtol},
            "phase_ms": {"forward": sum(a for a, _ in times) / len(times),
                         "adjoint_and_sensitivities": sum(b for _, b in times) / len(times)},
            "status": st["status"], "cg_iterations": st["cg_iters_fine"] + st["cg_iters_coarse"],
            "Theta": float(cyc.Theta)}


def large_run(name: str, steps: int) -> dict:
    """The large single design (2048 x 2048, 2048 steps in 128 slices, Gaussian-bump
    density; the same law at 512 x 512 with 512 steps in 32 slices): geometric
    multigrid PCG, FP32 inner CG with FP64 refinement, checkpointed storage. One
    cold cycle, then `steps` timed warm cycles (forward + adjoint + sensitivities)."""
    import torch

    from paper_2411_19030_amd import Problem
    from paper_2411_19030_amd.cycle import Cycle
    from workloads import workload, workload_density

    w = workload(name)
    dev = torch.device("cuda:0")
    prob = Problem(nx=w["nx"], ny=w["ny"], n_steps=w["n_steps"], n_slices=w["n_slices"],
                   pnorm=w["p"], cg_rtol=w["rtol"], max_iter=20000, precond=1, precision=1,
                   storage=1)
    cyc = Cycle(prob, dev)
    rho = torch.tensor(workload_density(name), dtype=torch.float64, device=dev)
    cyc.run(rho)
    torch.cuda.synchronize()
    st_cold = cyc.status()
    print(f"{name}: cold cycle done", file=sys.stderr, flush=True)
    gT, gth, gl = cyc.uT.clone(), cyc.utheta.clone(), cyc.lam.clone()
    stream = torch.cuda.current_stream()
    times = []
    for _ in range(steps):
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(3)]
        ev[0].record(stream)
        cyc.forward(rho, gT, gth)
        ev[1].record(stream)
        cyc.adjoint(rho, gl)
        cyc.sensitivities(rho)
        ev[2].record(stream)
        torch.cuda.synchronize()
        times.append((ev[0].elapsed_time(ev[1]), ev[1].elapsed_time(ev[2])))
        print(f"{name}: warm cycle {sum(times[-1]):.0f} ms", file=sys.stderr, flush=True)
    st = cyc.status()
    cells = prob.n_elem * prob.n_steps
    ms = sum(a + b for a, b in times) / len(times)
    return {"metric": "fine-step cell-updates/s (fwd+adjoint+sens per cycle)",
            "value": cells / (ms * 1e-3), "unit": "cell-updates/s", "n_gpus": 1,
            "steps": steps, "ms_per_step": ms, "higher_is_better": True, "dtype": "f32+f64",
            "data": "synthetic",
            "config": {"workload": name, "nx": prob.nx, "ny": prob.ny, "n_steps": prob.n_steps,
                       "n_slices": prob.n_slices, "cg_rtol": prob.cg_rtol,
                       "precision": "fp32_refine", "preconditioner": "gmg",
                       "storage": "checkpoint"},
            "phase_ms": {"forward": sum(a for a, _ in times) / len(times),
                         "adjoint_and_sensitivities": sum(b for _, b in times) / len(times)},
            "cold_status": st_cold["status"], "status": st["status"],
            "Theta": float(cyc.Theta),
            "workspace_gb": cyc.ws.numel() / 1e9, "state_gb": cyc.S.numel() * 8 / 1e9}


def main():
    args = parse()
    if args.cpu_sample_only:
        print(json.dumps(cpu_sample(args.cpu_sample_only)))
        return
    if args.copy_calibration:
        copy_calibration()
        return
    if args.gpus != 1:
        print(f"bench.py runs on one GPU; --gpus {args.gpus} is not supported (the passes "
              "would shard by time slices across GPUs, with the sequential sweeps handed on "
              "from GPU to GPU)",
              file=sys.stderr)
        sys.exit(2)
    if args.lane_trace and args.workload not in (WORKLOAD, "cmesh_fp64_256"):
        print(f"bench.py: --lane-trace takes the headline workload or cmesh_fp64_256, "
              f"not {args.workload}", file=sys.stderr)
        sys.exit(2)
    import torch

    from paper_2411_19030_amd import Problem, load_library
    from paper_2411_19030_amd.cycle import Cycle
    from workloads import workload, workload_density

    load_library()
    if args.lane_trace:
        w = workload(WORKLOAD)
        cm = args.workload == "cmesh_fp64_256"
        prob = Problem(nx=w["nx"], ny=w["ny"], n_steps=w["n_steps"], n_slices=w["n_slices"],
                       pnorm=w["p"], k0=w["k0"], kmin=w["kmin"], pk=w["pk"], c0=w["c0"],
                       cmin=w["cmin"], pc=w["pc"], q=w["q"], t_final=w["t_final"], bc=w["bc"],
                       iterations=1, cg_rtol=w["rtol"], max_iter=20000,
                       propagator=2 if cm else 0)
        rho = torch.tensor(workload_density(WORKLOAD), dtype=torch.float64,
                           device=torch.device("cuda:0"))
        # per-round phase times exist in FP64 launches without coarse-mesh lanes
        for rec in lane_trace(prob, rho, timers=not cm):
            print(json.dumps(rec), flush=True)
        return
    if args.workload == "diff_fp64_512":
        print(json.dumps(plain_run(args.workload, max(1, min(args.steps, 5)),
                                   max(0, min(args.warmup, 2)))))
        return
    if args.workload in ("large_2048", "large_law_512"):
        print(json.dumps(large_run(args.workload, max(1, min(args.steps, 3)))))
        return
    if args.workload == "batch_fp32_64":
        print(json.dumps(batch_autotune() if args.autotune else batch_compare()))
        return
    if args.workload == "paper_100":
        print(json.dumps(paper_sweep()))
        return
    if args.workload == "one_shot_chain":
        print(json.dumps(one_shot_chain()))
        return
    if args.workload == "plt_fp64_256":
        # the PLT cycle of the headline workload on its own (FP64, converged
        # guesses), e.g. for profiling the streaming engine
        w = workload(WORKLOAD)
        prob = Problem(nx=w["nx"], ny=w["ny"], n_steps=w["n_steps"], n_slices=w["n_slices"],
                       pnorm=w["p"], k0=w["k0"], kmin=w["kmin"], pk=w["pk"], c0=w["c0"],
                       cmin=w["cmin"], pc=w["pc"], q=w["q"], t_final=w["t_final"], bc=w["bc"],
                       iterations=1, cg_rtol=w["rtol"], max_iter=20000)
        rho = torch.tensor(workload_density(WORKLOAD), dtype=torch.float64,
                           device=torch.device("cuda:0"))
        print(json.dumps(plt_compare(prob, rho, None, None,
                                     precisions=(("fp64", 0, prob.cg_rtol),),
                                     repeats=max(1, args.steps))))
        return
    if args.workload == "cmesh_fp64_256":
        # the coarse-spatial-mesh cycle of the headline workload on its own
        # (FP64, guesses from its cold cycle), e.g. for profiling its kernels
        w = workload(WORKLOAD)
        prob = Problem(nx=w["nx"], ny=w["ny"], n_steps=w["n_steps"], n_slices=w["n_slices"],
                       pnorm=w["p"], k0=w["k0"], kmin=w["kmin"], pk=w["pk"], c0=w["c0"],
                       cmin=w["cmin"], pc=w["pc"], q=w["q"], t_final=w["t_final"], bc=w["bc"],
                       iterations=1, cg_rtol=w["rtol"], max_iter=20000)
        rho = torch.tensor(workload_density(WORKLOAD), dtype=torch.float64,
                           device=torch.device("cuda:0"))
        print(json.dumps({"workload": "cmesh_fp64_256",
                          **coarse_mesh_compare(prob, rho, repeats=max(1, args.steps))}))
        return
    w = workload(WORKLOAD)
    prob = Problem(nx=w["nx"], ny=w["ny"], n_steps=w["n_steps"], n_slices=w["n_slices"],
                   pnorm=w["p"], k0=w["k0"], kmin=w["kmin"], pk=w["pk"], c0=w["c0"],
                   cmin=w["cmin"], pc=w["pc"], q=w["q"], t_final=w["t_final"], bc=w["bc"],
                   iterations=1, cg_rtol=w["rtol"], max_iter=20000)
    dev = torch.device("cuda:0")
    cyc = Cycle(prob, dev)
    rho = torch.tensor(workload_density(WORKLOAD), dtype=torch.float64, device=dev)
    # cold cycle: the guess of the timed warm cycles
    cyc.run(rho)
    torch.cuda.synchronize()
    gT, gth, gl = cyc.uT.clone(), cyc.utheta.clone(), cyc.lam.clone()
    stream = torch.cuda.current_stream()

    def step(events=None):
        if events:
            events[0].record(stream)
        cyc.forward(rho, gT, gth)
        if events:
            events[1].record(stream)
        cyc.adjoint(rho, gl)
        if events:
            events[2].record(stream)
        cyc.sensitivities(rho)
        if events:
            events[3].record(stream)

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    # per-pass CG iteration counts (identical every cycle: same design and guess)
    cyc.forward(rho, gT, gth)
    st_f = cyc.status()
    cyc.adjoint(rho, gl)
    st_a = cyc.status()
    cyc.sensitivities(rho)
    torch.cuda.synchronize()

    evs = [[torch.cuda.Event(enable_timing=True) for _ in range(4)] for _ in range(args.steps)]
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for k in range(args.steps):
        step(evs[k])
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    t_fwd = sum(e[0].elapsed_time(e[1]) for e in evs) / args.steps
    t_adj = sum(e[1].elapsed_time(e[2]) for e in evs) / args.steps
    t_sen = sum(e[2].elapsed_time(e[3]) for e in evs) / args.steps
    ms = wall * 1e3 / args.steps
    st = cyc.status()

    Nn, Ne, Nt = prob.n_nodes, prob.n_elem, prob.n_steps
    cells = Ne * Nt
    it_f = st_f["cg_iters_fine"] + st_f["cg_iters_coarse"]
    it_a = st_a["cg_iters_fine"] + st_a["cg_iters_coarse"]
    bytes_f = 8.0 * Nn * (12 * it_f + 4 * Nt)
    bytes_a = 8.0 * Nn * (12 * it_a + 7 * Nt)
    # one engine launch per pass: per launch, the mean of the two
    alg_per_launch = 0.5 * (bytes_f + bytes_a)
    launch_s = 0.5 * (t_fwd + t_adj) * 1e-3
    achieved = alg_per_launch / launch_s / 1e9
    traffic = traffic_per_launch()
    out = {
        "metric": "fine-step cell-updates/s (fwd+adjoint+sens per cycle), % HBM peak, vs FP64",
        "value": cells / (ms * 1e-3),
        "unit": "cell-updates/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64",
        "data": "synthetic",
        "config": {"workload": WORKLOAD, "nx": prob.nx, "ny": prob.ny, "n_steps": Nt,
                   "n_slices": prob.n_slices, "pnorm": prob.pnorm, "cg_rtol": prob.cg_rtol,
                   "parareal_iterations": 1, "guess": "previous (cold) cycle",
                   "precision": "fp64", "preconditioner": "jacobi"},
        "roofline": {"bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBS,
                     "unit": "GB/s", "frac": achieved / HBM_PEAK_GBS, "traffic": traffic,
                     "per": "engine launch (one per pass; mean of the forward and adjoint)",
                     "algorithmic_bytes_per_launch": alg_per_launch,
                     "launch_ms": launch_s * 1e3,
                     "measured_hbm_GBps": (traffic / launch_s / 1e9 if traffic else None),
                     "measured_hbm_frac": (traffic / launch_s / 1e9 / HBM_PEAK_GBS
                                           if traffic else None)},
        "pct_hbm_peak": 100.0 * achieved / HBM_PEAK_GBS,
        "phase_ms": {"forward": t_fwd, "adjoint": t_adj, "sensitivities": t_sen},
        "cg_iterations": {"forward": it_f, "adjoint": it_a},
        "status": st["status"],
        "Theta": float(cyc.Theta),
    }
    if not args.no_precision_compare:
        out["vs_fp64"] = precision_compare(prob, rho, gT, gth, gl)
    if not args.no_plt:
        out["coarse_truncated"] = coarse_compare(prob, rho, ms, float(cyc.Theta), cyc.grad.clone())
        out["coarse_mesh"] = coarse_mesh_compare(prob, rho, ms, float(cyc.Theta),
                                                 cyc.grad.clone())
        out["plt"] = plt_compare(prob, rho, ms, float(cyc.Theta))
        seq = sequential_reference(prob, rho)
        seq["speedup_parareal_fp64"] = seq["ms_per_cycle"] / ms
        seq["speedup_coarse_mesh_fp64"] = seq["ms_per_cycle"] / out["coarse_mesh"]["ms_per_cycle"]
        seq["speedup_plt_fp64"] = seq["ms_per_cycle"] / out["plt"]["fp64"]["ms_per_cycle"]
        out["sequential_reference"] = seq
    if not args.no_batch:
        del cyc
        torch.cuda.empty_cache()
        out["batch"] = batch_compare()
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline()
    print(json.dumps(out))


def release_gpu():
    """Drops this process's device memory and events before the interpreter
    exits: main's tensors and events are gone once it returns; torch's cached
    blocks go back to the runtime here, so nothing of this program is left
    for the runtime's (or a profiler's) teardown to release."""
    import gc
    gc.collect()
    if "torch" in sys.modules:
        import torch
        if torch.cuda.is_initialized():
            torch.cuda.synchronize()
            torch.cuda.empty_cache()


if __name__ == "__main__":
    main()
    release_gpu()
