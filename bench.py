"""Benchmark: Newton-CG voxel-iterations/s of the Fourier-Galerkin solve at 128^3, FP64.

One step = one full fft_homog_solve of the 3D finite-strain workload (compressible
Neo-Hookean, 128^3 two-phase Gaussian-random-field cell, mu 1 vs 20, lam = 2 mu,
F-bar = diag(1.05, 1, 1) in 10 load increments, Newton and CG tolerance 1e-10),
starting from the undeformed state.  value = N * (CG iterations of all timed
steps) / wall time of the timed steps, inputs resident in HBM.

Prints one JSON line (rank 0, one GPU) with a ``roofline`` entry for the
dominant kernel of the CG iteration (algorithmic bytes / average launch time,
HIP events on the library's stream) and a ``cpu_baseline`` entry (the CPU
oracle timed on a bounded sample of CG iterations of the same workload).

``--workload uq256`` / ``tangents32`` instead time homogenized tangents/s of many
small-strain cells (256 cells of edge 32..96, or 1024 cells of 32^3) through
multi-cell handles; one step = the 6x6 tangents of every cell, phase maps
resident in HBM.  Their ``roofline`` is the whole job's effective bandwidth
(algorithmic bytes of all CG iterations / wall time).
"""

import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0
KERNELS = ["x_op", "reduce_pq", "y_fwd", "outer_fwd", "y_inv", "outer_inv", "reduce_rr"]


CG_KERNEL_SOURCES = ["common.h", "dual.h", "fft_lds.h", "kernels.h", "kernels.hip", "kernels_fixed.hip",
                     "launch_geometry.cpp", "materials.h", "pass_kernels.h", "xpass_law.h", "xpass_nh.hip"]


def kernel_source_hash():
    """sha256 of the sources of the CG-iteration kernels (device code and the headers it includes)
    and of the flags they are compiled with; HBM counter records are valid only for the kernels
    they were taken on."""
    import hashlib

    from paper_2408_03804_amd import build as _build

    h = hashlib.sha256()
    for f in CG_KERNEL_SOURCES:
        h.update(open(os.path.join(ROOT, "paper_2408_03804_amd", "csrc", f), "rb").read())
    flags = [f for f in _build.FLAGS + _build.PER_FILE.get("kernels.hip", []) if os.sep not in f]
    h.update(" ".join(flags).encode())
    return h.hexdigest()


def counted_traffic(kernel):
    """Per-launch HBM bytes of `kernel` from the committed rocprofv3 counter record, or None if stale."""
    path = os.path.join(ROOT, "profiles", "traffic_nh3d_grf_128.json")
    if not os.path.exists(path):
        return None
    rec = json.load(open(path))
    if rec.get("source_hash") != kernel_source_hash() or kernel not in rec.get("kernels", {}):
        return None
    k = rec["kernels"][kernel]
    return int(k["read_bytes"] + k["write_bytes"])


def log(msg):
    sys.stderr.write("[bench] %s\n" % msg)
    sys.stderr.flush()


def algorithmic_bytes_per_voxel(c, N, Nh, material_reads_strain=True, rows=False):
    """HBM bytes per voxel each kernel of an iteration of the 3D CG on displacements must move (FP64).

    The x pass reads and writes the half spectrum of c components and reads the
    linearisation point F and the phase id; the y passes read and write the half
    spectrum once; the forward outer pass reads it and reads and writes r (three
    complex components per wavevector), the inverse one reads r, p, x and writes p, x
    and the half spectrum.  rows: the finite-strain passes run row by row, and between
    the y passes the spectrum has two instead of three components per row of F.
    """
    f = 8.0 * c               # one packed field
    s = 16.0 * c * Nh / N     # one half spectrum (nx/2+1 bins per row), per voxel
    u = 16.0 * 3 * Nh / N     # one displacement vector
    inner = s * 2.0 / 3.0 if rows else s
    return {"x_op": 2 * s + (f if material_reads_strain else 0.0) + 1.0, "reduce_pq": 0.0, "y_fwd": s + inner,
            "outer_fwd": inner + 2 * u, "y_inv": inner + s, "outer_inv": inner + 5 * u, "reduce_rr": 0.0}


# the survey's byte model of one CG iteration (c = 9, finite strain): 8 CG-vector fields, the
# linearisation point and 4 half-spectrum transfers in a two-stage 3D FFT
def survey_model_bytes_per_voxel(c, N, Nh):
    return 8 * 8.0 * c + 8.0 * c + 4 * 16.0 * c * Nh / N


def host_cores():
    """Cores this process may run on (the box's share, not os.cpu_count())."""
    return len(os.sched_getaffinity(0))


def cpu_oracle_sample(w, iters_all, iters_one):
    """Time CG iterations of the CPU oracle on the first load increment of the workload: on all
    the host cores this process may use (the FFTs multi-threaded; the oracle's element-wise NumPy
    work stays on one thread), and on one thread."""
    from threadpoolctl import threadpool_limits

    from oracle import newton_cg, spectral

    shape = w["shape"]
    tab = np.asarray(w["table"])
    lam, mu = tab[w["phase"], 0], tab[w["phase"], 1]
    prob = newton_cg.Problem(shape, w["material"], lam, mu)
    d = len(shape)
    Fbar = w["macro"].reshape(d, d)
    F1 = np.eye(d) + (Fbar - np.eye(d)) / w["n_increments"]
    field = prob.uniform(F1)
    b = prob.rhs(field)
    N = prob.N
    out = {}
    for cores, iters in ((host_cores(), iters_all), (1, iters_one)):
        spectral.FFT_WORKERS = cores
        with threadpool_limits(limits=cores):
            t0 = time.perf_counter()
            _, k, st = newton_cg.conjugate_gradient(lambda v: prob.operator(field, v), b, 0.0, iters)
            t1 = time.perf_counter()
        out[cores] = (N * k / (t1 - t0), k, t1 - t0)
    spectral.FFT_WORKERS = 1
    allc = host_cores()
    v, k, t = out[allc]
    v1, k1, t1 = out[1]
    return {"value": v, "unit": "voxel-iter/s", "cores": allc, "kind": "oracle",
            "sample": "%d CG iterations (operator G*(K:p) + textbook CG update) of the CPU oracle on the first "
                      "load increment of the same %s workload, FFTs on %d threads (the host cores this process "
                      "may use), %.1f s" % (k, w["name"], allc, t),
            "single_thread": {"value": v1, "cores": 1,
                              "sample": "%d CG iterations, one thread, %.1f s" % (k1, t1)}}


def cpu_tangent_sample(cells, budget_s):
    """Tangents/s of the CPU oracle (implicit tangent at the reference state) on the first cells, one thread."""
    from threadpoolctl import threadpool_limits

    from oracle import newton_cg

    done, t = 0, 0.0
    with threadpool_limits(limits=1):
        for cell in cells:
            tab = np.asarray(cell["table"])
            prob = newton_cg.Problem(cell["shape"], "linear_elastic", tab[cell["phase"], 0], tab[cell["phase"], 1])
            t0 = time.perf_counter()
            newton_cg.homogenized_tangent(prob, newton_cg.initial_state(prob), tol_cg=1e-10)
            t += time.perf_counter() - t0
            done += 1
            if t >= budget_s:
                break
    return {"value": done / t, "unit": "tangents/s", "cores": 1, "kind": "oracle",
            "sample": "implicit 6x6 tangent (6 textbook CG solves, tol 1e-10) of the first %d cell(s) of "
                      "shape %s of the same workload, single thread, %.1f s" % (done, cells[0]["shape"], t)}


def bench_cells(args, name, cells, description):
    """Homogenized tangents/s of many linear elastic cells through multi-cell handles."""
    import torch

    from paper_2408_03804_amd.batch import TangentBatcher

    dev = [dict(phase=torch.as_tensor(c["phase"]).to("cuda:0"), table=c["table"]) for c in cells]
    b = TangentBatcher(tol_cg=1e-10, max_cg=20000, graph=not args.no_graph, autotune=not args.no_autotune,
                       max_bytes=int(args.max_gb * (1 << 30)), device="cuda:0", concurrent=args.concurrent)
    for i in range(args.warmup):
        C, info = b.tangents(dev)
        log("warmup %d: %s" % (i, ", ".join("%s x%d cg %d %.3fs" % (r["shape"][0], r["cells"], r["cg_total"],
                                                                   r["seconds"]) for r in info)))
    for key, shp in b.shapes.items():
        log("launch shape %s: %s" % (key, shp))
    torch.cuda.synchronize()
    # monotonic-clock bounds of the timed region (the clock of rocprofv3's kernel timestamps), so that
    # a kernel trace of this run can be cut to it
    mono0 = time.monotonic_ns()
    t0 = time.perf_counter()
    vox_iters = 0
    cg = 0
    cg_group = {}
    for i in range(args.steps):
        C, info = b.tangents(dev)
        for r in info:
            if r["status"] != "ok":
                raise RuntimeError("tangent solve failed: %s" % r)
            vox_iters += int(np.prod(r["shape"])) * r["cg_total"]
            cg += r["cg_total"]
            cg_group[str(r["shape"])] = cg_group.get(str(r["shape"]), 0) + r["cg_total"]
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    log("timed window monotonic ns %d %d" % (mono0, time.monotonic_ns()))
    # whole-job effective bandwidth: algorithmic bytes of every CG iteration run / wall time
    groups = {}
    for r in info:
        groups.setdefault(r["shape"], []).append(r)
    alg = 0.0
    for shape, rs in groups.items():
        n = shape[0]
        N = n ** 3
        Nh = (n // 2 + 1) * n * n
        bpv = sum(algorithmic_bytes_per_voxel(6, N, Nh, False).values())
        alg += bpv * N * sum(r["cg_total"] for r in rs)
    alg *= args.steps
    eff = alg / wall / 1e9
    cpu = None
    if not args.no_cpu:
        small = sorted(cells, key=lambda c: c["phase"].size)
        cpu = cpu_tangent_sample(small, args.cpu_seconds)
        log("cpu oracle: %.3e tangents/s" % cpu["value"])
    out = {
        "metric": "homogenized 6x6 tangents/s (FP64 Fourier-Galerkin CG, %s)" % name,
        "value": len(cells) * args.steps / wall,
        "unit": "tangents/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": wall / args.steps * 1e3,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f64", "data": "synthetic",
        "config": {"workload": description, "cells": len(cells),
                   "groups": {str(k): sum(r["cells"] for r in v) for k, v in groups.items()},
                   "graph": not args.no_graph, "autotune": not args.no_autotune, "concurrent": args.concurrent,
                   "launch_shapes": {str(k): v for k, v in b.shapes.items()},
                   "cg_iterations_per_step": cg // args.steps,
                   "cg_iterations_per_step_by_group": {k: v // args.steps for k, v in cg_group.items()},
                   "voxel_iters_per_s": vox_iters / wall},
        "roofline": {"bound": "hbm", "kernel": "whole tangent job (all CG passes, effective)",
                     "achieved": round(eff, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": round(eff / HBM_PEAK_GBS, 4), "traffic": None},
        "cpu_baseline": cpu,
    }
    b.close()
    print(json.dumps(out), flush=True)


def surrogate_flops_per_cell(n=32, channels=(1, 32, 64, 128, 256), hidden=256, n_feat=1, n_out=21):
    """Multiply-add flops (2 per product) of one forward pass of one member: the conv blocks as the
    GEMMs [outputs x 27 Ci] . [27 Ci x Co] and the two dense layers."""
    f, e = 0, n
    for l in range(1, 5):
        e //= 2
        f += 2 * e ** 3 * channels[l] * 27 * channels[l - 1]
    return f + 2 * (channels[4] + n_feat) * hidden + 2 * hidden * n_out


def cpu_surrogate_sample(sur, phase, tables, reject_frac, budget_s):
    """The with-fallback job on the CPU oracle: both members' float64 forward passes (oracle/surrogate.py)
    on the first cells until the budget, plus the oracle tangent of one cell times the rejected fraction
    (the cells the indicator sends to the solver)."""
    from threadpoolctl import threadpool_limits

    from oracle import newton_cg
    from oracle import surrogate as OS
    from paper_2408_03804_amd.surrogate import StiffnessSurrogate

    kw = dict(channels=OS.CHANNELS, hidden=256, n_feat=1, n_out=21)
    thetas = [net.get_params().cpu().numpy().astype(np.float64) for net in sur.nets]
    done, t = 0, 0.0
    while t < budget_s and done < phase.shape[0]:
        ph = phase[done:done + 4].cpu().numpy()
        ft = StiffnessSurrogate.features(tables[done:done + 4])
        t0 = time.perf_counter()
        for th in thetas:
            OS.predict(th, ph, ft, **kw)
        t += time.perf_counter() - t0
        done += ph.shape[0]
    t_sur = t / done
    ph0 = phase[0].cpu().numpy()
    tab = np.asarray(tables[0])
    prob = newton_cg.Problem(ph0.shape, "linear_elastic", tab[ph0, 0], tab[ph0, 1])
    with threadpool_limits(limits=1):
        t0 = time.perf_counter()
        newton_cg.homogenized_tangent(prob, newton_cg.initial_state(prob), tol_cg=1e-10)
        t_tan = time.perf_counter() - t0
    per_cell = t_sur + reject_frac * t_tan
    import torch
    return {"value": 1.0 / per_cell, "unit": "tangents/s", "cores": torch.get_num_threads(), "kind": "oracle",
            "sample": "float64 forward passes of the %d members on %d held-out cells (torch CPU, %d threads, "
                      "%.1f s) plus %.3f x the oracle tangent of one cell (6 textbook CG solves, one thread, "
                      "%.1f s) for the rejected fraction" % (len(thetas), done, torch.get_num_threads(), t,
                                                             reject_frac, t_tan)}


def bench_surrogate(args):
    """Stiffness surrogate against the solver on 32^3 cells: training data from the solver, training,
    held-out error, and tangents/s of both (surrogate with its indicator and solver fallback)."""
    import torch

    from paper_2408_03804_amd import workloads
    from paper_2408_03804_amd.batch import TangentBatcher
    from paper_2408_03804_amd.surrogate import StiffnessSurrogate, full6

    ntr, ncal, nte = args.train_cells, args.cal_cells, args.test_cells
    t0 = time.perf_counter()
    cells = workloads.workload_tangent_cells(ntr + ncal + nte, seed=0)
    phase = torch.stack([torch.as_tensor(c["phase"]) for c in cells]).to("cuda:0")
    tables = np.stack([c["table"] for c in cells])
    del cells
    log("%d cells generated in %.1f s" % (ntr + ncal + nte, time.perf_counter() - t0))

    # training data and held-out references from the FP64 solver
    b = TangentBatcher(tol_cg=1e-10, max_cg=20000, graph=True, autotune=True, max_bytes=int(48 << 30),
                       device="cuda:0")
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    C_all, info = b.tangents([dict(phase=phase[i], table=tables[i]) for i in range(ntr + ncal + nte)])
    torch.cuda.synchronize()
    t_data = time.perf_counter() - t0
    b.close()
    log("solver tangents of %d cells: %.1f s (%.1f tangents/s)" % (ntr + ncal + nte, t_data,
                                                                   (ntr + ncal + nte) / t_data))

    sur = StiffnessSurrogate(n=32, max_batch=max(args.batch, nte), device="cuda:0", seed=0, members=args.members)
    t0 = time.perf_counter()
    hist = sur.fit(phase[:ntr], tables[:ntr], C_all[:ntr], epochs=args.epochs, batch=args.batch, lr=args.lr,
                   log=log)
    torch.cuda.synchronize()
    t_train = time.perf_counter() - t0
    log("training: %.1f s, final losses %s" % (t_train, [h[-1] for h in hist]))

    # the indicator's spread limit from the calibration split (held out from training and from the report)
    sur.tol = args.check_tol
    cal = sur.calibrate(phase[ntr:ntr + ncal], tables[ntr:ntr + ncal], C_all[ntr:ntr + ncal], target=args.target,
                        safety=args.safety)
    log("calibration: %s" % cal)
    if args.dump:
        # per-cell indicator statistics of the calibration and test splits (analysis of the indicator)
        dump = {}
        for tag, sl in (("cal", slice(ntr, ntr + ncal)), ("test", slice(ntr + ncal, ntr + ncal + nte))):
            Cq, okq, spq = sur.predict_checked(phase[sl], tables[sl], max_spread=1e30, want_spread=True)
            Cf = full6(Cq.cpu().numpy().astype(np.float64))
            Cr = C_all[sl]
            dump[tag + "_err"] = np.linalg.norm((Cf - Cr).reshape(len(Cr), -1), axis=1) / np.linalg.norm(
                Cr.reshape(len(Cr), -1), axis=1)
            dump[tag + "_ok"] = okq.cpu().numpy()
            dump[tag + "_spread"] = spq.cpu().numpy()
            dump[tag + "_feat"] = StiffnessSurrogate.features(tables[sl])[:, 0]
            dump[tag + "_frac"] = StiffnessSurrogate.fractions(phase[sl])
        np.savez(args.dump, **dump)
    tp, tt, Ct = phase[ntr + ncal:], tables[ntr + ncal:], C_all[ntr + ncal:]
    kw = {}
    for _ in range(2):
        sur.predict_checked(tp, tt, **kw)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        C21, ok = sur.predict_checked(tp, tt, **kw)
    torch.cuda.synchronize()
    t_sur = (time.perf_counter() - t0) / args.steps
    Cp = full6(C21.cpu().numpy().astype(np.float64))
    okh = ok.cpu().numpy().astype(bool)
    err = np.linalg.norm((Cp - Ct).reshape(nte, -1), axis=1) / np.linalg.norm(Ct.reshape(nte, -1), axis=1)

    # the solver alone on the held-out cells, and on the cells the indicator rejects
    b = TangentBatcher(tol_cg=1e-10, max_cg=20000, graph=True, autotune=True, max_bytes=int(48 << 30),
                       device="cuda:0")
    test_cells = [dict(phase=tp[i], table=tt[i]) for i in range(nte)]
    b.tangents(test_cells)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        b.tangents(test_cells)
    torch.cuda.synchronize()
    t_sol = (time.perf_counter() - t0) / args.steps
    rej = [test_cells[i] for i in np.nonzero(~okh)[0]]
    t_fb = 0.0
    if rej:
        b.tangents(rej)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        b.tangents(rej)
        torch.cuda.synchronize()
        t_fb = time.perf_counter() - t0
    b.close()
    parts = sur.indicator_parts(tp, tt, **kw)
    reasons = {k: int((~v).sum()) for k, v in parts.items()}
    lc = np.abs(StiffnessSurrogate.features(tt)[:, 0])
    edges = np.percentile(lc, [0, 33.3, 66.7, 100])
    by_contrast = []
    for lo_, hi_ in zip(edges[:-1], edges[1:]):
        sel = (lc >= lo_) & (lc <= hi_)
        by_contrast.append({"abs_log_contrast": [round(float(lo_), 3), round(float(hi_), 3)],
                            "mean": float(err[sel].mean()), "p95": float(np.percentile(err[sel], 95)),
                            "rejected": int((~okh[sel]).sum()), "cells": int(sel.sum())})
    final_err = err.copy()
    final_err[~okh] = 0.0  # rejected cells are answered by the solver
    out = {
        "metric": "homogenized tangents/s, stiffness surrogate with solver fallback vs FP64 solver (32^3)",
        "value": nte / (t_sur + t_fb),
        "unit": "tangents/s",
        "n_gpus": 1, "steps": args.steps, "warmup": 2, "ms_per_step": (t_sur + t_fb) * 1e3,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "bf16", "data": "synthetic",
        "config": {"workload": "surrogate32: %d training + %d calibration + %d held-out test small-strain linear "
                               "elastic 32^3 cells (Gaussian random field l=8, top 30%% stiff, E1, E2 ~ "
                               "lognormal(0,0.5), nu=0.3); CNN 1-32-64-128-256 stride-2 3^3 conv blocks, GELU, mean "
                               "pool, MLP 257-256-21, bf16 MFMA / fp32 accumulation, Adam %d epochs batch %d, "
                               "ensemble of %d, indicator: Voigt-Reuss bounds (tol %g), central 95%% of the training "
                               "contrasts, member spread <= %.4g (calibrated: accepted calibration errors <= %g x %g)"
                               % (ntr, ncal, nte, args.epochs, args.batch, args.members, args.check_tol,
                                  sur.max_spread, args.safety, args.target),
                   "calibration": cal,
                   "solver_tangents_per_s": nte / t_sol,
                   "surrogate_only_tangents_per_s": nte / t_sur,
                   "speedup_vs_solver": t_sol / (t_sur + t_fb),
                   "rel_error_frobenius": {"mean": float(err.mean()), "median": float(np.median(err)),
                                           "p95": float(np.percentile(err, 95)), "max": float(err.max()),
                                           "frac_le_2pct": float((err <= 0.02).mean())},
                   "after_fallback": {"mean": float(final_err.mean()), "p95": float(np.percentile(final_err, 95)),
                                      "max": float(final_err.max()),
                                      "frac_le_2pct": float((final_err <= 0.02).mean())},
                   "accepted_fraction": float(okh.mean()),
                   "rejected_by_indicator": int((~okh).sum()),
                   "error_by_contrast_tercile": by_contrast,
                   "rejections_by_test": reasons,
                   "accepted_error": {"mean": float(err[okh].mean()) if okh.any() else None,
                                      "p95": float(np.percentile(err[okh], 95)) if okh.any() else None,
                                      "max": float(err[okh].max()) if okh.any() else None},
                   "training_s": t_train, "data_generation_s": t_data,
                   "final_train_loss": [h[-1] for h in hist]},
        "roofline": None,
        "cpu_baseline": None,
    }
    # the surrogate's own kernels: bf16 MFMA work of both members' forward passes over the
    # surrogate-only time (the indicator's work is negligible beside it)
    fl = surrogate_flops_per_cell() * len(sur.nets) * nte / t_sur
    out["roofline"] = {"bound": "mfma", "kernel": "surrogate inference: all layers of the %d members (effective)"
                       % len(sur.nets), "achieved": round(fl / 1e12, 2), "peak": 2500.0, "unit": "TFLOP/s",
                       "frac": round(fl / 2.5e15, 4), "traffic": None,
                       "flops_per_cell_per_member": surrogate_flops_per_cell(),
                       "note": "bf16 dense peak; the with-fallback value is dominated by the FP64 solver on the "
                               "rejected cells (solver rooflines: the nh128 and tangents32 lines)"}
    if not args.no_cpu:
        out["cpu_baseline"] = cpu_surrogate_sample(sur, tp, tt, float((~okh).mean()), args.cpu_seconds)
    sur.close()
    print(json.dumps(out), flush=True)


def bench_paper_example(args, w, k_mode, paper_seconds, paper_note):
    """One of the paper's 2D examples solved end to end: seconds per solve and voxel-iterations/s,
    beside a bounded sample of the CPU oracle on the same cell."""
    import torch

    from paper_2408_03804_amd.binding import FFTHomog

    shape = w["shape"]
    N = int(np.prod(shape))
    d = len(shape)
    h = FFTHomog(shape, w["kinematics"], w["material"], 2, device="cuda:0", tol_newton=w["tol_newton"],
                 tol_cg=w["tol_cg"], max_newton=50, max_cg=20000, k_mode=k_mode)
    h.set_material(w["phase"], w["table"])
    shape_info = h.autotune(reps=5) if args.autotune else h.launch_shape()

    def step():
        h.reset()
        S, psi, st = h.solve(w["macro"], w["n_increments"])
        if st["status"] != "ok":
            raise RuntimeError("solve failed: %s" % st["status"])
        return st

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    cg = 0
    for _ in range(args.steps):
        st = step()
        cg += st["cg_total"]
    torch.cuda.synchronize()
    wall = (time.perf_counter() - t0) / args.steps
    cpu = None
    if not args.no_cpu:
        from threadpoolctl import threadpool_limits

        from oracle import newton_cg, plasticity

        tab = np.asarray(w["table"])
        if w["material"] == "j2_plastic":
            prob = plasticity.PlasticProblem(shape, tab[w["phase"], 0], tab[w["phase"], 1], tab[w["phase"], 2],
                                             tab[w["phase"], 3])
        else:
            prob = newton_cg.Problem(shape, w["material"], tab[w["phase"], 0], tab[w["phase"], 1])
        with threadpool_limits(limits=1):
            t0 = time.perf_counter()
            ref = newton_cg.solve(prob, w["macro"], n_increments=w["n_increments"], tol_newton=w["tol_newton"],
                                  tol_cg=w["tol_cg"])
            tc = time.perf_counter() - t0
        cpu = {"value": 1.0 / tc, "unit": "solves/s", "cores": 1, "kind": "oracle",
               "sample": "the full solve of the same cell by the CPU oracle, single thread, %.1f s "
                         "(%d Newton, %d CG iterations)" % (tc, ref["stats"]["newton"], ref["stats"]["cg_total"])}
    out = {
        "metric": "seconds per solve, %s" % w["name"],
        "value": wall, "unit": "s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": wall * 1e3, "higher_is_better": False, "scaling": "weak", "vs_baseline": None,
        "dtype": "f64", "data": "synthetic",
        "config": {"workload": w["name"], "grid": list(shape), "material": w["material"],
                   "n_increments": w["n_increments"], "k_mode": "stored" if k_mode else "recompute",
                   "launch_shape": shape_info,
                   "newton_iterations": st["newton"], "cg_iterations": st["cg_total"],
                   "voxel_iters_per_s": N * cg / (wall * args.steps),
                   "paper_seconds_context": paper_seconds, "paper_context": paper_note},
        "roofline": None,
        "cpu_baseline": cpu,
    }
    print(json.dumps(out), flush=True)


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=3)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--n", type=int, default=128, help="grid points per axis")
    ap.add_argument("--timing-every", type=int, default=32,
                    help="sample every k-th CG iteration of the timed solves for the per-kernel times")
    ap.add_argument("--cpu-iters", type=int, default=7, help="CPU oracle CG iterations timed on all host cores")
    ap.add_argument("--cpu-iters-one", type=int, default=5, help="... and on one thread")
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--k-mode", type=int, default=0)
    ap.add_argument("--train-cells", type=int, default=20000)
    ap.add_argument("--test-cells", type=int, default=1024)
    ap.add_argument("--epochs", type=int, default=80)
    ap.add_argument("--batch", type=int, default=256)
    ap.add_argument("--lr", type=float, default=1e-3)
    ap.add_argument("--check-tol", type=float, default=0.02, help="surrogate: Voigt-Reuss bounds slack")
    ap.add_argument("--cal-cells", type=int, default=1024, help="surrogate: calibration cells (held out)")
    ap.add_argument("--dump", default="", help="surrogate: write per-cell indicator statistics to this .npz")
    ap.add_argument("--target", type=float, default=0.02, help="surrogate: relative tangent error target")
    ap.add_argument("--safety", type=float, default=0.8,
                    help="surrogate: accepted calibration errors must stay below safety x target")
    ap.add_argument("--members", type=int, default=2)
    ap.add_argument("--workload", default="nh128",
                    choices=["nh128", "uq256", "tangents32", "surrogate32", "e2_stvk299", "e3_j2_199"],
                    help="nh128: the Newton-CG solve (default); uq256: tangents of 256 cells of uneven size; "
                         "tangents32: tangents of 1024 cells of 32^3")
    ap.add_argument("--no-graph", action="store_true")
    ap.add_argument("--no-autotune", action="store_true", help="many-cell workloads: keep the default launch shape")
    ap.add_argument("--autotune", action="store_true", help="nh128: tune the launch shape before timing")
    ap.add_argument("--graph", action="store_true", help="nh128: replay CG chunks from a captured HIP graph")
    ap.add_argument("--max-gb", type=float, default=96.0, help="workspace budget per multi-cell handle")
    ap.add_argument("--concurrent", action="store_true", help="many-cell workloads: run the size groups concurrently")
    ap.add_argument("--cpu-seconds", type=float, default=10.0)
    ap.add_argument("--increments", type=int, default=0,
                    help="nh128: load increments per solve (0: the workload's 10); fewer only for short "
                         "counter-collection runs, never for the reported metric")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="only run a plain 512 MiB device-to-device copy 3 times (HBM counter calibration)")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py runs on exactly one GPU: this build has no multi-GPU path "
              "(--gpus %d requested)" % args.gpus, file=sys.stderr)
        sys.exit(2)

    import torch

    from paper_2408_03804_amd import workloads
    from paper_2408_03804_amd.binding import FFTHomog

    assert torch.cuda.is_available(), "bench.py needs a HIP device"
    if args.copy_calibration:
        src = torch.ones(64 << 20, dtype=torch.float64, device="cuda:0")
        dst = torch.empty_like(src)
        for _ in range(3):
            dst.copy_(src)
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(10):
            dst.copy_(src)
        e1.record()
        torch.cuda.synchronize()
        t = e0.elapsed_time(e1) / 10 * 1e-3
        print(json.dumps({"copy_bytes_read": src.numel() * 8, "copy_bytes_written": dst.numel() * 8,
                          "copy_GBs": round(2 * src.numel() * 8 / t / 1e9, 1)}))
        return
    if args.workload == "surrogate32":
        return bench_surrogate(args)
    if args.workload == "e2_stvk299":
        return bench_paper_example(args, workloads.workload_e2_stvk(), 0, 19.5,
                                   "JAX on one CPU core of an EPYC 9654, AD via jvp (the paper's section 4.1.1)")
    if args.workload == "e3_j2_199":
        return bench_paper_example(args, workloads.workload_e3_j2(), 1, 0.25,
                                   "JAX on one CPU core of an EPYC 9654, AD via linearize (the paper's section 4.1.2)")
    if args.workload == "uq256":
        cells = workloads.workload_uq_cells(256)
        log("workload generated")
        return bench_cells(args, "256 uneven cells", cells,
                           "uq256: 256 small-strain linear elastic cells, edge drawn from {32,48,64,96}, "
                           "thresholded Gaussian random fields (l ~ U[4,12], stiff fraction ~ U[0.1,0.5]), "
                           "E_matrix ~ lognormal(0,0.2), E_stiff = 10 E_matrix, nu=0.3, 6 unit loads each, CG tol 1e-10")
    if args.workload == "tangents32":
        cells = workloads.workload_tangent_cells(1024)
        log("workload generated")
        return bench_cells(args, "1024 cells of 32^3", cells,
                           "tangents32: 1024 small-strain linear elastic 32^3 cells, Gaussian random field "
                           "(l=8) top 30%% stiff, E1, E2 ~ lognormal(0,0.5), nu=0.3, 6 unit loads each, CG tol 1e-10")
    n = args.n
    w = workloads.workload_neohookean3d(n=n)
    if args.increments > 0:
        w["n_increments"] = args.increments
    shape = w["shape"]
    N = n ** 3
    c = 9
    log("workload %s generated" % w["name"])
    h = FFTHomog(shape, "finite", "neo_hookean", 2, device="cuda:0", tol_newton=1e-10, tol_cg=1e-10,
                 max_newton=50, max_cg=20000, k_mode=args.k_mode, graph=args.graph)
    h.set_material(w["phase"], w["table"])
    # work-vector placement, timed on this handle (set-up, outside the timed region): the same
    # kernels run the x pass in 180-232 us at 128^3 depending on where the work vectors sit
    stagger = h.tune_placement(reps=10)
    log("work-vector stagger: %d bytes" % stagger)
    shape_info = h.launch_shape()
    if args.autotune:
        # launch-shape tuning is set-up work, outside the timed region (at 128^3 its gain is
        # within the spread between GPUs; the default shape is the one the parity test and
        # the committed profile cover)
        shape_info = h.autotune(reps=10)
        log("launch shape: %s" % shape_info)
    ident = torch.zeros((9,) + shape, dtype=torch.float64, device="cuda:0")
    ident[0] = ident[4] = ident[8] = 1.0
    eye = np.eye(3).reshape(-1)

    def step():
        h.set_field(ident, eye)
        S, psi, st = h.solve(w["macro"], w["n_increments"])
        if st["status"] != "ok":
            raise RuntimeError("solve failed: %s" % st["status"])
        return S, psi, st

    for i in range(args.warmup):
        S, psi, st = step()
        log("warmup %d: newton %d, cg %d, %.3f s" % (i, st["newton"], st["cg_total"], st["seconds"]))
    # per-kernel device time, sampled inside the timed solves: HIP events on the library's
    # stream around the launches of every `timing_every`-th CG iteration
    h.set_kernel_timing(args.timing_every)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    total_cg = 0
    stats = []
    for i in range(args.steps):
        S, psi, st = step()
        total_cg += st["cg_total"]
        stats.append(st)
        log("step %d: newton %d, cg %d, %.3f s" % (i, st["newton"], st["cg_total"], st["seconds"]))
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    wall = t1 - t0
    value = N * total_cg / wall

    ms, samples = h.kernel_timing()
    h.set_kernel_timing(0)
    if samples == 0:
        raise RuntimeError("no CG iteration was sampled for kernel timing")
    log("kernel ms (%d sampled CG iterations): " % samples + ", ".join("%s %.4f" % (k, v) for k, v in zip(KERNELS, ms)))
    Nh = (n // 2 + 1) * n * n
    bpv = algorithmic_bytes_per_voxel(c, N, Nh, True, rows=True)
    dom = int(np.argmax(ms))
    name = KERNELS[dom]
    achieved = bpv[name] * N / (ms[dom] * 1e-3) / 1e9
    events_ms = float(np.sum(ms))
    # wall time per CG iteration of the whole timed solves (Newton-level work, host checks and
    # launch gaps included): never below the kernels' own time
    wall_ms = wall / total_cg * 1e3
    iter_bytes = sum(bpv.values()) * N
    survey_bytes = survey_model_bytes_per_voxel(c, N, Nh) * N
    roofline = {"bound": "hbm", "kernel": name, "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS,
                "unit": "GB/s", "frac": round(achieved / HBM_PEAK_GBS, 4), "traffic": counted_traffic(name),
                "kernel_ms": round(float(ms[dom]), 5),
                "timing": "HIP events on the library stream inside the timed solves, every %d-th CG "
                          "iteration (%d samples); an interval runs from the previous launch's end event to "
                          "this launch's end event" % (args.timing_every, samples),
                "algorithmic_bytes_per_launch": int(bpv[name] * N),
                "cg_iteration": {"ms_wall": round(wall_ms, 5), "ms_events": round(events_ms, 5),
                                 "algorithmic_bytes": int(iter_bytes),
                                 "achieved_GBs_wall": round(iter_bytes / (wall_ms * 1e-3) / 1e9, 1),
                                 "frac_wall": round(iter_bytes / (wall_ms * 1e-3) / 1e9 / HBM_PEAK_GBS, 4),
                                 "survey_model_bytes": int(survey_bytes),
                                 "survey_model_frac_wall": round(survey_bytes / (wall_ms * 1e-3) / 1e9 / HBM_PEAK_GBS, 4),
                                 "kernels_ms": {k: round(float(v), 5) for k, v in zip(KERNELS, ms)}}}

    cpu = None
    if not args.no_cpu:
        log("timing the CPU oracle (%d + %d CG iterations at %d^3)" % (args.cpu_iters, args.cpu_iters_one, n))
        cpu = cpu_oracle_sample(w, args.cpu_iters, args.cpu_iters_one)
        log("cpu oracle: %.3e voxel-iter/s on %d cores, %.3e on one" % (cpu["value"], cpu["cores"],
                                                                      cpu["single_thread"]["value"]))

    out = {
        "metric": "Newton-CG voxel-iters/s at 128^3 FP64",
        "value": value,
        "unit": "voxel-iter/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": wall / args.steps * 1e3,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64",
        "data": "synthetic",
        "config": {"workload": w["name"] + ": 3D finite-strain compressible Neo-Hookean, %d^3 voxels, Gaussian "
                   "random field (l=8 voxels) thresholded at 30%% stiff, mu 1 vs 20, lam=2mu, F-bar=diag(1.05,1,1) "
                   "in %d increments, Newton/CG tol 1e-10, tangent by dual-number JVP" % (n, w["n_increments"]),
                   "grid": [n, n, n], "n_increments": w["n_increments"], "k_mode": "stored" if args.k_mode else "recompute",
                   "launch_shape": shape_info, "work_vector_stagger": stagger, "graph": args.graph,
                   "cg_iterations_per_step": [s["cg_total"] for s in stats],
                   "newton_iterations_per_step": [s["newton"] for s in stats]},
        "roofline": roofline,
        "cpu_baseline": cpu,
    }
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
