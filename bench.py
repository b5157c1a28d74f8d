#!/usr/bin/env python3
"""Benchmark of the DPG multigrid hot path on one MI355X.

One step = one pass of the whole GPU path over the workload: the element DPG
stage (Gram Cholesky, B^H G^-1 B, static condensation), the multigrid
hierarchy (macro condensation, Galerkin coarse operators, vertex-patch
inverses, coarsest factorisation) and the preconditioned CG solve to the
workload's tolerance.  The mesh topology (integer numbering, maps, patch lists)
is built once per mesh by dpg_setup before the timed region, like the inputs.

Prints one JSON line.  value = n_trace * PCG iterations / seconds of the solve
phase (the metric's definition); the setup phases of every step are reported
beside it, and a mixed-precision workload is also solved in FP64 for the
time-to-tolerance comparison.  Default workload: 32^3, p = 4, mixed precision.
"""
import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0        # MI355X HBM3E
FP64_PEAK_TFLOPS = 78.6      # MI355X dense FP64 matrix (= vector) peak
FP32_PEAK_TFLOPS = 157.3
FP32_VECTOR_PEAK_TFLOPS = 78.6   # one multiply-add per lane (no packed pairs)


def make_options(D, w, torch_stream=None, device_ptrs=True, columnwise=False, recompute=False):
    return D.dpg_default_options(
        nu_pre=w.nu_pre, nu_post=w.nu_post, theta=w.theta,
        precision=D.DPG_MIXED if w.precision == "mixed" else D.DPG_FP64,
        flags=(D.DPG_DEVICE_PTRS if device_ptrs else 0) | (D.DPG_COLUMNWISE if columnwise else 0)
        | (D.DPG_RECOMPUTE_PATCHES if recompute else 0),
        stream=torch_stream)


def loads_of(w):
    if w.sources is not None:
        return [dict(dir=(0.0, 0.0, 1.0), amp=0.0,
                     sources=[[*c, w.sigma, 1.0, 0.0]]) for c in w.sources]
    return [dict(dir=w.direction, amp=1.0)]


# Classes timed around exactly one kernel symbol; the composite dense classes
# (potrf, trsm, gemm) each cover several kernels and are reported separately.
SINGLE_KERNEL = ("apply64", "apply32", "applyb64", "applyb32", "applyg64", "applyg32", "gram",
                 "bmat", "load", "macro_asm", "patch_gather")
DENSE = ("potrf", "trsm", "gemm")
# the kernels of the dense routines, each launch timed alone (the setup runs on
# one stream while kernels are profiled)
DENSE_KERNELS = ("potrf_diag", "potrf_panel", "potrf_update", "trsm_solve", "trsm_update", "gemm")
TRAFFIC_FILE = os.path.join(ROOT, "profiles", "traffic.json")


def source_digest(path, symbol=None):
    """SHA-256 prefix of a kernel's source: the text of the __global__
    function `symbol` (from its template line to its closing brace at column
    0), or of the whole file when symbol is None."""
    import hashlib
    import re
    with open(path) as f:
        text = f.read()
    if symbol:
        base = symbol.split("<")[0]
        m = re.search(r"(template <[^\n]*>\n)?__global__[^\n]*\b" + re.escape(base) + r"\(", text)
        if m:
            end = text.find("\n}\n", m.start())
            text = text[m.start():end + 3]
    return hashlib.sha256(text.encode()).hexdigest()[:16]


def measured_traffic(symbol, workload):
    """HBM bytes per launch of `symbol` from the recorded PMC runs, or None if
    none were recorded for this workload or the kernel source changed since."""
    try:
        with open(TRAFFIC_FILE) as f:
            rec = json.load(f).get(symbol)
    except (OSError, ValueError):
        return None
    if not rec or rec.get("workload") != workload:
        return None
    if source_digest(os.path.join(ROOT, rec["source"]), symbol) != rec["source_sha256_16"]:
        return None
    return rec["bytes_per_launch"]


def roofline_for(stats, workload):
    """Roofline object for the single kernel with the largest total time."""
    from paper_2304_01728_amd import dpgmg as D
    single = {k: v for k, v in stats.items() if k in SINGLE_KERNEL}
    cls, (n, ms, work) = max(single.items(), key=lambda kv: kv[1][1])
    sym = D.KERNEL_SYMBOLS.get(cls, cls)
    avg_ms = ms / n
    if cls in ("apply64", "apply32"):
        achieved = work / n / (avg_ms * 1e-3) / 1e9
        return {"kernel": sym, "bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBS,
                "unit": "GB/s", "frac": achieved / HBM_PEAK_GBS,
                "traffic": measured_traffic(sym, workload), "launches": n, "avg_ms": avg_ms,
                "work_per_launch": work / n}
    if cls == "applyb32":   # FP32 matrix cores; work = algorithmic flops
        achieved = work / n / (avg_ms * 1e-3) / 1e12
        return {"kernel": sym, "bound": "mfma", "achieved": achieved, "peak": FP32_PEAK_TFLOPS,
                "unit": "TFLOP/s", "frac": achieved / FP32_PEAK_TFLOPS, "traffic": None,
                "launches": n, "avg_ms": avg_ms, "work_per_launch": work / n}
    if cls in ("applyg64", "applyg32"):   # vector units; work = algorithmic flops
        achieved = work / n / (avg_ms * 1e-3) / 1e12
        peak = FP64_PEAK_TFLOPS if cls == "applyg64" else FP32_VECTOR_PEAK_TFLOPS
        return {"kernel": sym, "bound": "valu", "achieved": achieved, "peak": peak,
                "unit": "TFLOP/s", "frac": achieved / peak, "traffic": None,
                "launches": n, "avg_ms": avg_ms, "work_per_launch": work / n}
    if cls == "applyb64":   # FP64 matrix cores; work = algorithmic flops
        achieved = work / n / (avg_ms * 1e-3) / 1e12
        return {"kernel": sym, "bound": "mfma", "achieved": achieved, "peak": FP64_PEAK_TFLOPS,
                "unit": "TFLOP/s", "frac": achieved / FP64_PEAK_TFLOPS, "traffic": None,
                "launches": n, "avg_ms": avg_ms, "work_per_launch": work / n}
    return {"kernel": sym, "bound": "hbm", "achieved": None, "peak": HBM_PEAK_GBS,
            "unit": "GB/s", "frac": None, "traffic": None, "launches": n, "avg_ms": avg_ms}


def roofline_setup(stats):
    """The dense setup routines (several kernels each) and their kernels one by
    one (kernel symbols; each launch's share of its routine's LAPACK flop
    count) against the FP64 matrix-core peak, from the profiled step, in
    which the setup runs on one stream."""
    from paper_2304_01728_amd import dpgmg as D
    out = {}
    for cls in DENSE + DENSE_KERNELS:
        if cls in stats and stats[cls][2] > 0:
            n, ms, work = stats[cls]
            a = work / (ms * 1e-3) / 1e12
            key = cls if cls in DENSE else D.KERNEL_SYMBOLS[cls]
            if key in out:
                continue
            out[key] = {"bound": "mfma", "achieved": a, "peak": FP64_PEAK_TFLOPS,
                        "unit": "TFLOP/s", "frac": a / FP64_PEAK_TFLOPS, "ms": ms,
                        "launches": n, "tflop": work / 1e12}
    return out


def compare_precision(workload):
    """Time to tolerance of the FP64 and the mixed-precision path on the same
    workload (setup excluded), and the mixed solution's relative error against
    the FP64 GPU solution (the FP64 path is the one proven against the oracle
    at sizes the oracle can run)."""
    import dataclasses
    import torch
    from paper_2304_01728_amd import dpgmg as D
    from paper_2304_01728_amd import workloads as W
    base = W.ALL[workload]()
    out = {"workload": base.name, "tol": base.tol}
    xs = {}
    for prec in ("fp64", "mixed"):
        w = dataclasses.replace(base, precision=prec)
        torch.cuda.set_device(0)
        stream = torch.cuda.current_stream()
        ctx = D.dpg_setup(w.N, w.p, w.omega, loads_of(w), dp=w.dp,
                          options=make_options(D, w, torch_stream=stream.cuda_stream))
        nT = D.dpg_info(ctx).n_trace
        x = torch.zeros((w.nrhs, nT), dtype=torch.complex128, device="cuda:0")
        D.dpg_assemble(ctx)
        D.dpg_build_hierarchy(ctx)
        D.dpg_solve(ctx, nrhs=w.nrhs, tol=w.tol, x_out=x, device=True)   # warm
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        _, it, rr, code = D.dpg_solve(ctx, nrhs=w.nrhs, tol=w.tol, x_out=x, device=True)
        torch.cuda.synchronize()
        t = time.perf_counter() - t0
        out[prec] = {"time_to_tol_ms": 1e3 * t, "iterations": [int(v) for v in it],
                     "relres": float(np.max(rr)), "status": int(code),
                     "resident_GB": D.dpg_info(ctx).resident_bytes / 1e9}
        xs[prec] = x.cpu().numpy()
        ctx.close()
        del x
        torch.cuda.empty_cache()
    d = xs["mixed"] - xs["fp64"]
    out["mixed_rel_error_vs_fp64"] = float(np.linalg.norm(d) / np.linalg.norm(xs["fp64"]))
    out["speedup_mixed"] = out["fp64"]["time_to_tol_ms"] / out["mixed"]["time_to_tol_ms"]
    print(json.dumps(out), flush=True)


def store_vs_restrict(workload, omegas_over_pi=(2.0, 4.0, 8.0, 12.0)):
    """The paper's comparison of coarse operators (Sec. 4.2): PCG iterations
    and time to tolerance with Galerkin restriction and with operators stored
    (assembled directly on each coarser mesh), on the workload's mesh and
    order across frequencies."""
    import dataclasses
    import torch
    from paper_2304_01728_amd import dpgmg as D
    from paper_2304_01728_amd import workloads as W
    base = W.ALL[workload]()
    torch.cuda.set_device(0)
    stream = torch.cuda.current_stream()
    rows = []
    for om in omegas_over_pi:
        w = dataclasses.replace(base, omega=om * np.pi)
        row = {"omega_over_pi": om, "elements_per_wavelength": 2 * w.N / om}
        for name, flags in (("restrict", 0), ("store", D.DPG_STORE_COARSE)):
            opt = make_options(D, w, torch_stream=stream.cuda_stream)
            opt.flags |= flags
            ctx = D.dpg_setup(w.N, w.p, w.omega, loads_of(w), dp=w.dp, options=opt)
            nT = D.dpg_info(ctx).n_trace
            x = torch.zeros((w.nrhs, nT), dtype=torch.complex128, device="cuda:0")
            D.dpg_assemble(ctx)
            D.dpg_build_hierarchy(ctx)
            D.dpg_solve(ctx, nrhs=w.nrhs, tol=w.tol, x_out=x, device=True)
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            _, it, rr, code = D.dpg_solve(ctx, nrhs=w.nrhs, tol=w.tol, x_out=x, device=True)
            torch.cuda.synchronize()
            row[name] = {"iterations": int(np.max(it)), "time_to_tol_ms":
                         1e3 * (time.perf_counter() - t0), "status": int(code)}
            ctx.close()
            del x
            torch.cuda.empty_cache()
        print(f"[store-vs-restrict] omega = {om} pi: restrict {row['restrict']['iterations']}, "
              f"store {row['store']['iterations']}", file=sys.stderr, flush=True)
        rows.append(row)
    print(json.dumps({"comparison": "coarse operators: restrict vs store", "workload": base.name,
                      "tol": base.tol, "rows": rows}), flush=True)


def p_robustness(workload, p_max=4, elements_per_wavelength=(4.0, 2.0)):
    """The study of uniform p-refinements (Sec. 4.2): on the workload's mesh,
    with at least two elements per wavelength, the finest order p runs from 2
    to p_max over order levels down to p = 1 (then the mesh levels at p = 1),
    against the mesh levels alone at order p.  PCG iterations to the
    workload's tolerance, time to tolerance and setup time."""
    import dataclasses
    import torch
    from paper_2304_01728_amd import dpgmg as D
    from paper_2304_01728_amd import workloads as W
    base = W.ALL[workload]()
    torch.cuda.set_device(0)
    stream = torch.cuda.current_stream()
    rows = []
    for epw in elements_per_wavelength:
        for p in range(2, p_max + 1):
            w = dataclasses.replace(base, p=p, omega=2 * np.pi * base.N / epw)
            row = {"elements_per_wavelength": epw, "omega_over_pi": w.omega / np.pi, "p": p}
            for name, p_min in (("order_levels", 1), ("mesh_levels", 0)):
                opt = make_options(D, w, torch_stream=stream.cuda_stream)
                opt.p_min = p_min
                ctx = D.dpg_setup(w.N, w.p, w.omega, loads_of(w), dp=w.dp, options=opt)
                info = D.dpg_info(ctx)
                nT = info.n_trace
                x = torch.zeros((w.nrhs, nT), dtype=torch.complex128, device="cuda:0")
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                D.dpg_assemble(ctx)
                D.dpg_build_hierarchy(ctx)
                torch.cuda.synchronize()
                t_setup = time.perf_counter() - t0
                D.dpg_solve(ctx, nrhs=w.nrhs, tol=w.tol, x_out=x, device=True)
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                _, it, rr, code = D.dpg_solve(ctx, nrhs=w.nrhs, tol=w.tol, x_out=x, device=True)
                torch.cuda.synchronize()
                row[name] = {"iterations": int(np.max(it)), "status": int(code),
                             "time_to_tol_ms": 1e3 * (time.perf_counter() - t0),
                             "setup_ms": 1e3 * t_setup,
                             "levels": [[int(info.level_n[k]), int(info.level_p[k])]
                                        for k in range(info.nlevels)],
                             "resident_gb": D.dpg_info(ctx).resident_bytes / 1e9}
                row["n_trace"] = int(nT)
                ctx.close()
                del x
                torch.cuda.empty_cache()
            print(f"[p-robustness] {epw} elements per wavelength, p = {p}: order levels "
                  f"{row['order_levels']['iterations']}, mesh levels "
                  f"{row['mesh_levels']['iterations']} iterations", file=sys.stderr, flush=True)
            rows.append(row)
    print(json.dumps({"study": "uniform p-refinements: order levels vs mesh levels",
                      "mesh": base.N, "tol": base.tol, "precision": base.precision,
                      "smoothing": [base.nu_pre, base.nu_post], "rows": rows}), flush=True)


def recompute_study(workload, columns=(1, 8, 32)):
    """Stored patch inverses against inverses recomputed in every smoothing
    step (Sec. 5 and Sec. 6: a GPU code that recomputes the smoothing patches,
    amortised over several loads), FP64, on the workload's mesh and order with
    point sources (width 0.02, centres from seed 3): block solves of 1, 8 and
    32 right-hand sides, time per right-hand side and the device memory each
    context holds after dpg_release_setup."""
    import dataclasses
    import torch
    from paper_2304_01728_amd import dpgmg as D
    from paper_2304_01728_amd import workloads as W
    base = W.ALL[workload]()
    torch.cuda.set_device(0)
    stream = torch.cuda.current_stream()
    rows = []
    for nr in columns:
        cen = W.source_centres(3, nr)
        w = dataclasses.replace(base, precision="fp64", sources=cen, nrhs=nr, direction=None)
        row = {"columns": nr}
        for name, rec in (("stored", False), ("recomputed", True)):
            opt = make_options(D, w, torch_stream=stream.cuda_stream, recompute=rec)
            ctx = D.dpg_setup(w.N, w.p, w.omega, loads_of(w), dp=w.dp, options=opt)
            nT = D.dpg_info(ctx).n_trace
            x = torch.zeros((nr, nT), dtype=torch.complex128, device="cuda:0")
            D.dpg_assemble(ctx)
            D.dpg_build_hierarchy(ctx)
            D.dpg_release_setup(ctx)
            D.dpg_solve(ctx, nrhs=nr, tol=w.tol, x_out=x, device=True)   # warm (graphs)
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            _, it, rr, code = D.dpg_solve(ctx, nrhs=nr, tol=w.tol, x_out=x, device=True)
            torch.cuda.synchronize()
            t = time.perf_counter() - t0
            row[name] = {"solve_ms": 1e3 * t, "ms_per_column": 1e3 * t / nr,
                         "iterations": [int(v) for v in it], "status": int(code),
                         "resident_GB": D.dpg_info(ctx).resident_bytes / 1e9}
            ctx.close()
            del x
            torch.cuda.empty_cache()
        row["recomputed_over_stored"] = (row["recomputed"]["solve_ms"] /
                                         row["stored"]["solve_ms"])
        print(f"[recompute] {nr} columns: stored {row['stored']['ms_per_column']:.1f} ms, "
              f"recomputed {row['recomputed']['ms_per_column']:.1f} ms per column",
              file=sys.stderr, flush=True)
        rows.append(row)
    print(json.dumps({"study": "stored vs recomputed patch inverses, FP64 block solves",
                      "mesh": base.N, "p": base.p, "omega": base.omega, "tol": base.tol,
                      "smoothing": [base.nu_pre, base.nu_post], "rows": rows}), flush=True)


def calibrate_copy():
    """A plain device copy of known size, for scaling HBM counters."""
    import torch
    nbytes = 1 << 30
    x = torch.ones(nbytes // 8, dtype=torch.float64, device="cuda:0")
    y = torch.empty_like(x)
    for _ in range(3):
        y.copy_(x)
    torch.cuda.synchronize()
    print(json.dumps({"calibration": "copy", "bytes_read": nbytes, "bytes_written": nbytes,
                      "launches": 3}), flush=True)


def serving_child(n_req, seed, max_active, load_factor):
    """serving_stream in a child process (bench.py --serving); its JSON line."""
    import subprocess
    cmd = [sys.executable, os.path.abspath(__file__), "--serving", "--requests", str(n_req),
           "--seed", str(seed), "--max-active", str(max_active),
           "--load-factor", str(load_factor)]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, timeout=900, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"serving stream failed with status {res.returncode}")
    return json.loads(res.stdout.strip().splitlines()[-1])


def cpu_model():
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def cpu_oracle_job(w, N, threads):
    """The oracle's whole job on a plane-wave problem of the workload's order
    and smoothing on an N^3 mesh with the workload's elements per wavelength:
    topology, element stage, hierarchy, PCG to the workload's tolerance.
    threads: BLAS threads (None = the host BLAS default)."""
    from threadpoolctl import threadpool_info, threadpool_limits
    from oracle import dpg, multigrid
    omega = w.omega * N / w.N
    with threadpool_limits(threads):
        used = max([tp.get("num_threads", 1) for tp in threadpool_info()] + [1])
        t0 = time.perf_counter()
        if w.direction is not None:
            load = dict(u0=dpg.plane_wave_u0(omega, w.direction))
        else:
            load = dict(f=dpg.gaussian_sources(w.sources[:1], w.sigma, [1.0]))
        pr = dpg.Problem(N, w.p, omega, [load])
        t1 = time.perf_counter()
        S, s, _ = pr.condensed()
        rhs = dpg.assemble_vector(pr.edofs, s, pr.num.n)[:, 0]
        t2 = time.perf_counter()
        H = multigrid.Hierarchy(N, w.p, S, theta=w.theta, nu_pre=w.nu_pre, nu_post=w.nu_post)
        t3 = time.perf_counter()
        _, it, rr = H.solve(rhs, w.tol)
        t4 = time.perf_counter()
        # the solve phase is short: two more runs, the median of the three is reported
        ts = [t4 - t3]
        for _ in range(2):
            ta = time.perf_counter()
            H.solve(rhs, w.tol)
            ts.append(time.perf_counter() - ta)
    nT = pr.num.n
    t_solve = float(np.median(ts))
    return {"value": nT * it / t_solve, "threads": used, "iterations": int(it),
            "time_to_tol_s": t_solve, "solve_runs_s": [round(t, 4) for t in ts],
            "job_s": t4 - t0, "job_value": nT * it / (t4 - t0),
            "phase_s": {"topology": round(t1 - t0, 3), "element": round(t2 - t1, 3),
                        "hierarchy": round(t3 - t2, 3), "solve": round(t4 - t3, 3)},
            "n_trace": int(nT), "omega": omega}


def cpu_baseline(w, N_cpu=4):
    """The oracle timed on the host on a smaller mesh of the same order (the
    full workload does not fit the oracle's time), once on one core and once
    with the host BLAS threads.  value = n_trace x PCG iterations / time of
    the solve phase (the median of three runs of the oracle's PCG), the
    definition the GPU line uses, for the faster of the two settings;
    job_value counts the whole job."""
    from paper_2304_01728_amd import workloads as W
    one = cpu_oracle_job(w, N_cpu, 1)
    allc = cpu_oracle_job(w, N_cpu, None)
    # the smallest workload (4^3, p = 2, omega = 2 pi, V(1,1), tol 1e-10) at its own size
    w4 = W.plane_wave_4()
    small = {"workload": w4.name, "one_core": cpu_oracle_job(w4, w4.N, 1),
             "all_cores": cpu_oracle_job(w4, w4.N, None)}
    # threaded BLAS on the oracle's many small matrices can be slower than one
    # core: the faster of the two settings is the baseline, both are reported
    best = allc if allc["value"] >= one["value"] else one
    return {"value": best["value"], "unit": "trace-DOF*PCG-iters/s", "cores": best["threads"],
            "kind": "oracle",
            "sample": ("the whole oracle job (topology, element stage, hierarchy, PCG to "
                       "tol %g) for one right-hand side of the workload's kind on the %d^3 "
                       "mesh of order %d at omega = %.4f (the workload's "
                       "elements per wavelength), V(%d,%d): %d trace unknowns, %d iterations; "
                       "the workload's own mesh is beyond the oracle's time"
                       % (w.tol, N_cpu, w.p, allc["omega"], w.nu_pre, w.nu_post,
                          allc["n_trace"], allc["iterations"])),
            "cpu_model": cpu_model(), "host_cpus": os.cpu_count(),
            "all_cores": allc, "one_core": one, "plane_wave_4": small}


def serving_stream(n_req, seed, max_active, load_factor):
    """The layered-medium point-source stream: a pool of 8 operators drawn
    once (N in {8, 12, 16, 24, 32}, p in {2, 3, 4}, four z-layers, speeds
    U[1, 4], five elements per shortest wavelength), Poisson arrivals at
    load_factor x the measured single-request capacity, 1-16 sources per
    request, mixed precision, tol 1e-8.  The hierarchies that fit the HBM
    budget are built before the clock starts (a server keeps them resident);
    operators admitted later are built on arrival and counted in latency.
    The capacity is measured on the warm server itself: one 8-source request
    per resident operator, alone, through the same batch path (the second of
    two runs; the first captures the batch's graphs).  Returns the result
    as a dict."""
    import torch
    from paper_2304_01728_amd import serving as S
    torch.cuda.set_device(0)
    free, total = torch.cuda.mem_get_info(0)
    budget = int(0.85 * free)
    ops = S.draw_pool(seed=seed)
    srv = S.Server(ops, budget_bytes=budget, max_active=max_active)
    try:
        # warm the resident set in pool order while it fits
        warm = []
        for op in ops:
            if sum(r.nbytes for r in srv.resident.values()) + srv.estimate(op) > budget:
                break
            print(f"[serving] build op {op.key}: N={op.N} p={op.p} omega={op.omega:.2f}",
                  file=sys.stderr, flush=True)
            r = S.Request(-1 - op.key, op.key, np.array([[0.5, 0.5, 0.5, 0.02, 1.0, 0.0]]))
            srv.submit(r)
            r.done.wait()
            if r.error is not None:
                raise RuntimeError(f"operator {op.key}: {r.error}")
            warm.append(op.key)
        # service time of one 8-source request per operator, alone on the server
        probe = np.random.default_rng(seed + 2)
        service = []
        for key in warm:
            cen = probe.uniform(0.1, 0.9, size=(8, 3))
            src = np.column_stack([cen, np.full(8, 0.02), np.ones(8), np.zeros(8)])
            for rep in range(2):
                r = S.Request(-100 - key, key, src)
                t0 = time.perf_counter()
                srv.submit(r)
                r.done.wait()
                t = time.perf_counter() - t0
                if r.error is not None:
                    raise RuntimeError(f"operator {key}: {r.error}")
            service.append(t)
        capacity = 1.0 / float(np.mean(service))
        rate = load_factor * capacity
        reqs = S.draw_requests(ops, n_req, rate, seed=seed)
        builds0, evict0 = srv.builds, srv.evictions
        print(f"[serving] capacity {capacity:.2f} req/s, rate {rate:.2f} req/s, {n_req} requests, "
              f"warm operators {warm}", file=sys.stderr, flush=True)
        wall, lat = S.run_stream(srv, reqs)
        builds, evictions = srv.builds - builds0, srv.evictions - evict0
    finally:
        srv.close()
    batches = [r.batch for r in reqs]
    return {
        "metric": "solves/s", "value": n_req / wall, "unit": "solves/s", "n_gpus": 1,
        "higher_is_better": True, "dtype": "f64+f32",
        "data": "synthetic",
        "latency_ms": {"p50": 1e3 * S.percentile(lat, 50), "p99": 1e3 * S.percentile(lat, 99),
                       "mean": 1e3 * float(np.mean(lat)), "max": 1e3 * float(np.max(lat))},
        "requests": n_req, "wall_s": wall, "arrival_rate": rate,
        "single_request_capacity": capacity, "load_factor": load_factor,
        "mean_batch": float(np.mean(batches)), "max_batch": int(np.max(batches)),
        "joined_running_batch": int(sum(r.joined_running for r in reqs)),
        "batch_note": ("batch = most columns a request's operator batch ran while the request "
                       "was in it; joined_running_batch = requests admitted into a block solve "
                       "already part-way through"),
        "builds_during_stream": builds,
        "evictions_during_stream": evictions,
        "hbm_budget_GB": budget / 1e9,
        "config": {"workload": "serving stream: 8 layered-medium operators, N 8-32, p 2-4, "
                               "Poisson arrivals, 1-16 Gaussian sources per request",
                   "operators": [{"N": o.N, "p": o.p, "omega": round(o.omega, 4),
                                  "speeds": sorted(set(np.round(o.c, 4).tolist()))}
                                 for o in ops],
                   "seed": seed, "max_active": max_active, "tol": 1e-8},
    }


def fp64_twin(w, x_mixed):
    """The same workload solved in FP64 throughout: time to tolerance (setup
    excluded, mean of two solves after a warm one) and the error of the
    mixed-precision solution against it (the FP64 path is the one proven
    against the oracle)."""
    import dataclasses
    import torch
    from paper_2304_01728_amd import dpgmg as D
    w64 = dataclasses.replace(w, precision="fp64")
    stream = torch.cuda.current_stream()
    ctx = D.dpg_setup(w64.N, w64.p, w64.omega, loads_of(w64), dp=w64.dp,
                      options=make_options(D, w64, torch_stream=stream.cuda_stream))
    nT = D.dpg_info(ctx).n_trace
    x = torch.zeros((w64.nrhs, nT), dtype=torch.complex128, device="cuda:0")
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    D.dpg_assemble(ctx)
    t1 = time.perf_counter()
    D.dpg_build_hierarchy(ctx)
    torch.cuda.synchronize()
    t2 = time.perf_counter()
    D.dpg_solve(ctx, nrhs=w64.nrhs, tol=w64.tol, x_out=x, device=True)   # warm
    torch.cuda.synchronize()
    ts = []
    for _ in range(2):
        ta = time.perf_counter()
        _, it, rr, code = D.dpg_solve(ctx, nrhs=w64.nrhs, tol=w64.tol, x_out=x, device=True)
        torch.cuda.synchronize()
        ts.append(time.perf_counter() - ta)
    resident = D.dpg_info(ctx).resident_bytes
    x64 = x.cpu().numpy()
    ctx.close()
    del x
    torch.cuda.empty_cache()
    t = float(np.mean(ts))
    iters = int(np.sum(it))
    return {"time_to_tol_ms": 1e3 * t, "iterations": iters, "relres": float(np.max(rr)),
            "status": int(code), "value": nT * iters / t,
            "ms_per_iteration": 1e3 * t / max(iters, 1),
            "setup_ms": {"assemble": 1e3 * (t1 - t0), "hierarchy": 1e3 * (t2 - t1)},
            "resident_GB": resident / 1e9,
            "mixed_rel_error_vs_fp64": float(np.linalg.norm(x_mixed - x64) / np.linalg.norm(x64))}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=3)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--workload", default="plane_wave_32_mixed")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--recompute-patches", action="store_true",
                    help="smooth with patch inverses recomputed in every application (FP64 "
                         "workloads; no stored inverses)")
    ap.add_argument("--no-kernel-stats", action="store_true",
                    help="skip the extra step timed kernel by kernel with HIP events (for runs "
                         "under a hardware-counter profiler)")
    ap.add_argument("--no-fp64-twin", action="store_true",
                    help="skip the FP64 solve of a mixed-precision workload")
    ap.add_argument("--columnwise", action="store_true",
                    help="solve several right-hand sides one by one instead of as a block")
    ap.add_argument("--compare-precision", action="store_true",
                    help="solve the workload in FP64 and in mixed precision; report times "
                         "to tolerance and the mixed solution's error against the FP64 one")
    ap.add_argument("--store-vs-restrict", action="store_true",
                    help="iterations and time to tolerance with restricted and with stored "
                         "coarse operators across frequencies, on the workload's mesh")
    ap.add_argument("--p-robustness", action="store_true",
                    help="iterations as the finest order grows, with order levels down to "
                         "p = 1 and with mesh levels only (Sec. 4.2)")
    ap.add_argument("--recompute-study", action="store_true",
                    help="stored vs recomputed patch inverses on FP64 block solves of 1, 8 "
                         "and 32 point sources (time per right-hand side, memory)")
    ap.add_argument("--calibrate-copy", action="store_true",
                    help="run only a 1 GiB device copy (for HBM counter calibration)")
    ap.add_argument("--serving", action="store_true",
                    help="run the layered-medium request stream through the serving loop; "
                         "report solves/s and p50/p99 latency")
    ap.add_argument("--requests", type=int, default=200)
    ap.add_argument("--serving-requests", type=int, default=100,
                    help="requests of the serving stream the default run reports beside the "
                         "solver line (0: none)")
    ap.add_argument("--seed", type=int, default=4)
    ap.add_argument("--max-active", type=int, default=8)
    ap.add_argument("--load-factor", type=float, default=0.7)
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py measures one GPU: the library has no multi-GPU path; "
              "run it with --gpus 1", file=sys.stderr)
        sys.exit(2)
    if args.calibrate_copy:
        calibrate_copy()
        return
    if args.compare_precision:
        compare_precision(args.workload)
        return
    if args.store_vs_restrict:
        store_vs_restrict(args.workload)
        return
    if args.p_robustness:
        p_robustness(args.workload)
        return
    if args.recompute_study:
        recompute_study(args.workload)
        return
    if args.serving:
        print(json.dumps(serving_stream(args.requests, args.seed, args.max_active,
                                        args.load_factor)), flush=True)
        return

    import torch
    from paper_2304_01728_amd import dpgmg as D
    from paper_2304_01728_amd import workloads as W

    w = W.ALL[args.workload]()
    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    stream = torch.cuda.current_stream(dev)
    opt = make_options(D, w, torch_stream=stream.cuda_stream, columnwise=args.columnwise,
                       recompute=args.recompute_patches)
    print(f"[bench] {w.name}: setup", file=sys.stderr, flush=True)
    t0 = time.perf_counter()
    ctx = D.dpg_setup(w.N, w.p, w.omega, loads_of(w), dp=w.dp, options=opt)
    setup_s = time.perf_counter() - t0
    info = D.dpg_info(ctx)
    nT = info.n_trace
    x = torch.zeros((w.nrhs, nT), dtype=torch.complex128, device=dev)

    def step():
        D.dpg_assemble(ctx)
        D.dpg_build_hierarchy(ctx)
        _, it, rr, code = D.dpg_solve(ctx, nrhs=w.nrhs, tol=w.tol, x_out=x, device=True)
        return it, rr, code

    for k in range(args.warmup):
        step()
        print(f"[bench] warmup step {k + 1}/{args.warmup} done", file=sys.stderr, flush=True)
    torch.cuda.synchronize()
    iters_total = 0
    phase = {"assemble": 0.0, "hierarchy": 0.0, "solve": 0.0}
    t_start = time.perf_counter()
    for _ in range(args.steps):
        ta = time.perf_counter()
        D.dpg_assemble(ctx)
        tb = time.perf_counter()
        D.dpg_build_hierarchy(ctx)
        tc = time.perf_counter()
        _, it, rr, code = D.dpg_solve(ctx, nrhs=w.nrhs, tol=w.tol, x_out=x, device=True)
        td = time.perf_counter()
        phase["assemble"] += tb - ta
        phase["hierarchy"] += tc - tb
        phase["solve"] += td - tc
        iters_total += int(np.sum(it))
        iters_cols = [int(v) for v in it]
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t_start
    print(f"[bench] {args.steps} timed steps done ({elapsed:.2f} s)", file=sys.stderr, flush=True)
    # one more step with per-kernel HIP events for the kernel statistics (the
    # events serialise the launches, so the timed steps above run without them)
    stats = {}
    if not args.no_kernel_stats:
        D.dpg_profile(ctx, True)
        step()
        torch.cuda.synchronize()
        stats = D.dpg_kernel_stats(ctx)
        D.dpg_profile(ctx, False)
    resident = D.dpg_info(ctx).resident_bytes
    D.dpg_release_setup(ctx)
    resident_solve = D.dpg_info(ctx).resident_bytes
    x_host = x.cpu().numpy() if (w.precision == "mixed" and w.nrhs == 1) else None
    ctx.close()
    del x
    torch.cuda.empty_cache()
    iters_per_step = iters_total / args.steps
    solve_s = phase["solve"] / args.steps
    # the metric (trace-DOF x PCG iterations / s) is defined on the solve phase;
    # the setup phases are reported beside it
    value = nT * iters_per_step / solve_s
    out = {
        "metric": "trace-DOF*PCG-iters/s",
        "value": value,
        "unit": "trace-DOF*PCG-iters/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": 1e3 * elapsed / args.steps,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64" if w.precision == "fp64" else "f64+f32",
        "data": "synthetic",
        "config": {"workload": w.name + (" recomputed patches" if args.recompute_patches else ""),
                   "N": w.N, "p": w.p, "dp": w.dp, "omega": w.omega,
                   "nu": [w.nu_pre, w.nu_post], "theta": w.theta, "tol": w.tol,
                   "precision": w.precision, "nrhs": w.nrhs, "n_trace": nT,
                   "n_macro": info.n_macro, "levels": list(info.level_n)[:info.nlevels]},
        "value_definition": ("n_trace x PCG iterations / solve-phase seconds (dpg_solve entry "
                             "to return, mean over the timed steps); every step also runs the "
                             "element stage and the hierarchy, timed in phases_ms"),
        "iterations": iters_per_step,
        "iterations_per_column": iters_cols if w.nrhs > 1 else None,
        "relres": float(np.max(rr)),
        "time_to_tol_ms": 1e3 * solve_s,
        "ms_per_iteration": 1e3 * solve_s / max(iters_per_step / max(w.nrhs, 1), 1),
        "solves_per_s": w.nrhs / solve_s,
        "rhs_mode": "columnwise" if args.columnwise or w.nrhs == 1 else "block",
        "whole_step": {"value": nT * iters_total / elapsed, "unit": "trace-DOF*PCG-iters/s",
                       "note": "n_trace x iterations / (element stage + hierarchy + solve)"},
        "phases_ms": {k: 1e3 * v / args.steps for k, v in phase.items()},
        "setup_topology_ms": 1e3 * setup_s,
        "resident_GB": resident / 1e9,
        "resident_after_release_GB": resident_solve / 1e9,
        "roofline": roofline_for(stats, w.name) if stats else None,
        "roofline_setup": roofline_setup(stats),
        "kernels": {k: {"launches": n, "ms": ms, "work": wk} for k, (n, ms, wk) in stats.items()},
        "kernels_note": ("per-kernel HIP events over one extra profiled step, in which the "
                         "setup runs on one stream (each launch timed alone)"),
    }
    if x_host is not None and not args.no_fp64_twin:
        print("[bench] FP64 solve of the same workload", file=sys.stderr, flush=True)
        tw = fp64_twin(w, x_host)
        out["fp64_vs_mixed"] = {
            "time_to_tol_ms": {"fp64": tw["time_to_tol_ms"], "mixed": 1e3 * solve_s},
            "iterations": {"fp64": tw["iterations"], "mixed": iters_per_step},
            "speedup_mixed": tw["time_to_tol_ms"] / (1e3 * solve_s),
            "mixed_rel_error_vs_fp64": tw["mixed_rel_error_vs_fp64"],
            "fp64": tw}
    if args.serving_requests > 0:
        # in a process of its own, as a server runs: after the legs above have
        # allocated and freed most of the HBM, the same process serves slower
        print("[bench] serving stream (child process)", file=sys.stderr, flush=True)
        out["serving"] = serving_child(args.serving_requests, args.seed, args.max_active,
                                       args.load_factor)
    if not args.no_cpu_baseline:
        print("[bench] CPU oracle baseline", file=sys.stderr, flush=True)
        out["cpu_baseline"] = cpu_baseline(w)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
