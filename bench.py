#!/usr/bin/env python3
"""Benchmark: RandRAND-preconditioned PCG versus plain CG on one MI355X.

Workload (one step = the whole hot path on one synthetic problem): matrix-free
kernel ridge regression, n = 50,000 points in d = 16 from a 10-component
Gaussian mixture, RBF kernel with median-distance bandwidth, A = K/n,
mu = 1e-4, SRHT test matrix with l = 500, float32 kernel entries with float64
accumulation, dots/projections in float64, stop at relative residual 1e-6.

A step = rr_build_precond (Omega, kernel-GEMM sketch on MFMA, sketched
Cholesky QR, core, tau power iterations) + rr_solve (PCG with restarts).  The
same solve with l = 0 (plain CG, identical kernels) is timed beside it.

Prints one JSON line.  `value` is solves per second (inputs resident in HBM).
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_LANE_OPS = 256 * 4 * 16 * 2.4e9      # CUs x SIMDs x lanes x clock (non-packed VALU)
PEAK_FP32_MFMA_TFLOPS = 157.3
PEAK_BF16_TFLOPS = 2500.0
PEAK_HBM_GBS = 8000.0


def _src_hash(*names):
    h = hashlib.sha256()
    for n in names:
        with open(os.path.join(ROOT, "paper_2509_19747_amd", "csrc", n), "rb") as f:
            h.update(f.read())
    return h.hexdigest()[:16]


def _traffic(kernel: str, src_hash: str):
    """HBM bytes per launch from committed rocprofv3 counter runs, if still current."""
    p = os.path.join(ROOT, "profiles", "traffic.json")
    try:
        with open(p) as f:
            t = json.load(f).get(kernel)
    except (OSError, ValueError):
        return None
    if not t or t.get("src_hash") != src_hash:
        return None
    return t.get("bytes_per_launch")


TRAFFIC_SOURCES = ("kernels_ksym_mma.hip", "kmma.hpp", "kentry.hpp", "common.hpp")
TRAFFIC_KERNEL = "k_ksym_mma<1, 16, 1, double>"


def traffic_from_counters(d: str, out_path: str | None = None) -> dict:
    """HBM bytes of the headline matvec from two rocprofv3 --pmc csv runs under d
    (written to out_path as JSON when given; the command line writes profiles/traffic.json).

    d/FETCH_SIZE and d/WRITE_SIZE hold one run each of the headline step with
    --copy-calibration.  Each counter is scaled by what it reads for the 1 GiB
    device-to-device copy (bytes moved / counter KiB), and the headline matvec's
    bytes per launch are the scaled medians over its launches.
    """
    import csv

    med, cal = {}, {}
    for c in ("FETCH_SIZE", "WRITE_SIZE"):
        with open(os.path.join(d, c, f"{c}_counter_collection.csv")) as f:
            rows = list(csv.DictReader(f))
        copy = [float(r["Counter_Value"]) for r in rows if "copy" in r["Kernel_Name"].lower()]
        km = sorted(float(r["Counter_Value"]) for r in rows if TRAFFIC_KERNEL in r["Kernel_Name"])
        if not copy or not km:
            raise SystemExit(f"{c}: no calibration copy or no {TRAFFIC_KERNEL} launch in {d}")
        cal[c], med[c] = max(copy), km[len(km) // 2]
    fs, ws = (1 << 20) / cal["FETCH_SIZE"], (1 << 20) / cal["WRITE_SIZE"]
    fb, wb = med["FETCH_SIZE"] * fs * 1024, med["WRITE_SIZE"] * ws * 1024
    t = {"k_ksym_mma": {
        "src_hash": _src_hash(*TRAFFIC_SOURCES), "bytes_per_launch": fb + wb,
        "fetch_bytes": fb, "write_bytes": wb, "fetch_scale": fs, "write_scale": ws,
        "fetch_kib": med["FETCH_SIZE"], "write_kib": med["WRITE_SIZE"],
        "workload": "kernel ridge RBF n=50000 d=16, one float64-sum launch (1 column)",
        "calibration": "1 GiB device-to-device copy: FETCH_SIZE %d KiB, WRITE_SIZE %d KiB"
                       % (cal["FETCH_SIZE"], cal["WRITE_SIZE"])}}
    if out_path:
        with open(out_path, "w") as f:
            json.dump(t, f, indent=1)
            f.write("\n")
    return t


def trace_summary(db: str, top: int = 25) -> str:
    """Markdown table of the kernels in a rocprofv3 --kernel-trace results database.

    Per kernel: launches, total and mean duration, and the mean over the launches
    longer than a tenth of the kernel's median ("work": PCG iterations past a
    column's convergence, which the device-side stop flags turn into near-empty
    launches, are left out of it).
    """
    import sqlite3
    import statistics

    c = sqlite3.connect(db)
    rows = c.execute("select S.display_name, K.end - K.start from rocpd_kernel_dispatch K "
                     "join rocpd_info_kernel_symbol S on S.id = K.kernel_id and S.guid = K.guid"
                     ).fetchall()
    by = {}
    for name, dur in rows:
        by.setdefault(name, []).append(dur / 1000.0)
    total = sum(sum(v) for v in by.values())
    out = [f"Total kernel time {total / 1000:.1f} ms over {len(rows)} launches.", "",
           "| kernel | calls | total ms | avg us | avg us (work) | work calls | min us | max us | % |",
           "|---|---|---|---|---|---|---|---|---|"]
    for name, v in sorted(by.items(), key=lambda kv: -sum(kv[1]))[:top]:
        med = statistics.median(v)
        w = [x for x in v if x >= 0.1 * med]
        out.append(f"| `{name}` | {len(v)} | {sum(v) / 1000:.2f} | {sum(v) / len(v):.2f} | "
                   f"{sum(w) / len(w):.2f} | {len(w)} | {min(v):.2f} | {max(v):.2f} | "
                   f"{100 * sum(v) / total:.1f} |")
    return "\n".join(out)


def cpu_baseline(prob, iters_hint: int, restarts_hint: int, power_iters: int, full: bool = False):
    """Time the float64 oracle on the host cores and express it in solves/s.

    full=False (default, about 20 s): a bounded sample of the same solve.  One full
    float64 kernel matvec (row-blocked, all host cores), the oracle sketch on the
    first 2,000 of the n rows (scaled by n/2000), and the oracle's sketched Cholesky
    QR on an n x l matrix; the solve is then T_sketch + T_orth +
    (2 N_pow + iters + restarts + 2) T_matvec with the iteration count of the same
    algorithm measured on the GPU in this run.
    full=True: the oracle's whole C-RandRAND build and PCG solve with restarts,
    timed end to end (about 1.5 minutes on 16 cores).
    """
    import numpy as np

    from oracle import randrand as orr
    from oracle import rng as orng
    from oracle import solvers as osol
    from oracle.operators import Operator, kernel_block

    cores = _host_threads()
    op = Operator.from_problem(prob, threads=cores)
    n, l, mu = prob.n, prob.l, prob.mus[0]
    if full:
        t0 = time.perf_counter()
        Pr = orr.build(op, [mu], l, "srht", prob.omega_seed, omega_bf16=True,
                       power_iters=power_iters)[0]
        t_build = time.perf_counter() - t0
        res = osol.pcg(op.shifted(mu), Pr.apply, prob.b, prob.tol)
        t_all = time.perf_counter() - t0
        return {
            "value": 1.0 / t_all, "unit": "solves/s", "cores": cores, "kind": "oracle",
            "sample": (f"the whole float64 oracle solve, timed: build {t_build:.1f} s (sketch, "
                       f"sketched Cholesky QR, core, {power_iters}+{power_iters} power steps), PCG "
                       f"{t_all - t_build:.1f} s ({res.iters} iterations, {res.restarts} restarts, "
                       f"relres {res.relres:.2e})"),
            "s_per_solve": t_all,
        }
    u = np.random.default_rng(0).standard_normal(n)
    t0 = time.perf_counter()
    op.matmat(u)
    t_mv = time.perf_counter() - t0
    Om = orng.srht_omega(prob.omega_seed, n, l)
    rows = 2000
    t0 = time.perf_counter()
    Kb = kernel_block(op.kind, op.kconst, op.X[:rows], op.X)
    Yb = op.scale * (Kb @ Om) + mu * Om[:rows]
    t_sk = (time.perf_counter() - t0) * (n / rows)
    del Kb, Yb
    Y = np.random.default_rng(1).standard_normal((n, l))
    t0 = time.perf_counter()
    orr.sketched_cholqr(Y, orng.theta(prob.omega_seed, n, l))
    t_orth = time.perf_counter() - t0
    nmv = 2 * power_iters + iters_hint + restarts_hint + 2
    est = t_sk + t_orth + nmv * t_mv
    return {
        "value": 1.0 / est, "unit": "solves/s", "cores": cores, "kind": "oracle",
        "sample": (f"float64 oracle on the host: 1 full kernel matvec ({t_mv:.2f} s), sketch of "
                   f"{rows}/{n} rows scaled ({t_sk:.1f} s est.), sketched Cholesky QR of an "
                   f"{n}x{l} matrix ({t_orth:.1f} s); solve = {nmv} matvecs "
                   f"(2x{power_iters} power + {iters_hint} PCG + {restarts_hint}+2 residuals)"),
        "est_s_per_solve": est,
    }


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--n", type=int, default=50_000)
    ap.add_argument("--l", type=int, default=500)
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--cpu-full", action="store_true",
                    help="time the whole float64 oracle solve instead of the bounded sample")
    ap.add_argument("--no-cg", action="store_true")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="kernel-ridge: first copy 1 GiB device to device (a plain copy of known "
                         "size that scales rocprofv3 FETCH_SIZE / WRITE_SIZE counters)")
    ap.add_argument("--context-mu", type=float, nargs="*", default=[1e-6],
                    help="kernel-ridge: also time one RandRAND and one plain-CG solve at these "
                         "smaller shifts (reported under 'context', outside the timed steps)")
    ap.add_argument("--graph", action="store_true", help="replay PCG batches as hipGraphs")
    ap.add_argument("--workload", default="kernel-ridge",
                    choices=["kernel-ridge", "small", "precision", "batched", "serving", "variants"],
                    help="kernel-ridge is the headline step; the others measure the remaining "
                         "paths (dense mixed precision, batched multi-shift, serving) and "
                         "the solver and preconditioner variants")
    ap.add_argument("--requests", type=int, default=2200, help="serving: number of requests")
    ap.add_argument("--rate", type=float, default=200.0, help="serving: arrivals per second")
    ap.add_argument("--slots", type=int, default=16, help="serving: concurrent requests")
    ap.add_argument("--graph-iters", type=int, default=8,
                    help="serving: PCG iterations per replayed hipGraph batch (0: plain launches)")
    ap.add_argument("--budget-gb", type=float, default=96.0, help="serving: HBM budget")
    ap.add_argument("--lanes", type=int, default=0,
                    help="serving: grouped replay lanes (0: each request replays its own graph)")
    ap.add_argument("--dump", default="", help="serving: write per-request records (JSON lines)")
    ap.add_argument("--nrhs", type=int, default=256, help="batched: right-hand sides per shift")
    ap.add_argument("--traffic-from", default="",
                    help="no GPU work: derive profiles/traffic.json from the FETCH_SIZE and "
                         "WRITE_SIZE counter runs under this directory, then exit")
    ap.add_argument("--trace-summary", default="",
                    help="no GPU work: print a markdown table of the kernels in this rocprofv3 "
                         "--kernel-trace results database, then exit")
    ap.add_argument("--top", type=int, default=25, help="trace summary: kernels listed")
    args = ap.parse_args()
    if args.trace_summary:
        print(trace_summary(args.trace_summary, args.top))
        return
    if args.traffic_from:
        print(json.dumps(traffic_from_counters(args.traffic_from,
                                               os.path.join(ROOT, "profiles", "traffic.json"))))
        return
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (asked for --gpus {args.gpus}); the multi-GPU "
              "sharding is a design, not a build", file=sys.stderr)
        sys.exit(2)
    if args.workload != "kernel-ridge":
        {"small": bench_small, "precision": bench_precision, "batched": bench_batched,
         "serving": bench_serving, "variants": bench_variants}[args.workload](args)
        return

    import numpy as np
    import torch

    import paper_2509_19747_amd as rr
    from paper_2509_19747_amd import binding as rb
    import workloads

    assert torch.cuda.is_available(), "bench.py needs a GPU"
    if args.copy_calibration:
        src = torch.ones(1 << 27, dtype=torch.float64, device="cuda")   # 1 GiB
        dst = torch.empty_like(src)
        dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst
    prob = workloads.cfg_kernel_ridge(n=args.n, l=args.l)
    mu, n, l, d = prob.mus[0], prob.n, prob.l, prob.d
    pts = torch.from_numpy(prob.pts).cuda()
    b = torch.from_numpy(prob.b).cuda()
    kop = rr.kernel_operator(rr.OP_RBF, pts, prob.kconst, prob.scale)
    build_kw = dict(l=l, sketch="srht", seed=prob.omega_seed, prec="fp32", tau_rule="opt")
    solve_kw = dict(tol=prob.tol, certify=False, use_graph=args.graph, check_every=8)

    def step():
        P = rr.build_precond(kop, [mu], **build_kw)
        x, info = P.solve(b, **solve_kw)
        return P, x, info

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    rb.profile_enable(True)
    infos = []
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        P, x, info = step()
        infos.append(info)
    torch.cuda.synchronize()
    t_total = time.perf_counter() - t0
    kmv_n, kmv_ms = rb.profile_read(rb.PROF_KERNEL_MATVEC)
    sk_n, sk_ms = rb.profile_read(rb.PROF_KERNEL_SKETCH)
    k64_n, k64_ms = rb.profile_read(rb.PROF_KERNEL_MATVEC64)
    rb.profile_enable(False)
    ms_step = 1e3 * t_total / args.steps
    last = infos[-1]

    # accuracy of the last result against the float64 operator (outside the timed region)
    r64 = b - rr.apply_operator(kop, mu, "fp64", x)
    nb = float(torch.linalg.norm(b))
    relres_fp64 = float(torch.linalg.norm(r64)) / nb
    # per-result error bound for the float32-class working operator: ||dA|| by power
    # iteration on A_fp32 - A (once, outside the timed region)
    dA = rb.operator_delta_norm(kop, "fp32", iters=20)

    def bounds(xv, relres64):
        # relres64: the final float64 residual (refinement takes it with the float64
        # operator).  Forward error <= ||r|| / lambda_min(A_mu) with lambda_min >= mu;
        # without refinement the float64 residual would only be bounded by
        # tol + ||dA|| ||x|| / ||b|| (both reported).
        nx = float(torch.linalg.norm(xv))
        return {"fwd_err_bound": relres64 * nb / mu / nx,
                "relres_fp64_bound_without_refinement": prob.tol + dA * nx / nb}

    cg = None
    if not args.no_cg:
        def cg_step():
            P0 = rr.build_precond(kop, [mu], l=0, prec="fp32")
            return P0.solve(b, tol=prob.tol, certify=False, use_graph=args.graph, check_every=8)
        for _ in range(max(args.warmup, 1)):
            cg_step()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(args.steps):
            x0, i0 = cg_step()
        torch.cuda.synchronize()
        t_cg = (time.perf_counter() - t0) / args.steps
        r0 = b - rr.apply_operator(kop, mu, "fp64", x0)
        cg = {"ms": 1e3 * t_cg, "iters": i0["iters"], "restarts": i0["restarts"],
              "relres_work": i0["relres_work"],
              "relres_fp64": float(torch.linalg.norm(r0) / torch.linalg.norm(b)),
              **bounds(x0, i0["relres_fp64"])}

    # roofline of the dominant kernel (by device time inside the timed steps).  The
    # symmetric kernel matvec evaluates the n(n+1)/2 distinct pairs once each; the
    # algorithmic work per pair is 2d flops for the distance, one for the scale and
    # two for the row and column accumulations (2d + 3 = 35 at d = 16, plus one
    # exponential), so a launch does (2d + 3) n(n+1)/2 flops, priced against the
    # float32 vector rate (157.3 TFLOP/s): bound "alu".  The kernel's own issue-slot
    # model (5 vector-ALU slots per pair once the exponents come from bf16 MFMA) is
    # reported beside it.
    pairs = n * (n + 1) / 2.0
    kmv_avg = kmv_ms / max(kmv_n, 1)
    sk_avg = sk_ms / max(sk_n, 1)
    h = _src_hash(*TRAFFIC_SOURCES)
    flops_per_launch = (2 * d + 3) * pairs
    if kmv_ms >= sk_ms:
        ach = flops_per_launch / (kmv_avg * 1e-3) / 1e12
        slot_ach = pairs / (kmv_avg * 1e-3) / 1e9
        slot_peak = PEAK_LANE_OPS / 5 / 1e9
        roof = {"kernel": "k_ksym_mma (symmetric kernel matvec, bf16-MFMA pair terms)",
                "bound": "alu", "achieved": ach, "peak": PEAK_FP32_MFMA_TFLOPS, "unit": "TFLOP/s",
                "frac": ach / PEAK_FP32_MFMA_TFLOPS, "traffic": _traffic("k_ksym_mma", h),
                "avg_ms": kmv_avg, "launches": kmv_n,
                "per_unit": f"(2d+3) = {2 * d + 3} flops per distinct pair, n(n+1)/2 pairs per launch",
                "slot_model": {"achieved": slot_ach, "peak": slot_peak, "unit": "Gpair/s",
                               "frac": slot_ach / slot_peak,
                               "per_unit": "5 vector-ALU issue slots per pair (exp2 at half rate, "
                                           "float64 widening, two float64 FMAs)"}}
    else:
        flops = 2.0 * n * n * l
        ach = flops / (sk_avg * 1e-3) / 1e12
        roof = {"kernel": "k_ksketch_bf16x2 (sketch)", "bound": "mfma", "achieved": ach,
                "peak": PEAK_BF16_TFLOPS / 2, "unit": "TFLOP/s", "frac": ach / (PEAK_BF16_TFLOPS / 2),
                "traffic": None, "avg_ms": sk_avg, "launches": sk_n,
                "per_unit": "2 n^2 l flops, run as two bf16 passes (hi, lo)"}
    k64_avg = k64_ms / max(k64_n, 1) if k64_n else None
    sketch_tflops = (2.0 * n * n * l) / (sk_avg * 1e-3) / 1e12 if sk_n else None
    kmv_gpairs = pairs / (kmv_avg * 1e-3) / 1e9 if kmv_n else None

    # the same matrix at smaller shifts (the paper's kernel-ridge runs go down to
    # mu = 1e-6 and 1e-7), where plain CG needs many more iterations
    context = []
    for mu2 in (args.context_mu or []):
        ok = (rr.RR_OK, rr.RR_ENOCONV)

        def rr_solve(m=mu2):
            P2 = rr.build_precond(kop, [m], **build_kw)
            return P2.solve(b, ok=ok, maxit=20000, **solve_kw)
        rr_solve()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        _, i2 = rr_solve()
        torch.cuda.synchronize()
        t_rr = 1e3 * (time.perf_counter() - t0)
        entry = {"mu": mu2, "randrand_ms": t_rr, "randrand_iters": i2["iters"],
                 "randrand_status": i2["rc"]}
        if not args.no_cg:
            t0 = time.perf_counter()
            P0 = rr.build_precond(kop, [mu2], l=0, prec="fp32")
            _, c2 = P0.solve(b, tol=prob.tol, certify=False, use_graph=args.graph, check_every=8,
                             maxit=20000, ok=ok)
            torch.cuda.synchronize()
            t_cg2 = 1e3 * (time.perf_counter() - t0)
            entry.update({"plain_cg_ms": t_cg2, "plain_cg_iters": c2["iters"],
                          "plain_cg_status": c2["rc"], "speedup_vs_plain_cg": t_cg2 / t_rr})
        context.append(entry)
        _log(f"context mu={mu2:g}: {entry}")

    cpu = None
    if not args.no_cpu:
        cpu = cpu_baseline(prob, last["iters"], last["restarts"], rb.build_opts().power_iters, full=args.cpu_full)

    out = {
        "metric": "time-to-rel-residual 1e-6 and solves/s vs plain CG, same GPU; HBM GB/s",
        "value": 1e3 / ms_step,
        "unit": "solves/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32-class kernel entries (bf16x3 MFMA pair terms), f64 accumulation/dots/"
                 "projections; bf16 (hi+lo) MFMA sketch; f64 kernel at restarts (refinement)",
        "data": "synthetic",
        "config": {"workload": "kernel-ridge RBF, n=50000, d=16, 10-component mixture, "
                               "median bandwidth, A=K/n, mu=1e-4, SRHT l=500, tol 1e-6",
                   "n": n, "d": d, "l": l, "mu": mu, "tol": prob.tol,
                   "parallelism": "single GPU"},
        "time_to_solution_ms": ms_step,
        "build_ms": last["ms_build"], "solve_ms": last["ms_solve"],
        "pcg_iters": last["iters"], "pcg_restarts": last["restarts"],
        "relres_work": last["relres_work"], "relres_fp64": relres_fp64,
        "relres_fp64_library": last["relres_fp64"], **bounds(x, last["relres_fp64"]),
        "delta_A_norm": dA, "fp64_refinement": True,
        "kernel_matvec_fp64_avg_ms": k64_avg, "kernel_matvec_fp64_launches": k64_n,
        "tau": last["tau"], "normE": last["normE"], "lamhat": last["lamhat"],
        "orth_err": last["orth_err"],
        "plain_cg": cg,
        "speedup_vs_plain_cg": (cg["ms"] / ms_step) if cg else None,
        "kernel_matvec_gpairs_per_s": kmv_gpairs, "kernel_matvec_avg_ms": kmv_avg,
        "sketch_tflops": sketch_tflops, "sketch_avg_ms": sk_avg,
        "context": context,
        "roofline": roof,
        "cpu_baseline": cpu,
    }
    print(json.dumps(out), flush=True)


def _host_threads():
    """Host threads the oracle may use: the CPU count, capped by OMP_NUM_THREADS."""
    n = os.cpu_count() or 1
    try:
        return max(1, min(n, int(os.environ.get("OMP_NUM_THREADS", n))))
    except ValueError:
        return n


def _log(msg):
    print(f"[bench] {msg}", file=sys.stderr, flush=True)


def bench_precision(args):
    """Stored dense Matern-3/2 on 65,536 points, mixed precision with FP64 refinement to 1e-10."""
    import numpy as np
    import torch

    import paper_2509_19747_amd as rr
    from paper_2509_19747_amd import binding as rb
    import workloads

    prob = workloads.cfg_precision()
    n, l, mu, tol = prob.n, prob.l, prob.mus[0], prob.tol
    pts = torch.from_numpy(prob.pts).cuda()
    kop = rr.kernel_operator(rr.OP_MATERN32, pts, prob.kconst, 1.0)
    A = rr.kernel_to_dense(kop, "fp64")
    dop = rr.dense_operator(A)
    b = torch.from_numpy(prob.b).cuda()
    build_kw = dict(l=l, sketch="gaussian", seed=prob.omega_seed, prec="mixed")
    _log(f"precision: n={n} l={l} matrix formed")

    def step():
        P = rr.build_precond(dop, [mu], **build_kw)
        x, info = P.solve(b, tol=tol, certify=False, maxit=20000)
        return P, x, info

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    _log("precision: warmup done")
    rb.profile_enable(True)
    t0 = time.perf_counter()
    for i in range(args.steps):
        P, x, info = step()
        _log(f"precision: step {i} iters={info['iters']} restarts={info['restarts']}")
    torch.cuda.synchronize()
    ms = 1e3 * (time.perf_counter() - t0) / args.steps
    mv_n, mv_ms = rb.profile_read(rb.PROF_DENSE_MATVEC)
    sk_n, sk_ms = rb.profile_read(rb.PROF_DENSE_SKETCH)
    rb.profile_enable(False)
    r64 = b - rr.apply_operator(dop, mu, "fp64", x)
    relres64 = float(torch.linalg.norm(r64) / torch.linalg.norm(b))
    # forward error against the stored direct solution x* (float64 dense Cholesky on
    # the host, tests/golden/make_precision_xstar.py), when this is the default size
    fwd = None
    xs_path = os.path.join(os.path.dirname(os.path.abspath(__file__)), "tests", "golden",
                           "precision_matern32_n65536_xstar.npy")
    if n == 65_536 and os.path.exists(xs_path):
        xs = np.load(xs_path)
        fwd = float(np.linalg.norm(x.cpu().numpy() - xs) / np.linalg.norm(xs))
    cg = None
    if not args.no_cg:
        t0 = time.perf_counter()
        P0 = rr.build_precond(dop, [mu], l=0, prec="mixed")
        x0, i0 = P0.solve(b, tol=tol, certify=False, maxit=20000, ok=(rr.RR_OK, rr.RR_ENOCONV))
        torch.cuda.synchronize()
        cg = {"ms": 1e3 * (time.perf_counter() - t0), "iters": i0["iters"], "status": i0["rc"],
              "relres_work": i0["relres_work"]}
    mv_avg = mv_ms / max(mv_n, 1)
    sk_avg = sk_ms / max(sk_n, 1)
    gbs = 4.0 * n * (n + 1) / 2 / (mv_avg * 1e-3) / 1e9   # the upper triangle, read once
    tflops = 2.0 * n * n * l / (sk_avg * 1e-3) / 1e12 if sk_n else None
    out = {
        "metric": "time to float64 relative residual 1e-10 (dense, mixed precision)",
        "value": 1e3 / ms, "unit": "solves/s", "ms_per_step": ms, "steps": args.steps,
        "config": {"workload": "dense Matern-3/2, n=65536 uniform points in [0,1]^3, ell=0.1, A=K, "
                               "mu=1e-5, Gaussian l=1024, bf16 sketch, f32 matvec, f64 refinement"},
        "pcg_iters": info["iters"], "restarts": info["restarts"], "relres_fp64": relres64,
        "build_ms": info["ms_build"], "solve_ms": info["ms_solve"], "tau": info["tau"],
        "forward_error_vs_direct": fwd,
        "plain_cg": cg,
        "roofline": {"kernel": "k_dense_sym<float>", "bound": "hbm", "achieved": gbs,
                     "peak": PEAK_HBM_GBS, "unit": "GB/s", "frac": gbs / PEAK_HBM_GBS,
                     "avg_ms": mv_avg, "launches": mv_n, "per_unit": "2 n (n + 1) bytes per matvec (upper triangle)"},
        "sketch": {"kernel": "k_dense_gemm_bf16", "bound": "mfma", "achieved_tflops": tflops,
                   "peak": 2500.0, "avg_ms": sk_avg},
    }
    print(json.dumps(out), flush=True)


def bench_small(args):
    """Plain float64 method at small size: stored dense RBF, n = 2,000, d = 8, mu = 1e-3,
    Gaussian l = 100, tol 1e-8; RandRAND PCG against plain CG, both float64, iteration
    batches of 16 replayed as hipGraphs."""
    import numpy as np
    import torch

    import paper_2509_19747_amd as rr
    from paper_2509_19747_amd import binding as rb
    import workloads

    prob = workloads.cfg_small_dense()
    n, l, mu, tol = prob.n, prob.l, prob.mus[0], prob.tol
    kop = rr.kernel_operator(rr.OP_RBF, torch.from_numpy(prob.pts).cuda(), prob.kconst, prob.scale)
    A = rr.kernel_to_dense(kop, "fp64")
    dop = rr.dense_operator(A)
    b = torch.from_numpy(prob.b).cuda()

    # at this size an iteration is a few microseconds of work: both solves replay their
    # iteration batches as hipGraphs, which removes most of the per-kernel launch cost
    def run(ll):
        P = rr.build_precond(dop, [mu], l=ll, sketch="gaussian", seed=prob.omega_seed, prec="fp64")
        x, info = P.solve(b, tol=tol, use_graph=True, check_every=16)
        return x, info

    def timed(ll, steps):
        for _ in range(args.warmup):
            run(ll)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(steps):
            x, info = run(ll)
        torch.cuda.synchronize()
        return 1e3 * (time.perf_counter() - t0) / steps, x, info

    rb.profile_enable(True)
    ms, x, info = timed(l, args.steps)
    mv_n, mv_ms = rb.profile_read(rb.PROF_DENSE_MATVEC64)
    rb.profile_enable(False)
    ms0, x0, info0 = timed(0, args.steps)
    r = b - rr.apply_operator(dop, mu, "fp64", x)
    relres = float(torch.linalg.norm(r) / torch.linalg.norm(b))
    mv_avg = mv_ms / max(mv_n, 1)
    gbs = 8.0 * n * n / (mv_avg * 1e-3) / 1e9
    out = {
        "metric": "time-to-rel-residual 1e-8 and solves/s vs plain CG, same GPU (float64)",
        "value": 1e3 / ms, "unit": "solves/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": ms, "higher_is_better": True, "dtype": "f64", "data": "synthetic",
        "config": {"workload": "stored dense Gaussian RBF, n=2000 points ~ N(0, I_8), bandwidth 1, "
                               "mu=1e-3, Gaussian l=100, tol 1e-8, float64", "n": n, "l": l},
        "pcg_iters": info["iters"], "restarts": info["restarts"], "relres_fp64": relres,
        "build_ms": info["ms_build"], "solve_ms": info["ms_solve"], "tau": info["tau"],
        "plain_cg": {"ms": ms0, "iters": info0["iters"], "relres_work": info0["relres_work"]},
        "speedup_vs_plain_cg": ms0 / ms,
        "roofline": {"kernel": "k_dense_matvec<double>", "bound": "hbm", "achieved": gbs,
                     "peak": PEAK_HBM_GBS, "unit": "GB/s", "frac": gbs / PEAK_HBM_GBS, "avg_ms": mv_avg,
                     "launches": mv_n, "per_unit": "8 n^2 bytes per matvec (the 32 MB matrix stays in the "
                                                 "256 MB last-level cache, so this can exceed HBM)"},
    }
    if not args.no_cpu:
        from oracle import randrand as orr
        from oracle import solvers as osol
        from oracle.operators import Operator
        op = Operator.from_problem(prob)
        t0 = time.perf_counter()
        Po = orr.build(op, [mu], l, "gaussian", prob.omega_seed)[0]
        res = osol.pcg(op.shifted(mu), Po.apply, prob.b, tol)
        t_all = time.perf_counter() - t0
        out["cpu_baseline"] = {"value": 1.0 / t_all, "unit": "solves/s", "cores": _host_threads(),
                               "kind": "oracle", "sample": f"the whole float64 oracle build and PCG solve "
                                                           f"({res.iters} iterations), timed once"}
    print(json.dumps(out), flush=True)


def bench_variants(args):
    """The paper's other solvers and preconditioner forms on the headline problem (kernel
    ridge, RBF, n = 50,000, d = 16, mu = 1e-4, tol 1e-6, float32-class entries with float64
    refinement), each timed on one GPU and checked against the float64 operator:
      * C-RandRAND with CG and with MINRES, R-RandRAND (Algorithm RandRAND_CG) with CG and
        MINRES and split R-RandRAND (Algorithm RandRAND_CG_split), all on one SRHT handle
        (l = 500; its build timed once);
      * block MINRES and block CG over 8 right-hand sides (Section 7.2.2), beside the
        per-column batched PCG on the same block;
      * the basis-less handle (Algorithm BL_RandRAND_PCG, column sampling, l = 500);
      * q = 1 (eq. testmatrix), adaptive l from 64 (eq. ad_criterion, l_max = 1,024), and
        the shifted-Cholesky sweep over the shifts 1e-3 .. 1e-6 (Section 5.1).
    Times are medians over `steps` runs after `warmup` runs."""
    import statistics

    import numpy as np
    import torch

    import paper_2509_19747_amd as rr
    from paper_2509_19747_amd import binding as rb
    import workloads

    assert torch.cuda.is_available(), "bench.py needs a GPU"
    prob = workloads.cfg_kernel_ridge()
    n, l, mu, tol = prob.n, prob.l, prob.mus[0], prob.tol
    kop = rr.kernel_operator(rr.OP_RBF, torch.from_numpy(prob.pts).cuda(), prob.kconst, prob.scale)
    b = torch.from_numpy(prob.b).cuda()
    nb = float(torch.linalg.norm(b))
    steps, warm = max(args.steps, 1), args.warmup

    def timed(fn):
        for _ in range(warm):
            fn()
        torch.cuda.synchronize()
        ts, out = [], None
        for _ in range(steps):
            t0 = time.perf_counter()
            out = fn()
            torch.cuda.synchronize()
            ts.append(1e3 * (time.perf_counter() - t0))
        return statistics.median(ts), out

    def relres64(x, m=mu, rhs=b, nrm=nb):
        return float(torch.linalg.norm(rhs - rr.apply_operator(kop, m, "fp64", x))) / nrm

    def line(info, x, **extra):
        return {"iters": info["iters"], "restarts": info["restarts"], "status": info["rc"],
                "relres_fp64": relres64(x), **extra}

    rows = {}
    rb.profile_enable(True)
    srht = dict(l=l, sketch="srht", seed=prob.omega_seed, prec="fp32")
    build_ms, P = timed(lambda: rr.build_precond(kop, [mu], **srht))
    rows["build (SRHT l=500, shared by the next six)"] = {"ms": build_ms}
    for method, krylov in (("c", "cg"), ("c", "minres"), ("r", "cg"), ("r", "minres"),
                           ("split", "cg"), ("split", "minres")):
        ms, (x, info) = timed(lambda: P.solve(b, tol=tol, method=method, krylov=krylov, certify=False,
                                              check_every=8, maxit=5000))
        label = {"c": "C", "r": "R", "split": "split R"}[method]
        rows[f"{label}-RandRAND {krylov.upper()}"] = line(info, x, ms=ms, total_ms=build_ms + ms)
        _log(f"variants: {method}/{krylov} {ms:.1f} ms, {info['iters']} iterations")

    bp = workloads.cfg_batched(nrhs=8, mus=(mu,))
    B = torch.from_numpy(np.ascontiguousarray(bp.B)).cuda()
    Pb = rr.build_precond(kop, [mu], l=l, sketch="srht", seed=bp.omega_seed, prec="fp32")
    nB = torch.linalg.norm(B, dim=0)
    for krylov in ("block_minres", "block_cg", "cg"):
        ms, (X, infos, st) = timed(lambda: Pb.solve_batch(B, [0] * 8, tol=tol, krylov=krylov, check_every=8))
        R = B - rr.apply_operator_block(kop, mu, "fp64", X.contiguous())
        rel = (torch.linalg.norm(R, dim=0) / nB).max().item()
        name = {"block_minres": "block MINRES", "block_cg": "block CG", "cg": "batched PCG (per column)"}[krylov]
        rows[f"{name}, 8 right-hand sides"] = {"ms": ms, "columns_per_s": 8e3 / ms, "status": st,
                                              "max_iters": max(i["iters"] for i in infos),
                                              "max_relres_fp64": rel}
        _log(f"variants: {krylov} x 8 {ms:.1f} ms")

    def build_solve(mus_, idx=0, **kw):
        def fn():
            Q = rr.build_precond(kop, mus_, **kw)
            x_, i_ = Q.solve(b, mu_index=idx, tol=tol, certify=False, check_every=8, maxit=5000)
            return Q, x_, i_
        return fn

    cs = dict(l=l, sketch="colsample", seed=prob.omega_seed, prec="fp32")
    ms, (Q, x, info) = timed(build_solve([mu], basis="less", **cs))
    rows["basis-less C-RandRAND (column sampling l=500), build + solve"] = line(info, x, ms=ms, total_ms=ms)
    ms, (Q, x, info) = timed(build_solve([mu], **cs))
    rows["explicit basis, same column sample, build + solve"] = line(info, x, ms=ms, total_ms=ms)
    ms, (Q, x, info) = timed(build_solve([mu], q=1, **srht))
    rows["q = 1 (Omega = A X), build + solve"] = line(info, x, ms=ms, total_ms=ms)
    ad = dict(srht, l=64, l_max=1024)
    ms, (Q, x, info) = timed(build_solve([mu], **ad))
    rows["adaptive l from 64 (l_max 1024), build + solve"] = line(info, x, ms=ms, total_ms=ms,
                                                                  l_chosen=Q.shape[1])
    mus4 = [1e-3, 1e-4, 1e-5, 1e-6]
    ms, Q = timed(lambda: rr.build_precond(kop, mus4, multi="shifted_chol", **srht))
    sweep = {"build_ms": ms}
    for k, m in enumerate(mus4):
        ms_k, (x, info) = timed(lambda: Q.solve(b, mu_index=k, tol=tol, certify=False, check_every=8,
                                                maxit=5000))
        sweep[f"mu={m:g}"] = {"ms": ms_k, "iters": info["iters"], "status": info["rc"],
                              "relres_fp64": relres64(x, m)}
    rows["shifted-Cholesky sweep, 4 shifts (one orthogonalisation)"] = sweep
    kmv_n, kmv_ms = rb.profile_read(rb.PROF_KERNEL_MATVEC)
    rb.profile_enable(False)

    kmv_avg = kmv_ms / max(kmv_n, 1)
    pairs = n * (n + 1) / 2
    ach = (2 * prob.d + 3) * pairs / (kmv_avg * 1e-3) / 1e12
    # the fastest single right-hand-side variant, build included (total_ms)
    best = min((v["total_ms"], k) for k, v in rows.items() if "total_ms" in v)
    out = {
        "metric": "time-to-rel-residual 1e-6 (build + solve) by solver and preconditioner variant",
        "value": 1e3 / best[0], "unit": "solves/s", "best": best[1], "n_gpus": 1, "steps": steps,
        "warmup": warm, "higher_is_better": True, "dtype": "f32-class kernel entries, f64 sums",
        "data": "synthetic",
        "config": {"workload": "kernel ridge RBF n=50000 d=16 mu=1e-4 tol 1e-6, float64 refinement; "
                               "solver and preconditioner variants", "n": n, "l": l},
        "variants": rows,
        "roofline": {"kernel": "k_ksym_mma (symmetric kernel matvec)", "bound": "alu", "achieved": ach,
                     "peak": PEAK_FP32_MFMA_TFLOPS, "unit": "TFLOP/s", "frac": ach / PEAK_FP32_MFMA_TFLOPS,
                     "avg_ms": kmv_avg, "launches": kmv_n, "traffic": None,
                     "per_unit": "(2d+3) = 35 flops per distinct pair, n(n+1)/2 pairs per launch"},
    }
    print(json.dumps(out), flush=True)


def bench_batched(args):
    """256 RHS x 4 shifts on the kernel-ridge matrix: one joint basis, fused batched PCG."""
    import numpy as np
    import torch

    import paper_2509_19747_amd as rr
    from paper_2509_19747_amd import binding as rb
    import workloads

    prob = workloads.cfg_batched(nrhs=args.nrhs)
    n, l = prob.n, prob.l
    pts = torch.from_numpy(prob.pts).cuda()
    kop = rr.kernel_operator(rr.OP_RBF, pts, prob.kconst, prob.scale)
    k = prob.B.shape[1]
    mus_idx = [j for j in range(len(prob.mus)) for _ in range(k)]
    B = torch.from_numpy(np.concatenate([prob.B] * len(prob.mus), axis=1)).cuda()
    m = B.shape[1]
    torch.cuda.synchronize()
    rb.profile_enable(True)
    t0 = time.perf_counter()
    P = rr.build_precond(kop, prob.mus, l=l, sketch="srht", seed=prob.omega_seed, prec="fp32")
    torch.cuda.synchronize()
    t_build = time.perf_counter() - t0
    _log(f"batched: joint basis built in {t_build:.2f} s, solving {m} columns")
    X, infos, st = P.solve_batch(B, mus_idx, tol=prob.tol, certify=False, check_every=4,
                                 ok=(rr.RR_OK, rr.RR_ENOCONV))
    torch.cuda.synchronize()
    t_total = time.perf_counter() - t0
    mm_n, mm_ms = rb.profile_read(rb.PROF_KERNEL_MATMAT)
    rb.profile_enable(False)
    iters = [i["iters"] for i in infos]
    per_mu = {str(mu): int(max(iters[j] for j in range(m) if mus_idx[j] == g))
              for g, mu in enumerate(prob.mus)}
    mm_avg = mm_ms / max(mm_n, 1)
    tflops = 12.0 * n * n * m / (mm_avg * 1e-3) / 1e12   # six bf16 piece products
    ok = sum(1 for i in infos if i["status"] == rr.RR_OK)
    out = {
        "metric": "columns solved per second (batched multi-RHS, multi-shift)",
        "value": m / t_total, "unit": "columns/s", "total_s": t_total, "build_s": t_build,
        "columns": m, "converged": ok, "max_iters_per_mu": per_mu,
        "config": {"workload": f"kernel-ridge RBF n={n}, d=16, {k} RHS x 4 shifts "
                               "{1e-3,1e-4,1e-5,1e-6}, joint SRHT basis l=500, tol 1e-6"},
        "roofline": {"kernel": "k_kgemm_bf16x6 (fused K*P, exact bf16 pieces, float64 sums)", "bound": "mfma",
                     "achieved": tflops, "peak": PEAK_BF16_TFLOPS, "unit": "TFLOP/s",
                     "frac": tflops / PEAK_BF16_TFLOPS, "avg_ms": mm_avg, "launches": mm_n},
    }
    print(json.dumps(out), flush=True)


def bench_serving(args):
    """Poisson stream of independent RBF ridge problems through rr_serve."""
    import numpy as np

    from paper_2509_19747_amd import binding as rb
    import workloads

    stream = workloads.serving_stream(num=args.requests, rate=args.rate)
    reqs = []
    for r in stream:
        p = r.problem
        reqs.append(dict(kind=p.kind, pts=p.pts, kconst=p.kconst, scale=p.scale, mu=p.mus[0],
                         l=p.l, seed=p.omega_seed, B=p.B, t_arrival=r.t_arrival))
    kw = dict(build=dict(prec="fp32", sketch="gaussian"), solve=dict(tol=1e-6, certify=False))
    _log(f"serving: {len(reqs)} requests generated")
    res, stats = rb.serve(reqs, hbm_budget=int(args.budget_gb * (1 << 30)), max_slots=args.slots,
                          graph_iters=args.graph_iters, grouped=args.lanes, **kw)
    lat = np.array([r["t_done"] - q["t_arrival"] for r, q in zip(res, reqs) if r is not None])
    warm = 200 if len(lat) > 400 else 0
    ok = sum(1 for r in res if r is not None and r["info"]["status"] == 0)
    infos = [r["info"] for r in res if r is not None]
    out = {
        "metric": "serving latency and throughput at a Poisson arrival rate",
        "value": stats["solves_per_s"], "unit": "solves/s",
        "p50_ms": float(np.percentile(lat[warm:], 50) * 1e3),
        "p99_ms": float(np.percentile(lat[warm:], 99) * 1e3), "server_stats": stats,
        "requests": len(reqs), "ok": ok, "rate": args.rate, "slots": args.slots,
        "graph_iters": args.graph_iters, "lanes": args.lanes,
        "mean_build_ms": float(np.mean([i["ms_build"] for i in infos])),
        "mean_solve_ms": float(np.mean([i["ms_solve"] for i in infos])),
        "mean_iters": float(np.mean([i["iters"] for i in infos])),
        "config": {"workload": "RBF ridge requests, n log-uniform [1000, 32768], d in {4,8,16}, "
                               "mu log-uniform [1e-6, 1e-2], l=ceil(n/32), 1-8 RHS, tol 1e-6"},
    }
    print(json.dumps(out), flush=True)
    if args.dump:
        with open(args.dump, "w") as f:
            for q, r in zip(reqs, res):
                if r is not None:
                    i = r["info"]
                    f.write(json.dumps({"n": q["pts"].shape[1], "d": q["pts"].shape[0], "l": q["l"],
                                        "nrhs": q["B"].shape[1], "mu": q["mu"],
                                        "t_arrival": q["t_arrival"], "t_done": r["t_done"],
                                        "ms_build": i["ms_build"], "ms_solve": i["ms_solve"],
                                        "iters": i["iters"], "status": i["status"]}) + "\n")


if __name__ == "__main__":
    main()
