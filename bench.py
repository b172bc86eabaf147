#!/usr/bin/env python3
"""Benchmark of the PDBO hot path on one MI355X.

Workload: dense QUBO, n = 10,000, Q symmetric with integer entries U{-100..100}
(diagonal included), c ~ U{-100..100}, B = 1,024 restarts, Alg. 1 with g = x^2 - x,
y_bar = 6, alpha = beta = 0.025, delta = 2^-7 and the convex-start scale s.  A
"step" is one iteration of the whole hot path over all restarts: the fused
gradient GEMM + Alg. 1 epilogue, the exact evaluation of every rounded restart
(incremental from the recorded rounding changes; in the first 64 iterations
after init the int8 GEMM for column blocks that need a full product, later a
by-rows evaluation for such restarts) and the best-of-B / incumbent update,
which runs inside the next step launch.

Prints one JSON line.  `value` is the restart-iterations/s of the fastest
mixed-precision form whose best objective after T iterations is within 0.1% of
the plain FP32 form's on every seed: B*T/t_loop with t_loop from HIP events
around a whole run of T = 2000 iterations (transient included), the median over
5 seeds after one untimed warm-up run.  Every form is listed under `forms` with
its per-seed runs, the best objective found by 1 s, a steady-state window past
the transient (--steps/--warmup) and kernel times.  The roofline is that of the
dominant kernel, the step GEMM, from HIP events around every fifth of its
launches in one whole run.  The CPU oracle baseline closes the line.

    python bench.py [--steps K] [--warmup W] [--gpus 1]
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

METRIC = "restart-iters/s + best objective at 1 s, mixed-prec vs FP32 plain, n=10k"
UNIT = "restart-iterations/s"
PEAK_TFLOPS = {"bf16": 2500.0, "fp8": 5000.0, "fp32": 157.3, "i8": 5000.0}
HBM_PEAK_GBS = 8000.0


def log(msg):
    print(f"[bench] {msg}", file=sys.stderr, flush=True)


def dense_source_hash():
    """Hash of the dense kernels' code: dense.hip and common.h with comments and
    blank space removed, so that an edit of the comments keeps a measurement."""
    import re
    h = hashlib.sha256()
    for f in ("dense.hip", "common.h"):
        src = open(os.path.join(ROOT, "paper_2509_21064_amd", "csrc", f)).read()
        src = re.sub(r"/\*.*?\*/", " ", src, flags=re.S)
        src = re.sub(r"//[^\n]*", " ", src)
        h.update(" ".join(src.split()).encode())
    return h.hexdigest()[:16]


def read_traffic(form, n, B):
    """HBM bytes per launch of the step kernel, from the committed rocprofv3
    counter summary, if it was taken on the current kernel source."""
    p = os.path.join(ROOT, "profiles", f"dense_{form}_step_n{n}_B{B}_traffic.txt")
    if not os.path.exists(p):
        return None
    kv = {}
    for line in open(p):
        for key in ("kernel code sha256[:16]", "hbm_bytes_per_launch"):
            if line.startswith(key + ":"):
                kv[key] = line[len(key) + 1:].strip()
    if kv.get("kernel code sha256[:16]") != dense_source_hash():
        return None
    try:
        return float(kv["hbm_bytes_per_launch"])
    except (KeyError, ValueError):
        return None


def run_form(P, q, s, x0s, form, args):
    """One operand form: an untimed warm-up run, then one whole run of T
    iterations per seed (fresh starting points, incumbent cleared), each timed
    with HIP events on the library's stream from before the first step to
    after the last; a run with the step kernel's launches timed (every
    time_stride-th) for the roofline; a steady-state window past the
    transient."""
    import statistics

    import torch

    import workloads as W

    B, n, T = args.B, q.n, args.T
    p = W.gda_params("qubo", B=B, T=T, scale=s, precision=form, tile=args.tile,
                     graph_chunk=args.graph_chunk)
    t0 = time.time()
    ctx = P.qubo_gda_init(q, p, x0s[0])
    init_s = time.time() - t0
    log(f"{form}: init {init_s:.1f}s (tile {ctx.tile_name})")
    ctx.step(T)  # warm-up run: first launch of every kernel, caches
    torch.cuda.synchronize()
    runs = []
    for seed, x0 in enumerate(x0s):
        ctx.restart(x0)
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        w0 = time.perf_counter()
        e0.record()
        ctx.step(T)
        e1.record()
        torch.cuda.synchronize()
        t_loop = e0.elapsed_time(e1) * 1e-3
        rec = dict(seed=seed, t_loop_s=t_loop, restart_it_per_s=B * T / t_loop)
        if seed == 0 and not args.quick:
            # the same run goes on until it has lasted 1 s, so that the best
            # objective at 1 s is read off a run that got there
            total = T
            while time.perf_counter() - w0 < 1.02:
                ctx.step(250)
                torch.cuda.synchronize()
                total += 250
            tr = ctx.trace()
            at1 = [int(F) for F, sec in zip(tr["F"], tr["sec"]) if sec <= 1.0]
            atT = [int(F) for F, t in zip(tr["F"], tr["t"]) if t <= T]
            r = ctx.result()
            rec.update(best_at_T=(atT[-1] if atT else None), best_at_1s=(at1[-1] if at1 else None),
                       iterations_in_1s_run=total, best_at_end=int(r["best_obj"]),
                       time_to_best_s=float(r["time_to_best_s"]), iter_of_best=int(r["best_iter"]))
        else:
            rec.update(best_at_T=int(ctx.result()["best_obj"]), best_at_1s=None)
        runs.append(rec)
        log(f"{form}: seed {seed} T={T} in {t_loop:.4f}s = {B * T / t_loop:.4g} restart-it/s, "
            f"best@T {rec['best_at_T']}")
    rates = [r["restart_it_per_s"] for r in runs]
    t_med = statistics.median(r["t_loop_s"] for r in runs)
    # roofline run: every time_stride-th step launch bracketed by events
    ctx.restart(x0s[0])
    ctx.timing(True, classes=[P.PDBO_K_STEP], stride=args.time_stride)
    ctx.step(T)
    k_step = ctx.kernel_time(P.PDBO_K_STEP)
    # the other kernels of the iteration past the transient, timed on their own
    ctx.timing(True, classes=[P.PDBO_K_EVAL, P.PDBO_K_INCR, P.PDBO_K_ARGMIN])
    ctx.step(args.breakdown_steps)
    k_eval = ctx.kernel_time(P.PDBO_K_EVAL)
    k_arg = ctx.kernel_time(P.PDBO_K_ARGMIN)
    k_inc = ctx.kernel_time(P.PDBO_K_INCR)
    ctx.timing(False)
    # steady-state window: W untimed, then K timed iterations, all past the
    # evaluation transient whatever W is
    ctx.step(args.warmup)
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    ctx.step(args.steps)
    e1.record()
    torch.cuda.synchronize()
    t_win = e0.elapsed_time(e1) * 1e-3
    ctx.destroy()
    out = dict(value=statistics.median(rates), ms_per_step=1e3 * t_med / T, T=T,
               runs=runs, init_s=init_s,
               step_kernel_ms=k_step[0] / max(k_step[1], 1), step_launches_timed=k_step[1],
               eval_kernel_ms=k_eval[0] / max(k_eval[1], 1), eval_launches=k_eval[1],
               eval_incr_kernel_ms=k_inc[0] / max(k_inc[1], 1),
               argmin_kernel_ms=k_arg[0] / max(k_arg[1], 1), argmin_launches=k_arg[1],
               breakdown_steps=args.breakdown_steps,
               steady_state=dict(restart_it_per_s=B * args.steps / t_win,
                                 ms_per_step=1e3 * t_win / args.steps, steps=args.steps,
                                 warmup=args.warmup, first_iteration=T + args.breakdown_steps
                                 + args.warmup + 1))
    r0 = runs[0]
    out.update(best_at_T=r0["best_at_T"], best_at_1s=r0["best_at_1s"])
    log(f"{form}: median {out['value']:.4g} restart-it/s ({out['ms_per_step']:.4f} ms/it over T={T}), "
        f"step kernel {out['step_kernel_ms']:.4f} ms avg over the run, steady state "
        f"{out['steady_state']['ms_per_step']:.4f} ms/it; incr eval {out['eval_incr_kernel_ms']:.4f} ms, "
        f"best@1s {r0['best_at_1s']}")
    return out


def cpu_baseline(q, s, x0, args):
    import numpy as np

    import workloads as W
    from oracle import gda
    from oracle import qubo as oq

    Bs = args.cpu_restarts
    prob = oq.QuboProblem(q, s)
    # size the sample to about cpu_seconds of host work: one calibration iteration first
    p1 = W.gda_params("qubo", B=Bs, T=1, scale=s)
    t0 = time.perf_counter()
    gda.run(prob, x0[:Bs], p1, T=1)
    t1 = time.perf_counter() - t0
    Ts = int(min(args.T, max(1, round(args.cpu_seconds / max(t1, 1e-3)))))
    p = W.gda_params("qubo", B=Bs, T=Ts, scale=s)
    t0 = time.perf_counter()
    gda.run(prob, x0[:Bs], p, T=Ts)
    el = time.perf_counter() - t0
    cores = os.cpu_count()
    try:
        from threadpoolctl import threadpool_info
        th = [i.get("num_threads", 0) for i in threadpool_info() if i.get("user_api") == "blas"]
        if th:
            cores = max(th)
    except Exception:
        pass
    v = Bs * Ts / el
    log(f"cpu oracle: {v:.4g} restart-it/s over {Bs} restarts x {Ts} iterations ({el:.1f}s, {cores} threads)")
    return dict(value=v, unit=UNIT, cores=cores, kind="oracle",
                sample=f"FP64 oracle (numpy/BLAS), first {Bs} of the {args.B} restarts, {Ts} "
                       f"iterations incl. exact int64 evaluation, same instance and x0; {el:.1f} s")


def _cores():
    cores = os.cpu_count()
    try:
        from threadpoolctl import threadpool_info
        th = [i.get("num_threads", 0) for i in threadpool_info() if i.get("user_api") == "blas"]
        if th:
            cores = max(th)
    except Exception:
        pass
    return cores


def _cpu_rate(problem, x0, p, Bs, seconds, T):
    """Oracle restart-iterations/s on Bs restarts, about `seconds` of host work."""
    from oracle import gda
    t0 = time.perf_counter()
    gda.run(problem, x0[:Bs], dict(p, B=Bs), T=1)
    t1 = time.perf_counter() - t0
    Ts = int(min(T, max(1, round(seconds / max(t1, 1e-3)))))
    t0 = time.perf_counter()
    gda.run(problem, x0[:Bs], dict(p, B=Bs), T=Ts)
    el = time.perf_counter() - t0
    return dict(value=Bs * Ts / el, unit=UNIT, cores=_cores(), kind="oracle",
                sample=f"FP64 oracle, {Bs} restarts x {Ts} iterations, same instance and x0; {el:.1f} s")


def workload_c2(args, P):
    """Sparse Max-Cut n=2000 (G(n,M=6000), +-1), B=256, T=5000: one persistent launch."""
    import torch

    import workloads as W
    from oracle import qubo as oq
    q = W.maxcut_c2(0)
    B, T = 256, args.T if args.T != 2000 else 5000
    x0 = W.x0_uniform(2, 0, B, q.n)
    p = W.gda_params("maxcut", B=B, T=T)
    ctx = P.qubo_gda_init(q, p, x0)
    ctx.step(T)  # warm-up run (first launch of the kernel), then the timed run from x0
    ctx.restart(x0)
    ctx.timing(True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    ctx.step(T)
    torch.cuda.synchronize()
    el = time.perf_counter() - t0
    kms, _ = ctx.kernel_time(P.PDBO_K_PERSISTENT)
    r = ctx.result()
    nnz = int(q.row_ptr[-1])
    bytes_step = 16 * q.n * B + 4 * (q.n + 1) + 8 * nnz   # x, y read+write, CSR
    out = dict(metric="restart-iterations/s, sparse Max-Cut", value=B * T / el, unit=UNIT,
               workload=f"Max-Cut G(n=2000, M=6000) +-1, CSR, B={B}, T={T}, persistent kernel",
               ms_total=1e3 * el, kernel_ms=kms, best_cut=-r["best_obj"], iter_of_best=r["best_iter"],
               effective_hbm_gbs=bytes_step * T / (kms * 1e-3) / 1e9,
               effective_hbm_frac=bytes_step * T / (kms * 1e-3) / 1e9 / HBM_PEAK_GBS,
               note="x of each restart stays in LDS for all T iterations; the algorithmic "
                    "bytes are an effective figure, HBM is touched only at the launch edges")
    if not args.no_cpu:
        out["cpu_baseline"] = _cpu_rate(oq.QuboProblem(q, 1.0), x0, p, 64, args.cpu_seconds, T)
    return out


def workload_c5(args, P):
    """Weighted random 3-SAT n=20000, m=84000, B=256, entropy g, persistent kernel;
    plus the autograd adjoint on the same formula."""
    import numpy as np
    import torch

    import workloads as W
    from oracle import maxsat as om
    f = W.maxsat_c5(0)
    s = W.maxsat_scale(f)
    B, T = 256, args.T
    x0 = W.x0_uniform(5, 0, B, f.n)
    p = W.gda_params("maxsat", B=B, T=T, scale=s)
    ctx = P.maxsat_gda_init(f, p, x0)
    ctx.step(T)  # warm-up run (first launch of the kernel), then the timed run from x0
    ctx.restart(x0)
    ctx.timing(True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    ctx.step(T)
    torch.cuda.synchronize()
    el = time.perf_counter() - t0
    kms, _ = ctx.kernel_time(P.PDBO_K_PERSISTENT)
    r = ctx.result()
    # autograd forward + backward through the hand-written adjoint
    x = torch.rand(B, f.n, device="cuda", requires_grad=True)
    y = torch.rand(B, f.n, device="cuda", requires_grad=True)
    for _ in range(2):
        P.MaxSATLagrangian.apply(x, y, ctx).sum().backward()
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    reps = 20
    for _ in range(reps):
        P.MaxSATLagrangian.apply(x, y, ctx).sum().backward()
    torch.cuda.synchronize()
    ag = (time.perf_counter() - t1) / reps
    out = dict(metric="restart-iterations/s, weighted MaxSAT", value=B * T / el, unit=UNIT,
               workload=f"weighted 3-SAT n={f.n} m={f.m} w~U{{1..10}}, B={B}, T={T}, entropy g",
               ms_total=1e3 * el, kernel_ms=kms, best_unsat_weight=r["best_obj"],
               iter_of_best=r["best_iter"], autograd_fwd_bwd_ms=1e3 * ag)
    if not args.no_cpu:
        out["cpu_baseline"] = _cpu_rate(om.MaxSatProblem(f, s), x0, p, 16, args.cpu_seconds, T)
    return out


def _timed_run(ctx, T, steps_cls, P, warm=2):
    """Wall time of T iterations from the starting point (HIP-event timed by
    the library per kernel class as well), after an untimed warm-up of `warm`
    iterations (one graph chunk records the graph) and a restart."""
    import torch
    ctx.step(warm)
    ctx.restart(None)
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    ctx.step(T)
    e1.record()
    torch.cuda.synchronize()
    return e0.elapsed_time(e1) * 1e-3


def workload_mis(args, P):
    """MIS on a d-regular graph (App. D): penalised QUBO with lam = 4, B = 10,
    y0 = 5, alpha = beta = 0.02 (tab:hyper_parameters), row-parallel CSR path."""
    import numpy as np

    import workloads as W
    from oracle import mis as om
    from oracle import qubo as oq
    n, d, B = args.mis_n, args.mis_d, 10
    T = args.T if args.T != 2000 else 10000  # the dual needs ~5000 iterations to reach y <= 0 at d = 100
    q = W.mis_qubo(n, d, 0)
    # with s = 1 the stiff all-ones direction (curvature lam d) makes the first
    # steps clip every coordinate to 0 at d = 100, and the regular graph never
    # breaks the symmetry; mis_scale documents the choice
    s = W.mis_scale(q)
    # iterations replayed as hipGraphs of 50 (two short launches each) unless
    # --graph-chunk says otherwise
    gc = args.graph_chunk or 50
    p = W.gda_params("qubo", B=B, T=T, scale=s, alpha=0.02, beta=0.02, y0=5.0, tile=2,
                     graph_chunk=gc)
    ctx = P.qubo_gda_init(q, p, None)
    el = _timed_run(ctx, T, None, P, warm=gc)
    # kernel times over a second run (timing on: launches recorded one by one)
    ctx.restart(None)
    ctx.timing(True, classes=[P.PDBO_K_STEP, P.PDBO_K_ARGMIN])
    ctx.step(T)
    k_step = ctx.kernel_time(P.PDBO_K_STEP)
    k_best = ctx.kernel_time(P.PDBO_K_ARGMIN)
    ctx.timing(False)
    r = ctx.result()
    E = q.meta["edges"]
    size, inside = om.set_size(E, r["best_x"][None])
    nnz = int(q.row_ptr[-1])
    step_ms = k_step[0] / max(k_step[1], 1)
    split = ctx.tile_name == "csr_split"  # x of a restart in LDS, entries read once per restart
    # compulsory bytes of one iteration: the CSR arrays once (one packed
    # 4-byte word per entry when n <= 65536 and |Ahat_ij| < 2^15, |Ahat_ij| at
    # most 2 max|Q_ij|; else column and value, 8 bytes), x read and written, y
    # read and written (node-major float32); the neighbour gathers (B floats
    # per nonzero) are served by the caches
    packed = n <= 65536 and 2 * int(np.abs(q.vals).max(initial=0)) < 32768
    hbm = (4 if packed else 8) * nnz + 4 * (n + 1) + 16 * n * B
    gath = 4 * (B - 1) * nnz if split else 4 * B * nnz
    out = dict(metric="restart-iterations/s, MIS (penalised QUBO, lam = 4)", value=B * T / el,
               unit=UNIT, workload=f"MIS d-regular n={n} d={d}, B={B}, T={T}, row-parallel CSR",
               ms_per_step=1e3 * el / T, step_kernel_ms=step_ms, best_kernel_ms=k_best[0] / max(k_best[1], 1),
               best_F=int(r["best_obj"]), iter_of_best=int(r["best_iter"]),
               set_size=int(size[0]) if inside[0] == 0 else None, edges_inside=int(inside[0]),
               exact=bool(r["best_obj"] == oq.objective(q, r["best_x"][None])[0]),
               roofline=dict(bound="hbm", kernel="csr_split<quad, step>" if split else "spmm_kernel<quad, step>",
                             achieved=(hbm + gath) / (step_ms * 1e-3) / 1e9, peak=HBM_PEAK_GBS,
                             unit="GB/s", frac=(hbm + gath) / (step_ms * 1e-3) / 1e9 / HBM_PEAK_GBS,
                             compulsory_bytes=hbm, gathered_bytes=gath,
                             note="achieved counts the entries read again for each restart (from L2)" if split
                             else "achieved counts the gathered bytes as well (served from L2/MALL)"))
    ctx.destroy()
    if not args.no_cpu:
        out["cpu_baseline"] = _cpu_rate(oq.QuboProblem(q, s), W.x0_uniform(6, 0, B, n), p, B,
                                        args.cpu_seconds, T)
    return out


def workload_kcut(args, P):
    """Max-3-Cut (App. B) on a G(n, M) graph with +-1 weights of the size of
    Gset's G67/G72 (n = 10,000, 20,000 edges), B = 100, y0 = 6,
    alpha = beta = 0.01 (tab:hyper_parameters)."""
    import workloads as W
    from oracle import kcut as ok
    n, M, k, B, T = 10000, 20000, 3, 100, args.T
    g = W.kcut_graph(n, M, k, rep=0)
    G = ok.Graph(g)
    gc = args.graph_chunk or 50  # hipGraphs of 50 iterations unless --graph-chunk says otherwise
    p = dict(B=B, T=T, alpha=0.01, beta=0.01, y0=6.0, delta=2.0 ** -7, scale=1.0, g="quad",
             graph_chunk=gc, seed=1)
    ctx = P.kcut_gda_init(g, p, None)
    el = _timed_run(ctx, T, None, P, warm=gc)
    ctx.restart(None)
    ctx.timing(True, classes=[P.PDBO_K_STEP, P.PDBO_K_ARGMIN, P.PDBO_K_PERSISTENT])
    ctx.step(T)
    k_step, k_pers = ctx.kernel_time(P.PDBO_K_STEP), ctx.kernel_time(P.PDBO_K_PERSISTENT)
    ctx.timing(False)
    r = ctx.result()
    nnz = int(g.row_ptr[-1])
    # one launch per iteration, or the resident kernel's launches over T
    step_ms = k_step[0] / k_step[1] if k_step[1] else k_pers[0] / T
    hbm = 8 * nnz + 4 * (n + 1) + (4 * 4 * k + 8) * n * B  # Z r/w, X r/w, y r/w
    gath = 4 * k * B * nnz
    out = dict(metric="restart-iterations/s, Max-3-Cut (softmax)", value=B * T / el, unit=UNIT,
               workload=f"Max-{k}-Cut G(n={n}, M={M}) +-1, B={B}, T={T}",
               ms_per_step=1e3 * el / T, step_kernel_ms=step_ms, best_F=int(r["best_obj"]),
               cut=int(G.total - r["best_obj"]), iter_of_best=int(r["best_iter"]),
               exact=bool(r["best_obj"] == ok.objective(G, r["best_x"][None])[0]),
               roofline=dict(bound="hbm", kernel="kcut_kernel<3, quad, step>" if k_step[1] else "kcut_resident<3, quad>",
                             achieved=(hbm + gath) / (step_ms * 1e-3) / 1e9, peak=HBM_PEAK_GBS,
                             unit="GB/s", frac=(hbm + gath) / (step_ms * 1e-3) / 1e9 / HBM_PEAK_GBS,
                             compulsory_bytes=hbm, gathered_bytes=gath,
                             note="an effective figure for the resident kernel: the state stays on "
                                  "chip" if not k_step[1] else None))
    ctx.destroy()
    if not args.no_cpu:
        out["cpu_baseline"] = _kcut_cpu_rate(G, p, n, k, args.cpu_seconds, T)
    return out


def _kcut_cpu_rate(G, p, n, k, seconds, T):
    """Max-k-Cut oracle restart-iterations/s on 10 restarts from the library's
    own start (the same Philox draws, seed 1), about `seconds` of host work."""
    from oracle import kcut as ok
    from oracle.philox import x0_philox
    Bs = 10
    Z0 = x0_philox(int(p["seed"]), Bs, n * k).reshape(Bs, n, k)
    t0 = time.perf_counter()
    ok.run(G, Z0, p, 1)
    t1 = time.perf_counter() - t0
    Ts = int(min(T, max(1, round(seconds / max(t1, 1e-3)))))
    t0 = time.perf_counter()
    ok.run(G, Z0, p, Ts)
    el = time.perf_counter() - t0
    return dict(value=Bs * Ts / el, unit=UNIT, cores=_cores(), kind="oracle",
                sample=f"FP64 oracle, {Bs} restarts x {Ts} iterations, same graph and start; {el:.1f} s")


def workload_dual(args, P):
    """Dual certificate (App. D) on the dense n = 10,000 instance: projected
    descent on L(., 6 * 1) through the INT8 step kernel, then the float64
    bound; beside the best objective of a T-iteration run."""
    import time as _t

    import torch

    import workloads as W
    q = W.qubo_c3(0, n=args.n)
    s = W.qubo_scale(q)
    p = W.gda_params("qubo", B=args.B, T=args.T, scale=s, precision="i8")
    ctx = P.qubo_gda_init(q, p, W.x0_uniform(3, 0, args.B, q.n))
    ctx.step(args.T)
    best = ctx.result()["best_obj"]
    torch.cuda.synchronize()
    t0 = _t.perf_counter()
    r = P.qubo_dual_bound(ctx, iters=args.dual_iters)
    el = _t.perf_counter() - t0
    ctx.destroy()
    return dict(metric="dual certificate (lower bound on min F)", value=r["lower_bound"],
                unit="objective", workload=f"dense QUBO n={q.n}, ybar=6, {args.dual_iters} descent "
                                           f"iterations (INT8 step kernel, one point)",
                seconds=el, best_F_at_T=int(best), gap_ratio=(best - r["lower_bound"]) / abs(best),
                frank_wolfe_gap=r["gap"], rounding_bound=r["rounding"], s_L_x=r["value"],
                higher_is_better=True)


def workload_c4(args, P):
    """64 dense QUBOs of uneven n in [500, 5000], density 1-10%, B=128 each:
    grouped launches (tiles of all instances in one launch per kernel, longest
    instances first) against per-instance launches, both replayed as hipGraphs
    of graph_chunk iterations past the evaluation transient."""
    import torch

    import workloads as W
    qs = W.batch_c4(0)
    B = 128
    gc = args.graph_chunk or 50
    ps = [W.gda_params("qubo", B=B, T=args.T, scale=W.qubo_scale(q), precision=args.c4_prec,
                       graph_chunk=gc) for q in qs]
    x0s = [W.x0_uniform(4, 0, B, q.n, i) for i, q in enumerate(qs)]
    flops = float(sum(2.0 * q.n * q.n * B for q in qs))
    steps = max(args.steps, gc)
    out = dict(metric="restart-iterations/s, batched uneven QUBO", unit=UNIT,
               workload=f"64 QUBOs n~U{{500..5000}}, density U[1%,10%], w~U{{-10..10}}, B={B}, "
                        f"{args.c4_prec}, hipGraph chunks of {gc}", flop_per_iteration=flops)
    for mode, grouped in (("grouped", 1), ("per_instance", 0)):
        ctx = P.qubo_gda_batch_init(qs, ps, x0s, grouped=grouped)
        ctx.step(max(args.warmup, 70))  # past the evaluation transient
        ctx.step(gc)  # records the graph of the steady-state iterations
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        ctx.step(steps)
        e1.record()
        torch.cuda.synchronize()
        el = e0.elapsed_time(e1) * 1e-3
        ctx.timing(True, classes=[P.PDBO_K_STEP])
        ctx.step(20)
        kms, kn = ctx.kernel_time(P.PDBO_K_STEP)
        ctx.timing(False)
        step_ms = kms / 20  # all step launches of one iteration
        out[mode] = dict(value=len(qs) * B * steps / el, ms_per_step=1e3 * el / steps,
                         step_kernels_ms_per_iteration=step_ms, step_launches_per_iteration=kn / 20,
                         tile=ctx.tile_name)
        ctx.destroy()
        log(f"c4 {mode}: {out[mode]['value']:.4g} restart-it/s, {out[mode]['ms_per_step']:.3f} ms/step, "
            f"step kernels {step_ms:.3f} ms/iteration")
    g = out["grouped"]
    t_step = g["step_kernels_ms_per_iteration"] * 1e-3
    achieved = flops / t_step / 1e12
    peak = PEAK_TFLOPS[args.c4_prec]
    # algorithmic bytes of one iteration's step launches: every instance's
    # operand copy of Ahat once (n^2 elements), and per (coordinate, restart)
    # x and y read and written (16 B), the operand shadow read by the GEMM and
    # written by the epilogue, and the rounded byte read and written
    eb = {"fp32": 4, "bf16": 2, "fp8": 1, "i8": 1}[args.c4_prec]
    nbytes = float(sum(q.n * q.n * eb + q.n * B * (16 + 2 * eb + 2) for q in qs))
    # 2 B operations per byte of Ahat: below the chip's ratio of MFMA peak to HBM
    # bandwidth, so the step launches are bound by HBM
    gbs = nbytes / t_step / 1e9
    out["roofline"] = dict(bound="hbm", kernel="dense_gemm_dma (grouped STEP)", achieved=gbs,
                           peak=HBM_PEAK_GBS, unit="GB/s", frac=gbs / HBM_PEAK_GBS,
                           bytes_per_iteration=nbytes, mfma_achieved_tflops=achieved,
                           mfma_peak_tflops=peak, mfma_frac=achieved / peak,
                           note=f"arithmetic intensity 2B/{eb} = {2 * B / eb:.0f} operations per byte of "
                                f"Ahat, below the {peak * 1e3 / HBM_PEAK_GBS:.0f} of the chip's "
                                f"{args.c4_prec} MFMA peak over its HBM bandwidth")
    out["value"] = g["value"]
    out["speedup_grouped"] = g["value"] / out["per_instance"]["value"]
    return out


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    # --steps / --warmup set the steady-state window (reported beside the
    # headline); the headline is the whole-run rate B*T/t_loop over T iterations
    ap.add_argument("--steps", type=int, default=50, help="iterations of the steady-state window")
    ap.add_argument("--warmup", type=int, default=20,
                    help="untimed iterations before the steady-state window (which starts past "
                         "the evaluation transient whatever this is)")
    ap.add_argument("--seeds", type=int, default=5,
                    help="timed whole runs per form (starting points of seeds 0..seeds-1)")
    ap.add_argument("--breakdown-steps", type=int, default=20,
                    help="steps after the roofline run that time the evaluation and argmin kernels")
    ap.add_argument("--time-stride", type=int, default=5,
                    help="in the roofline run, bracket every time-stride-th step launch with HIP events")
    ap.add_argument("--n", type=int, default=10000)
    ap.add_argument("--B", type=int, default=1024)
    ap.add_argument("--T", type=int, default=2000, help="iterations of one whole run")
    ap.add_argument("--forms", default="i8,fp8,bf16,fp32")
    ap.add_argument("--tile", type=int, default=0)
    ap.add_argument("--graph-chunk", type=int, default=0)
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--cpu-restarts", type=int, default=256)
    ap.add_argument("--cpu-seconds", type=float, default=12.0)
    ap.add_argument("--workload", default="c3",
                    choices=["c3", "c2", "c4", "c5", "mis", "kcut", "dual"],
                    help="c3 (default) is the headline dense n=10k line; the others report "
                         "the sparse, batched, MaxSAT, MIS, Max-3-Cut and dual-certificate "
                         "configurations")
    ap.add_argument("--mis-n", type=int, default=50000)
    ap.add_argument("--mis-d", type=int, default=100)
    ap.add_argument("--dual-iters", type=int, default=300)
    ap.add_argument("--c4-prec", default="bf16")
    ap.add_argument("--quick", action="store_true",
                    help="no continuation of the first run to 1 s and no CPU baseline (for runs "
                         "under the profiler)")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="only run a plain 256 MiB device copy three times (the reference for "
                         "scaling rocprofv3 FETCH_SIZE / WRITE_SIZE to bytes)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (got --gpus {args.gpus}); restarts shard trivially "
              "across GPUs but no multi-GPU path is built", file=sys.stderr)
        sys.exit(2)

    import torch

    import paper_2509_21064_amd as P
    import workloads as W

    assert torch.cuda.is_available(), "bench.py needs a GPU"
    torch.cuda.set_device(0)
    if args.copy_calibration:
        nbytes = 256 * 1024 * 1024
        src = torch.rand(nbytes // 4, device="cuda")
        dst = torch.empty_like(src)
        for _ in range(3):
            dst.copy_(src)
        torch.cuda.synchronize()
        print(json.dumps(dict(copy_bytes_per_dispatch=nbytes, dispatches=3)), flush=True)
        return
    P.load()
    if args.workload != "c3":
        fn = {"c2": workload_c2, "c4": workload_c4, "c5": workload_c5, "mis": workload_mis,
              "kcut": workload_kcut, "dual": workload_dual}[args.workload]
        res = fn(args, P)
        res.update(n_gpus=1, data="synthetic", higher_is_better=True)
        print(json.dumps(res), flush=True)
        return
    t0 = time.time()
    q = W.qubo_c3(0, n=args.n)
    s = W.qubo_scale(q)
    x0s = [W.x0_uniform(3, seed, args.B, q.n) for seed in range(args.seeds)]
    log(f"instance n={q.n} B={args.B} s={s:.2f} generated in {time.time() - t0:.1f}s")

    forms = [f for f in args.forms.split(",") if f]
    res = {f: run_form(P, q, s, x0s, f, args) for f in forms}
    flops = 2.0 * q.n * q.n * args.B
    for f, r in res.items():
        r["step_kernel_frac_of_peak"] = flops / (r["step_kernel_ms"] * 1e-3) / 1e12 / PEAK_TFLOPS[f]
    # quality: per seed, the mixed form's best objective after T iterations
    # against the plain FP32 form's on the same instance and starting points
    if "fp32" in res:
        for f, r in res.items():
            gaps = [(a["best_at_T"] - b["best_at_T"]) / abs(b["best_at_T"])
                    for a, b in zip(r["runs"], res["fp32"]["runs"])]
            r["rel_gap_best_at_T_vs_fp32"] = gaps
            r["within_0.1pct_all_seeds"] = bool(all(g <= 1e-3 for g in gaps))
    # headline: the fastest mixed-precision form within 0.1% of FP32 on every
    # seed (all forms are reported)
    mixed = [f for f in forms if f != "fp32"] or forms
    ok = [f for f in mixed if res[f].get("within_0.1pct_all_seeds", True)] or mixed
    head = max(ok, key=lambda f: res[f]["value"])
    h = res[head]
    achieved = flops / (h["step_kernel_ms"] * 1e-3) / 1e12
    traffic = read_traffic(head, q.n, args.B)
    roof = dict(bound="mfma", kernel=f"dense_gemm_dma<{head}, STEP>", achieved=achieved,
                peak=PEAK_TFLOPS[head], unit="TFLOP/s", frac=achieved / PEAK_TFLOPS[head],
                traffic=traffic, flop_per_launch=flops,
                avg_launch_ms=h["step_kernel_ms"], launches_timed=h["step_launches_timed"],
                launches_timed_every=args.time_stride,
                window=f"one whole run of T={args.T} iterations from x0 (transient included)",
                note="int8 multiply-adds count as 2 operations against the 5.0 POP/s int8 peak"
                     if head == "i8" else "")
    # Past the transient (64 iterations) the evaluation GEMM does not run; the
    # incremental kernel evaluates every restart exactly.  No roofline fraction
    # applies to either; their launch times are reported.
    ev = dict(kernel="eval_incr_kernel", incremental_kernel_ms=h["eval_incr_kernel_ms"],
              eval_gemm_launches=h["eval_launches"], eval_gemm_ms=h["eval_kernel_ms"],
              note="past the transient: exact objectives from the recorded rounding changes; the "
                   "int8 evaluation GEMM runs only in the first 64 iterations after init")
    line = dict(metric=METRIC, value=h["value"], unit=UNIT, n_gpus=1, steps=args.T,
                warmup=args.T, ms_per_step=h["ms_per_step"], higher_is_better=True,
                scaling="weak", vs_baseline=None, dtype=head, data="synthetic",
                config=dict(workload=f"dense QUBO n={q.n}, Q sym U{{-100..100}}, c U{{-100..100}}, "
                                     f"B={args.B}, T={args.T}",
                            n=q.n, B=args.B, T=args.T, scale=s, precision=head,
                            g="x^2-x", y0=6.0, alpha=0.025, beta=0.025, delta=2 ** -7),
                timing=(f"value = median over {args.seeds} seeds of B*T/t_loop, t_loop from HIP events "
                        f"around a whole run of T={args.T} iterations (after one untimed warm-up run); "
                        f"ms_per_step = median t_loop / T; steps and warmup are the timed run's T and "
                        f"the warm-up run's T; the --steps/--warmup window is steady_state"),
                steady_state=h["steady_state"],
                forms=res, roofline=roof, evaluation=ev)
    if "fp32" in res and head != "fp32":
        f32 = res["fp32"]
        line["speedup_vs_fp32"] = h["value"] / f32["value"]
        line["rel_gap_best_at_T_vs_fp32"] = h["rel_gap_best_at_T_vs_fp32"]
        if f32.get("best_at_1s") is not None and h.get("best_at_1s") is not None:
            line["rel_gap_best_at_1s_vs_fp32"] = (h["best_at_1s"] - f32["best_at_1s"]) / abs(f32["best_at_1s"])
    if not args.no_cpu and not args.quick:
        line["cpu_baseline"] = cpu_baseline(q, s, x0s[0], args)
    print(json.dumps(line), flush=True)


if __name__ == "__main__":
    main()
