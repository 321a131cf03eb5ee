"""Benchmark of the assembled SEM screened-Poisson operator and CG on one MI355X.

Workload: 32^3 affine hexahedra at N=7 (11,390,625 assembled DOFs, 16.8M local
nodes), lambda = 1, seeded U[-1,1) forcing.
One step = the paper's operator protocol (50 back-to-back operator calls) plus
one 100-iteration CG solve (the benchmark's fixed iteration count), all inputs
resident in HBM.  After the timed steps (outside them): 64 uneven problems
solved one by one in FP64 vs batched (FP64, and FP32 operator with FP64
residual replacement), and the serving recipe through the continuous-batching
engine vs one at a time in FP64, all to 1e-8 relative residual: its first R
arrivals, a 60 s window at 4 requests/s, and the configured 200 requests/s cut
off after 20 s of wall time.  Prints one JSON line.

  python bench.py [--gpus 1] [--steps K] [--warmup W] [--no-cpu-baseline] [--no-batch] [--serve-requests R]
                  [--no-serve-window]
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import re
import statistics
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

AX_CALLS = 50
CG_ITERS = 100
PEAK_HBM_GBS = 8000.0
FP64_PER_NODE = 97   # FP64 vector instructions of the operator per local node at N = 7
FP64_RATE = 36.5e12  # lanes of FP64 vector instructions per second (measured)
TRAFFIC_FILE = os.path.join(ROOT, "profiles", "ax_f64_box32_N7_traffic.json")
KERNEL_SOURCES = [os.path.join(ROOT, "paper_2202_12477_amd", "csrc", f) for f in ("ax_impl.h", "reduce.h", "tile.h", "walk.h")]


def kernel_hash() -> str:
    """Hash of the operator's source code with comments and white space removed, so
    the stored counter record stays valid across edits that do not change code."""
    h = hashlib.sha256()
    for f in KERNEL_SOURCES:
        src = open(f).read()
        src = re.sub(r"/\*.*?\*/", " ", src, flags=re.S)
        src = re.sub(r"//[^\n]*", " ", src)
        h.update(" ".join(src.split()).encode())
    return h.hexdigest()[:16]


def measured_traffic(schedule):
    """HBM bytes per operator launch from the committed rocprofv3 counter summary,
    or None when it is missing or was taken from a different kernel source or
    tile schedule."""
    try:
        rec = json.load(open(TRAFFIC_FILE))
    except (OSError, ValueError):
        return None
    if rec.get("kernel_hash") != kernel_hash() or rec.get("schedule") != schedule:
        return None
    return rec.get("bytes_per_launch")


def stream_rate(hb, torch, n=1 << 25, reps=20, warm=20):
    """Measured 8:1 streaming rate (GB/s), median of reps after `warm` untimed launches
    (run after the timed steps, with the device's clocks up)."""
    inp = torch.ones(8 * n, dtype=torch.float64, device="cuda")
    out = torch.empty(n, dtype=torch.float64, device="cuda")
    for _ in range(warm):
        hb.stream_probe(inp, out)
    times = []
    for _ in range(reps):
        s, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        s.record()
        hb.stream_probe(inp, out)
        e.record()
        e.synchronize()
        times.append(s.elapsed_time(e) * 1e-3)
    del inp, out
    return 9 * 8 * n / statistics.median(times) / 1e9


def host_cpu():
    """CPU model, logical CPUs of the host, and the CPUs this process may run on."""
    model = "unknown"
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                model = line.split(":", 1)[1].strip()
                break
    except OSError:
        pass
    try:
        allowed = len(os.sched_getaffinity(0))
    except AttributeError:
        allowed = os.cpu_count() or 1
    return model, os.cpu_count() or 1, allowed


def cpu_baseline(small, large, budget_s=8.0):
    """The oracle (oracle/oracle.c, plain C FP64) timed on this host's cores: its
    timing build (gcc -O3 -march=native -fopenmp, no FMA contraction; elements swept
    in 8 classes that share no node, vector loops and dot products split over the
    threads) on one thread and on every core this process may use (capped by
    OMP_NUM_THREADS when set).  Each configuration is its benchmark unit: one
    operator application plus 100 CG iterations from x0 = 0.  The one-thread run of
    the 32^3 N=7 box does as many CG iterations as fit in about budget_s seconds
    (a bounded sample, scaled per iteration); every other run is whole."""
    import numpy as np

    import oracle

    L = oracle.timing_lib(build=True)
    model, nproc, allowed = host_cpu()
    cap = int(os.environ.get("OMP_NUM_THREADS", "0") or 0)
    threads = min(allowed, cap) if cap > 0 else allowed
    out = {"cpu_model": model, "nproc": nproc, "cpus_allowed": allowed,
           "build": " ".join(["gcc", *oracle.TIMING_CFLAGS]), "configs": {}}
    for case in (small, large):
        m = oracle.Mesh(case.nx, case.ny, case.nz, case.N, jitter=case.jitter, seed=case.mesh_seed)
        b = oracle.rhs(m.NG, case.rhs_seed)
        rec = {"n_global": m.NG}
        for nt in sorted({1, threads}):
            used = L.oracle_set_threads(nt)
            t0 = time.perf_counter()
            m.ax_classes(b, case.lam, L=L)
            t_ax = time.perf_counter() - t0
            iters = case.iters
            if nt == 1 and case is large:
                iters = max(2, min(case.iters, int(budget_s / max(t_ax * 1.3, 1e-9))))
            t0 = time.perf_counter()
            r = m.cg_classes(b, case.lam, fixed_iters=iters, L=L)
            t_cg = time.perf_counter() - t0
            assert r["iters"] == iters and np.all(np.isfinite(r["res"]))
            rec[f"threads_{used}"] = {
                "ax_s": round(t_ax, 4), "ax_gdofs": round(m.NG / t_ax / 1e9, 5),
                "cg_iters_timed": iters, "cg_ms_per_iter": round(t_cg / iters * 1e3, 3),
                "cg_gdofs": round(m.NG * iters / t_cg / 1e9, 5),
                "unit_s": round(t_ax + t_cg / iters * case.iters, 3)}
        out["configs"][case.name] = rec
        del m, b
    used = L.oracle_set_threads(threads)
    best = out["configs"][large.name][f"threads_{used}"]
    one = out["configs"][large.name]["threads_1"]
    out.update({"value": best["ax_gdofs"], "unit": "GDOF/s", "cores": used, "kind": "oracle",
                "sample": f"{large.name}: one y = A x ({large.NG} DOFs) on {used} threads "
                          f"({best['ax_s']} s); beside it one thread ({one['ax_gdofs']} GDOF/s), and per "
                          f"configuration one A x plus 100 CG iterations (one thread on {large.name}: "
                          f"{one['cg_iters_timed']} iterations timed)"})
    return out


def paper_workload(hb, torch, metrics, B, n=50, N=7):
    """The paper's own single-GPU workload at N=7, for comparison with its figures
    (context, other hardware): a Dirichlet box of n^3 affine elements, (nN-1)^3 DOFs
    (42,508,549 at n=50), 50 back-to-back operator applications and 100 CG
    iterations, both FP64."""
    m = hb.Mesh(n, n, n, N, dirichlet=True)
    b = torch.empty(m.NG, dtype=torch.float64, device="cuda")
    hb.rhs_uniform(b, 3)
    y = torch.zeros_like(b)
    x = torch.empty_like(b)
    m.ax_add(1.0, b, y)
    m.cg(1.0, b, x, max_iter=10, fixed_iters=True, history=False)
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(3)]
    ev[0].record()
    for _ in range(AX_CALLS):
        m.ax_add(1.0, b, y)
    ev[1].record()
    res = m.cg(1.0, b, x, max_iter=CG_ITERS, fixed_iters=True, history=False)
    ev[2].record()
    ev[2].synchronize()
    assert res.iters == CG_ITERS and res.status == hb.HB_OK, res
    t_ax = ev[0].elapsed_time(ev[1]) * 1e-3 / AX_CALLS
    t_cg = ev[1].elapsed_time(ev[2]) * 1e-3
    gflops = metrics.ax_flops(m.E, N) / t_ax / 1e9
    out = {"workload": f"Dirichlet box {n}^3, N={N}, {m.NG} DOFs, affine, lambda=1",
           "ax_us": round(t_ax * 1e6, 1), "ax_gdofs": round(m.NG / t_ax / 1e9, 2), "ax_gflops": round(gflops, 1),
           "ax_frac_of_stream": round(metrics.ax_bytes(m.NG, m.E) / t_ax / 1e9 / B, 4),
           "ax_frac_of_paper_roofline": round(gflops / metrics.op_roofline(N, B), 4),
           "cg_gdofs": round(metrics.throughput(m.NG, CG_ITERS, 1, t_cg) / 1e9, 2),
           "cg_fom_gflops_nekbone": round(metrics.fom(m.E, N, CG_ITERS, t_cg) / 1e9, 1),
           "paper_mi250x_gcd_context": {"ax_gflops_n7": 1628.3, "cg_fom_gflops_n7_42.5M": 896.5,
                                        "cg_gdofs_n7_42.5M": 4.58}}
    m.close()
    return out


def small_config(hb, torch, inputs, reps=5):
    """The small configuration (4^3 jittered hexahedra, N=3, 2197 DOFs): one operator
    application and 100 fixed CG iterations, timed as launched one kernel at a time
    and as replays of one captured 100-iteration graph (best of reps, after a warm-up);
    at this size every step is launch- and latency-bound."""
    c = inputs.PLAIN_SMALL
    m = hb.Mesh(c.nx, c.ny, c.nz, c.N, jitter=c.jitter, seed=c.mesh_seed)
    b = torch.empty(m.NG, dtype=torch.float64, device="cuda")
    hb.rhs_uniform(b, c.rhs_seed)
    x = torch.empty_like(b)
    y = torch.empty_like(b)
    out = {"workload": f"{c.nx}x{c.ny}x{c.nz} jittered box, N={c.N}, {m.NG} DOFs, lambda={c.lam}"}

    def best(fn):
        fn()
        ts = []
        for _ in range(reps):
            s, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            s.record()
            fn()
            e.record()
            e.synchronize()
            ts.append(s.elapsed_time(e) * 1e-3)
        return min(ts)

    out["ax_us"] = round(best(lambda: m.ax(c.lam, b, y)) * 1e6, 2)
    for name, gk in (("cg_us_per_iter", 0), ("cg_graph_us_per_iter", c.iters)):
        t = best(lambda: m.cg(c.lam, b, x, max_iter=c.iters, fixed_iters=True, history=False, graph_k=gk))
        out[name] = round(t / c.iters * 1e6, 2)
    m.close()
    return out


def jacobi_vs_plain(hb, torch, n=32, N=7, jitter=0.2, rtol=1e-8):
    """Jacobi-preconditioned CG beside plain CG on a deformed Dirichlet box
    (n^3 elements with jittered vertices, N=7, FP64, U[-1,1) forcing): the cost
    of one iteration (100 fixed iterations each) and the time to a relative
    residual of rtol (the diagonal is computed once per mesh and lambda, timed
    on its own)."""
    m = hb.Mesh(n, n, n, N, jitter=jitter, seed=5, dirichlet=True)
    b = torch.empty(m.NG, dtype=torch.float64, device="cuda")
    hb.rhs_uniform(b, 7)
    x = torch.empty_like(b)
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]

    def timed(**kw):
        ev[0].record()
        res = m.cg(1.0, b, x, history=False, **kw)
        ev[1].record()
        ev[1].synchronize()
        return res, ev[0].elapsed_time(ev[1]) * 1e-3

    m.cg(1.0, b, x, max_iter=5, fixed_iters=True, history=False)
    _, t_first = timed(max_iter=1, fixed_iters=True, precond=hb.PRECOND_JACOBI)  # diagonal + one iteration
    _, t_one = timed(max_iter=1, fixed_iters=True, precond=hb.PRECOND_JACOBI)
    out = {"workload": f"deformed Dirichlet box {n}^3 (vertex jitter {jitter}), N={N}, {m.NG} DOFs, lambda=1",
           "diag_ms": round(max(t_first - t_one, 0.0) * 1e3, 3)}
    for name, pc in (("cg", hb.PRECOND_NONE), ("pcg", hb.PRECOND_JACOBI)):
        res, t = timed(max_iter=CG_ITERS, fixed_iters=True, precond=pc)
        assert res.iters == CG_ITERS and res.status == hb.HB_OK, res
        out[f"{name}_ms_per_iter"] = round(t / CG_ITERS * 1e3, 4)
        res, t = timed(max_iter=20000, fixed_iters=False, rtol=rtol, precond=pc)
        assert res.status == hb.HB_OK, res
        out[f"{name}_iters_to_{rtol:g}"] = res.iters
        out[f"{name}_s_to_{rtol:g}"] = round(t, 4)
    out["time_to_solution_speedup"] = round(out[f"cg_s_to_{rtol:g}"] / out[f"pcg_s_to_{rtol:g}"], 3)
    m.close()
    return out


def two_phase_vs_fused(hb, torch, metrics, B, n, N, dirichlet, label):
    """A mesh whose operator is reproducible whatever the schedule table holds
    (HB_MESH_GATHER) beside a plain one: y = A x (50 calls each) and 100 fixed CG
    iterations, FP64.  Both results are checked against each other, and the
    reproducible ones for bit-identity between repeats."""
    out = {"workload": label}
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(3)]
    ys = {}
    for name, gather in (("fused", False), ("two_phase", True)):
        m = hb.Mesh(n, n, n, N, dirichlet=dirichlet, gather=gather)
        b = torch.empty(m.NG, dtype=torch.float64, device="cuda")
        hb.rhs_uniform(b, 3)
        y, y2, x = torch.empty_like(b), torch.empty_like(b), torch.empty_like(b)
        m.ax(1.0, b, y2)
        m.cg(1.0, b, x, max_iter=10, fixed_iters=True, history=False)
        ev[0].record()
        for _ in range(AX_CALLS):
            m.ax(1.0, b, y)
        ev[1].record()
        res = m.cg(1.0, b, x, max_iter=CG_ITERS, fixed_iters=True, history=False)
        ev[2].record()
        ev[2].synchronize()
        assert res.iters == CG_ITERS and res.status == hb.HB_OK, res
        t_ax = ev[0].elapsed_time(ev[1]) * 1e-3 / AX_CALLS
        t_cg = ev[1].elapsed_time(ev[2]) * 1e-3 / CG_ITERS
        nbytes = metrics.ax_bytes(m.NG, m.E)
        out[f"{name}_ax_us"] = round(t_ax * 1e6, 1)
        out[f"{name}_ax_gdofs"] = round(m.NG / t_ax / 1e9, 2)
        out[f"{name}_ax_bytes"] = int(nbytes)
        out[f"{name}_ax_frac_of_stream"] = round(nbytes / t_ax / 1e9 / B, 4)
        out[f"{name}_cg_ms_per_iter"] = round(t_cg * 1e3, 4)
        if gather:
            out["two_phase_bit_identical_repeats"] = bool(torch.equal(y, y2))
        ys[name] = y
        m.close()
    d = torch.linalg.vector_norm(ys["two_phase"] - ys["fused"]) / torch.linalg.vector_norm(ys["fused"])
    out["rel_diff_two_phase_vs_fused"] = float(f"{d.item():.3e}")
    assert d.item() <= 1e-12, d.item()
    return out


def batched_vs_sequential(hb, torch, inputs, rtol=1e-8):
    """The 64 uneven problems: one-by-one FP64 CG vs the batched solver (FP64, FP64
    with the Jacobi preconditioner, and FP32 operator with FP64 residual
    replacement without and with Jacobi, with 25-iteration segments replayed
    from captured graphs, and with tile schedules tuned at the classes' sizes --
    the first such run includes the timing, the second installs the cached
    winners), all to rtol; solves/s."""
    cases = inputs.batched_cases()
    meshes, bs = [], []
    for c in cases:
        m = hb.Mesh(c.nx, c.ny, c.nz, c.N, jitter=c.jitter, seed=c.mesh_seed, fp32=True)
        b = torch.empty(m.NG, dtype=torch.float64, device="cuda")
        hb.rhs_uniform(b, c.rhs_seed)
        meshes.append(m)
        bs.append(b)
    xs = [torch.empty_like(b) for b in bs]
    out = {"problems": len(cases), "rtol": rtol, "n_global_total": int(sum(m.NG for m in meshes))}

    def seq():
        iters = 0
        for c, m, b, x in zip(cases, meshes, bs, xs):
            r = m.cg(c.lam, b, x, max_iter=100000, fixed_iters=False, rtol=rtol, history=False)
            assert r.status == hb.HB_OK, r
            iters += r.iters
        return iters

    def batch(prec, graph_k=0, precond=hb.PRECOND_NONE, autotune=False):
        st, res = hb.batch_solve(meshes, [c.lam for c in cases], bs, xs, max_iter=100000, rtol=rtol, prec=prec,
                                 graph_k=graph_k, precond=precond, autotune=autotune)
        assert st == hb.HB_OK, [r.status for r in res]
        return sum(r.iters for r in res)

    # the autotuned runs change the FP32 table; restored afterwards
    table = {N: hb.get_schedule(N, hb.PREC_FP32_RR) for N in sorted({c.N for c in cases})}
    for name, fn in (("sequential_fp64", seq), ("batched_fp64", lambda: batch(hb.PREC_FP64)),
                     ("batched_fp64_jacobi", lambda: batch(hb.PREC_FP64, precond=hb.PRECOND_JACOBI)),
                     ("batched_fp32rr", lambda: batch(hb.PREC_FP32_RR)),
                     ("batched_fp32rr_jacobi", lambda: batch(hb.PREC_FP32_RR, precond=hb.PRECOND_JACOBI)),
                     ("batched_fp32rr_graphs", lambda: batch(hb.PREC_FP32_RR, graph_k=25)),
                     ("batched_fp32rr_autotuned", lambda: batch(hb.PREC_FP32_RR, autotune=True)),
                     ("batched_fp32rr_autotuned_again", lambda: batch(hb.PREC_FP32_RR, autotune=True))):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        iters = fn()
        torch.cuda.synchronize()
        dt = time.perf_counter() - t0
        out[name] = {"solves_per_s": round(len(cases) / dt, 3), "wall_s": round(dt, 3), "cg_iterations": iters}
        print(f"# batch {name}: {len(cases) / dt:.2f} solves/s", file=sys.stderr, flush=True)
    degrees = sorted({c.N for c in cases})
    out["autotuned_schedules_fp32"] = {N: hb.get_schedule(N, hb.PREC_FP32_RR) for N in degrees}
    for N, v in table.items():
        hb.set_schedule(N, hb.PREC_FP32_RR, v)
    out["default_schedules_fp32"] = table
    for m in meshes:
        m.close()
    return out


def served_vs_sequential(hb, torch, inputs, count, rtol=1e-8):
    """The first `count` arrivals of the serving trace through the engine (FP32
    operator with FP64 residual replacement; FP64 and FP32 with residual
    replacement, both with the Jacobi preconditioner; 64 GB budget) and one at a
    time with FP64 CG; solves/s and latency percentiles."""
    from paper_2202_12477_amd import serving

    trace = inputs.serving_trace(count)
    out = {"requests": count, "rtol": rtol, "offered_per_s": round(count / trace[-1][0], 1),
           "trace_s": round(trace[-1][0], 3), "hbm_budget_gb": 64}
    out["engine_fp32rr"] = serving.replay_engine(trace, prec=hb.PREC_FP32_RR, rtol=rtol, progress=16)
    print(f"# serving engine: {out['engine_fp32rr']}", file=sys.stderr, flush=True)
    for name, prec in (("engine_fp64_jacobi", hb.PREC_FP64), ("engine_fp32rr_jacobi", hb.PREC_FP32_RR)):
        out[name] = serving.replay_engine(trace, prec=prec, rtol=rtol, precond=hb.PRECOND_JACOBI, progress=16)
        print(f"# serving {name}: {out[name]}", file=sys.stderr, flush=True)
    table = {N: hb.get_schedule(N, hb.PREC_FP32_RR) for N in range(1, 16)}
    out["engine_fp32rr_jacobi_autotuned"] = serving.replay_engine(trace, prec=hb.PREC_FP32_RR, rtol=rtol,
                                                                  precond=hb.PRECOND_JACOBI, progress=16,
                                                                  autotune=True)
    for N, v in table.items():
        hb.set_schedule(N, hb.PREC_FP32_RR, v)
    print(f"# serving autotuned: {out['engine_fp32rr_jacobi_autotuned']}", file=sys.stderr, flush=True)
    out["sequential_fp64"] = serving.replay_sequential(trace, rtol=rtol, progress=16)
    print(f"# serving sequential: {out['sequential_fp64']}", file=sys.stderr, flush=True)
    return out


def served_window_and_overload(hb, torch, inputs, rate=4.0, window=60.0, budget=20.0, rtol=1e-8):
    """The serving recipe over its time window: (1) a 60 s window of arrivals at an
    offered rate one GPU sustains with the engine, every request served to the end
    (FP32 operator with FP64 residual replacement and the Jacobi preconditioner)
    beside one at a time in FP64; (2) the configured 200 req/s trace, cut off after
    `budget` seconds of wall time: requests completed, their latency, and the
    backlog of arrived but unfinished ones."""
    from paper_2202_12477_amd import serving

    w = inputs.serving_window(window, rate)
    win = {"offered_per_s": rate, "window_s": window, "requests": len(w), "hbm_budget_gb": 64}
    win["engine_fp32rr_jacobi"] = serving.replay_engine(w, prec=hb.PREC_FP32_RR, rtol=rtol,
                                                        precond=hb.PRECOND_JACOBI, progress=50)
    print(f"# serving window engine: {win['engine_fp32rr_jacobi']}", file=sys.stderr, flush=True)
    win["sequential_fp64"] = serving.replay_sequential(w, rtol=rtol, progress=50)
    print(f"# serving window sequential: {win['sequential_fp64']}", file=sys.stderr, flush=True)
    trace = inputs.serving_trace(int(200 * budget * 1.2) + 64)
    over = {"offered_per_s": 200.0, "budget_s": budget, "hbm_budget_gb": 64}
    over["engine_fp32rr_jacobi"] = serving.replay_engine(trace, prec=hb.PREC_FP32_RR, rtol=rtol,
                                                         precond=hb.PRECOND_JACOBI, budget=budget)
    print(f"# serving overload engine: {over['engine_fp32rr_jacobi']}", file=sys.stderr, flush=True)
    over["sequential_fp64"] = serving.replay_sequential(trace, rtol=rtol, budget=budget)
    print(f"# serving overload sequential: {over['sequential_fp64']}", file=sys.stderr, flush=True)
    return {"window": win, "overload": over}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-batch", action="store_true", help="skip the batched-solves comparison")
    ap.add_argument("--no-jacobi", action="store_true", help="skip the Jacobi-preconditioned CG comparison")
    ap.add_argument("--no-two-phase", action="store_true", help="skip the two-phase operator comparison")
    ap.add_argument("--serve-requests", type=int, default=48,
                    help="arrivals of the serving trace to replay (0 skips the serving comparison)")
    ap.add_argument("--no-serve-window", action="store_true",
                    help="skip the 60 s serving window and the 200 req/s overload run")
    args = ap.parse_args()
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py measures one GPU only: the operator and CG of this library run on a single device "
              "(multi-GPU sharding is a design note, not built)", file=sys.stderr)
        sys.exit(2)

    import torch

    import inputs
    import paper_2202_12477_amd as hb
    from paper_2202_12477_amd import metrics

    case = inputs.PLAIN_LARGE
    torch.cuda.set_device(0)
    m = hb.Mesh(case.nx, case.ny, case.nz, case.N, jitter=case.jitter, seed=case.mesh_seed)
    NG, NL, E = m.NG, m.NL, m.E
    b = torch.empty(NG, dtype=torch.float64, device="cuda")
    hb.rhs_uniform(b, case.rhs_seed)
    y = torch.empty_like(b)
    yk = torch.zeros_like(b)
    x = torch.empty_like(b)

    def step(ev):
        ev[0].record()
        for _ in range(AX_CALLS):
            m.ax(case.lam, b, y)
        ev[1].record()
        for _ in range(AX_CALLS):
            m.ax_add(case.lam, b, yk)
        ev[2].record()
        res = m.cg(case.lam, b, x, max_iter=CG_ITERS, fixed_iters=True, history=False)
        ev[3].record()
        assert res.iters == CG_ITERS and res.status == hb.HB_OK, res

    for _ in range(args.warmup):
        step([torch.cuda.Event(enable_timing=True) for _ in range(4)])
    torch.cuda.synchronize()
    evs = []
    t0 = time.perf_counter()
    for _ in range(args.steps):
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
        step(ev)
        evs.append(ev)
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    t_ax = sum(e[0].elapsed_time(e[1]) for e in evs) * 1e-3
    t_kern = sum(e[1].elapsed_time(e[2]) for e in evs) * 1e-3
    t_cg = sum(e[2].elapsed_time(e[3]) for e in evs) * 1e-3
    t_step = sum(e[0].elapsed_time(e[3]) for e in evs) * 1e-3
    B = stream_rate(hb, torch)

    ax_gdofs = NG * AX_CALLS * args.steps / t_ax / 1e9
    kern_s = t_kern / (AX_CALLS * args.steps)
    ax_bytes = metrics.ax_bytes(NG, E)
    achieved = ax_bytes / kern_s / 1e9
    schedule = hb.get_schedule(case.N, hb.PREC_FP64)
    traffic = measured_traffic(schedule)
    out = {
        "metric": "Ax GDOF/s",
        "value": round(ax_gdofs, 3),
        "unit": "GDOF/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(t_step / args.steps * 1e3, 3),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64",
        "data": "synthetic",
        "config": {"workload": "box32_N7_affine: 32^3 hex elements, N=7, 11,390,625 DOFs, lambda=1, "
                               "U[-1,1) forcing; step = 50 operator calls + 100 CG iterations",
                   "E": E, "N": case.N, "n_global": NG, "n_local": NL},
        "roofline": {"bound": "hbm", "achieved": round(achieved, 1), "peak": PEAK_HBM_GBS, "unit": "GB/s",
                     "frac": round(achieved / PEAK_HBM_GBS, 4), "traffic": traffic,
                     "kernel": f"ax_kernel<{case.N},0,double,false,false,1> and halo_add_kernel",
                     "kernel_us": round(kern_s * 1e6, 2), "algorithmic_bytes": int(ax_bytes),
                     "fp64_issue_frac": round(FP64_PER_NODE * NL / FP64_RATE / kern_s, 4)},
        "ax_gdofs_kernel_only": round(NG / kern_s / 1e9, 3),
        "ax_gflops": round(metrics.ax_flops(E, case.N) / kern_s / 1e9, 1),
        "cg_gdofs": round(NG * CG_ITERS * args.steps / t_cg / 1e9, 3),
        "cg_ms_per_iter": round(t_cg / (CG_ITERS * args.steps) * 1e3, 4),
        "cg_fom_gflops_nekbone": round(metrics.fom(E, case.N, CG_ITERS * args.steps, t_cg) / 1e9, 1),
        "stream_8to1_gbs": round(B, 1),
        "frac_of_stream": round(achieved / B, 4),
        "wall_s": round(wall, 3),
    }
    m.close()
    del b, y, yk, x
    out["small_config"] = small_config(hb, torch, inputs)
    out["paper_workload"] = paper_workload(hb, torch, metrics, B)
    if not args.no_jacobi:
        out["jacobi"] = jacobi_vs_plain(hb, torch)
    if not args.no_two_phase:
        out["two_phase"] = [
            two_phase_vs_fused(hb, torch, metrics, B, case.nx, case.N, False,
                               f"{case.nx}^3 affine box, N={case.N}, {NG} DOFs"),
            two_phase_vs_fused(hb, torch, metrics, B, 50, 7, True, "Dirichlet box 50^3, N=7, 42508549 DOFs")]
    if not args.no_batch:
        out["batch"] = batched_vs_sequential(hb, torch, inputs)
    if args.serve_requests > 0:
        out["serving"] = served_vs_sequential(hb, torch, inputs, args.serve_requests)
    if not args.no_serve_window:
        out["serving_window"] = served_window_and_overload(hb, torch, inputs)
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(inputs.PLAIN_SMALL, case)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
