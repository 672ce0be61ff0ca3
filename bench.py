#!/usr/bin/env python3
"""Benchmark of the ELBM hot path on one MI355X.

Workload: D3Q27 entropic LBM Taylor-Green vortex, 512^3 periodic sites, FP32
population storage, FP64 site arithmetic, u0 = 0.05, Re = 1600 (beta from
nu = u0 L / Re, L = n / (2 pi)), closed-form alpha (Eqs. (8)-(9)).  One step
= one launch of the fused pull-stream + collide kernel over the whole box,
with the per-step counters (accepted alpha = 2, alpha range, mass, momentum)
on.  Inputs are resident in HBM before the timed region.

Prints ONE JSON line on stdout: MLUPS (value), the HBM roofline of the step
kernel, the Newton-alpha and BGK comparisons on the same box, a second timing
window late in the run (t near 5000), the serving streams, and the CPU
oracle timed on a bounded sample of the same workload.

    python bench.py [--steps K] [--warmup W] [--n 512]
    python bench.py --lattice d2q9 --n 4096 --only closed ...   (profiling
        runs of the D2Q9 kernels: the doubly periodic shear layer, Re = 3e4)
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import platform
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "MLUPS & % HBM roofline, closed-form vs Newton α; p50/p99 batched latency"
HBM_PEAK_GBS = 8000.0
BYTES = {"f64": 8, "f32": 4, "f32dev": 4, "f16dev": 2}
# site arithmetic: (dtype of the JSON line, description)
ARITH = {"fp64": ("f64", "FP64"), "mixed": ("f32+f64", "mixed (FP32 on deviations, FP64 alpha)"),
         "fp32": ("f32", "FP32")}


def log(msg: str) -> None:
    print(f"[bench {time.strftime('%H:%M:%S')}] {msg}", file=sys.stderr, flush=True)


# Sources that make up the step kernels (host runtime and server excluded).
STEP_KERNEL_SOURCES = ("elbm_internal.hpp", "elbm_site.hpp", "elbm_pull.hpp",
                       "elbm_step_impl.hpp",
                       "elbm_step_d1.hip", "elbm_step_d2.hip", "elbm_step_d3.hip",
                       "elbm_step_fused.hip")


def kernel_source_hash() -> str:
    """Hash of the step kernels' sources and compile flags: a stored counter
    measurement is used only while this hash is unchanged."""
    from paper_1904_00866_amd import build as B
    h = hashlib.sha256(" ".join(f for f in B.flags() if not f.startswith("-I")).encode())
    csrc = os.path.join(ROOT, "paper_1904_00866_amd", "csrc")
    for name in STEP_KERNEL_SOURCES:
        with open(os.path.join(csrc, name), "rb") as fh:
            h.update(name.encode() + b"\0" + fh.read())
    return h.hexdigest()[:16]


def measured_traffic(workload_key: str):
    """HBM bytes per launch from the committed rocprofv3 counter summary, if
    it was taken on the current kernel sources (else None)."""
    path = os.path.join(ROOT, "profiles", f"step_{workload_key.replace('d3q27_', 'd3q27_n')}_traffic.json")
    try:
        with open(path) as fh:
            rec = json.load(fh).get(workload_key)
    except (OSError, ValueError):
        return None
    if not rec or rec.get("source_hash") != kernel_source_hash():
        return None
    return rec.get("bytes_per_launch")


def roofline(elbm, box, storage, mode, arith, diag, ms, steps, traffic) -> dict:
    """The state's traffic in a timed call of `steps` steps of `ms` each: a
    launch reads and writes every population once, whether it takes one step or
    several.  traffic: counter bytes of a single step's launch, if known."""
    lattice, dims = box
    cfg = elbm.make_config(lattice, *dims, storage=storage, mode=mode, fp64=arith, diag=diag)
    launches = elbm.batch_launches([cfg], [steps])
    D, Q = elbm.lattice_dq(cfg.lattice)
    alg_bytes = 2 * Q * BYTES[storage] * dims[0] * dims[1] * dims[2]
    achieved = alg_bytes * launches / (ms * 1e-3 * steps) / 1e9
    single = launches == steps
    return {"bound": "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS,
            "unit": "GB/s", "frac": round(achieved / HBM_PEAK_GBS, 4),
            "traffic": traffic if single else None,
            "algorithmic_bytes_per_launch": alg_bytes,
            "steps_per_launch": round(steps / launches, 3),
            "kernel": (f"k_step<{D},Store{storage},{mode},{arith}>" if single else
                       f"k_fused<Store{storage},{mode},{arith}>, the last step k_step")}


def _window(torch, sim, steps):
    """ms per step of `steps` steps, from HIP events on the launch stream."""
    t0 = torch.cuda.Event(enable_timing=True)
    t1 = torch.cuda.Event(enable_timing=True)
    t0.record(sim.stream)
    sim.step(steps)
    t1.record(sim.stream)
    torch.cuda.synchronize()
    return t0.elapsed_time(t1) / steps


def time_mode(elbm, torch, box, storage, beta, mode, steps, warmup, diag, rho, u, arith="fp64",
              late_to=0, late_steps=50, checkpoint=None):
    """Warm-up, then one timed window of `steps` steps; with late_to > 0 the
    run continues (untimed) to t = late_to and times a second window of
    late_steps steps there.  With checkpoint = (blob, t) the simulation
    starts from that stored state (elbm_import) instead of t = 0."""
    lattice, dims = box
    sim = elbm.Simulation(lattice, *dims, rho0=rho, u0=u, device="cuda:0",
                          storage=storage, beta=beta, mode=mode, diag=diag,
                          root_max_iter=200, fp64=arith)
    if checkpoint is not None:
        sim.import_(*checkpoint)
    sim.step(warmup)
    torch.cuda.synchronize()
    w0 = time.perf_counter()
    t_start = sim.t
    ms = _window(torch, sim, steps)
    wall = time.perf_counter() - w0
    stats = sim.stats() if diag & elbm.DIAG_COUNTS else None
    if stats is not None:
        stats["t_start"] = t_start
    late = None
    if late_to > sim.t + late_steps:
        sim.step(late_to - late_steps - sim.t)
        torch.cuda.synchronize()
        ckpt = sim.export()  # the late state, for the comparison modes
        t_late = sim.t
        late_ms = _window(torch, sim, late_steps)
        late = {"t_start": t_late, "steps": late_steps, "ms_per_step": round(late_ms, 4),
                "stats": sim.stats() if diag & elbm.DIAG_COUNTS else None,
                "checkpoint": ckpt}
    sim.close()
    del sim
    torch.cuda.empty_cache()
    return ms, wall, stats, late


def cpu_model() -> str:
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return platform.processor() or platform.machine()


def cpu_baseline(n_full, beta, budget_s=10.0):
    """The FP64 oracle as it stands, OpenMP over sites, on a 128^3 sample of
    the same Taylor-Green workload, for about budget_s seconds on the host
    threads this process may use (at most 16, the host share of one GPU on a
    shared box), then on one thread."""
    import oracle
    from paper_1904_00866_amd import workloads as Wk
    nproc = os.cpu_count() or 1
    try:
        allowed = len(os.sched_getaffinity(0))
    except AttributeError:
        allowed = nproc
    cores = max(1, min(allowed, 16))
    m = 128
    rho, u = Wk.taylor_green_3d(m)
    cfg = oracle.Config(D=3, nx=m, ny=m, nz=m, beta=beta, nthreads=cores)
    f = oracle.init(cfg, rho, u)
    steps, t0 = 0, time.perf_counter()
    while True:
        f, _, _ = oracle.step(cfg, f)
        steps += 1
        el = time.perf_counter() - t0
        if el >= budget_s or steps >= 200:
            break
    closed = m ** 3 * steps / el / 1e6
    # the Newton comparison on the same state, for a third of the budget
    cfgn = oracle.Config(D=3, nx=m, ny=m, nz=m, beta=beta, mode="newton", nthreads=cores)
    nsteps, t0 = 0, time.perf_counter()
    while True:
        f, _, _ = oracle.step(cfgn, f)
        nsteps += 1
        eln = time.perf_counter() - t0
        if eln >= budget_s / 3 or nsteps >= 100:
            break
    newton = m ** 3 * nsteps / eln / 1e6
    # one thread, the same sample, about a fifth of the budget
    cfg1 = oracle.Config(D=3, nx=m, ny=m, nz=m, beta=beta, nthreads=1)
    s1, t0 = 0, time.perf_counter()
    while True:
        f, _, _ = oracle.step(cfg1, f)
        s1 += 1
        el1 = time.perf_counter() - t0
        if el1 >= budget_s / 5 or s1 >= 20:
            break
    single = m ** 3 * s1 / el1 / 1e6
    model = cpu_model()
    return {"value": round(closed, 3), "unit": "MLUPS", "cores": cores,
            "kind": "oracle",
            "sample": f"D3Q27 Taylor-Green {m}^3 (of the {n_full}^3 workload), closed-form "
                      f"alpha, FP64, {steps} steps in {el:.1f} s on {cores} threads "
                      f"({model}; nproc {nproc}, {allowed} allowed to this process); then "
                      f"Newton alpha, {nsteps} steps in {eln:.1f} s; then closed form on one "
                      f"thread, {s1} steps in {el1:.1f} s",
            "cpu_model": model, "nproc": nproc, "cores_allowed": allowed,
            "single_core_value": round(single, 3),
            "newton_value": round(newton, 3), "closed_over_newton": round(closed / newton, 2)}


def _serving_summary(res, rate):
    return {"n_req": res["n_req"], "rate_per_s": rate, "completed": res["completed"],
            "failed": res["failed"], "p50_s": round(res["p50_s"], 3),
            "p99_s": round(res["p99_s"], 3), "mean_s": round(res["mean_s"], 3),
            "queue_wait_p50_s": round(res["queue_p50_s"], 3),
            "queue_wait_p99_s": round(res["queue_p99_s"], 3),
            "aggregate_mlups": round(res["mlups"], 1), "span_s": round(res["span_s"], 2),
            "site_updates": res["site_updates"], "rounds": res["rounds"],
            "launches": res["launches"], "max_resident": res["max_resident"],
            "submit_lag_max_s": round(res["submit_lag_max_s"], 4)}


def serving_block(args) -> dict:
    """Two seeded Poisson streams of D2Q9 shear-layer requests through the
    continuous-batching server: the overloaded stream (arrivals faster than
    the GPU can serve) and one below capacity; eight sampled requests rerun
    alone and compared with their in-mix results."""
    import numpy as np
    import torch

    from paper_1904_00866_amd import serving
    from paper_1904_00866_amd import workloads as Wk

    max_active, round_steps = 64, 50
    reqs = Wk.serving_stream(args.serving_requests, rate=args.serving_rate)
    rng = np.random.default_rng(1)
    cand = [r["k"] for r in reqs if r["n"] <= 1024]
    sample = sorted(int(k) for k in rng.choice(cand, size=min(8, len(cand)), replace=False))
    log(f"serving: {len(reqs)} requests at {args.serving_rate}/s")
    res = serving.run_stream(reqs, max_active=max_active, round_steps=round_steps,
                             keep=sample, log=log)
    log(f"serving: p50 {res['p50_s']:.2f} s, p99 {res['p99_s']:.2f} s, "
        f"{res['mlups']:.0f} MLUPS")
    diff = 0.0
    for k in sample:
        r0, u0 = serving.run_alone(reqs[k])
        o = res["outputs"][k]
        diff = max(diff, (o[0] - r0).abs().max().item(), (o[1] - u0).abs().max().item())
    del res["outputs"]
    torch.cuda.empty_cache()
    out = {"workload": "D2Q9 doubly periodic shear layers, u0=0.04, kappa=80, delta=0.05; "
                       "edge uniform in {128,256,512,1024,2048}, Re log-uniform [1e3,1e5], "
                       "steps uniform [1000,20000], storage uniform {f32,f16dev}, "
                       "closed-form alpha, nu=0.04 n/Re; seeded Poisson arrivals",
           "seed": 20250101, "max_active": max_active, "round_steps": round_steps,
           "pool_bytes": res["pool_bytes"],
           "stream": _serving_summary(res, args.serving_rate),
           "alone_vs_mix": {"requests": sample, "max_abs_diff_rho_u": diff}}
    if args.serving_steady_requests > 0:
        reqs2 = Wk.serving_stream(args.serving_steady_requests, rate=args.serving_steady_rate,
                                  seed=20250102)
        log(f"serving: {len(reqs2)} requests at {args.serving_steady_rate}/s")
        res2 = serving.run_stream(reqs2, max_active=max_active, round_steps=round_steps,
                                  log=log)
        log(f"serving: p50 {res2['p50_s']:.2f} s, p99 {res2['p99_s']:.2f} s")
        del res2["outputs"]
        out["steady_stream"] = dict(_serving_summary(res2, args.serving_steady_rate),
                                    seed=20250102)
    return out


def main() -> int:
    ap = argparse.ArgumentParser(description=__doc__.split("\n\n")[0])
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=200)
    ap.add_argument("--warmup", type=int, default=20)
    ap.add_argument("--lattice", default="d3q27", choices=["d3q27", "d2q9"],
                    help="d3q27: the 3-D Taylor-Green vortex n^3 (the benchmark); d2q9: the "
                         "doubly periodic shear layer n^2 (Re = 3e4), for profiling runs")
    ap.add_argument("--n", type=int, default=None,
                    help="box edge (default 512 for d3q27, 4096 for d2q9)")
    ap.add_argument("--late-t", type=int, default=5000,
                    help="also time a window of 50 closed-form steps ending at t = late_t "
                         "(the end of the 5000-step workload; 0: skip)")
    ap.add_argument("--storage", default="f32", choices=sorted(BYTES))
    ap.add_argument("--arith", default="fp64", choices=sorted(ARITH),
                    help="site arithmetic: fp64 (default), or for the closed form mixed "
                         "(FP32 on the deviations, FP64 alpha) or fp32")
    ap.add_argument("--compare-steps", type=int, default=10)
    ap.add_argument("--no-compare", action="store_true")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--only", default=None, choices=["closed", "newton", "bisect", "bgk"],
                    help="time one alpha mode only (profiling runs)")
    ap.add_argument("--serving-requests", type=int, default=200,
                    help="requests of the Poisson serving stream (0: skip serving)")
    ap.add_argument("--serving-rate", type=float, default=20.0)
    ap.add_argument("--serving-steady-requests", type=int, default=120)
    ap.add_argument("--serving-steady-rate", type=float, default=6.2,
                    help="arrival rate of the second stream: its 120 requests (seed "
                         "20250102) average 8.5e9 site updates, so 6.2/s offers 5.3e10 "
                         "site updates per second, about 0.7 of the 7.5e10 the overloaded "
                         "stream reaches")
    ap.add_argument("--copy-probe-mib", type=int, default=0,
                    help="also run one device copy of this many MiB (a known-size kernel "
                         "that calibrates hardware byte counters in profiling runs)")
    args = ap.parse_args()
    if args.arith != "fp64" and args.only != "closed":
        print("--arith mixed / fp32 is built for the closed form: add --only closed",
              file=sys.stderr)
        return 2
    world = int(os.environ.get("WORLD_SIZE", "1"))
    if args.gpus != 1 or world != 1:
        print(f"bench.py measures one GPU only (got --gpus {args.gpus}, WORLD_SIZE {world}); "
              "the multi-GPU domain decomposition is a design, not a built path.",
              file=sys.stderr)
        return 2

    import numpy as np  # noqa: F401
    import torch

    from paper_1904_00866_amd import elbm
    from paper_1904_00866_amd import workloads as Wk

    if not torch.cuda.is_available():
        print("bench.py needs a GPU", file=sys.stderr)
        return 1
    elbm.lib()
    if args.copy_probe_mib > 0:
        a = torch.ones(args.copy_probe_mib * 2 ** 18, dtype=torch.float32, device="cuda:0")
        b = torch.empty_like(a)
        b.copy_(a)
        torch.cuda.synchronize()
        log(f"copy probe: {args.copy_probe_mib} MiB read + {args.copy_probe_mib} MiB written")
        del a, b
        torch.cuda.empty_cache()
    storage = args.storage
    three_d = args.lattice == "d3q27"
    n = args.n or (512 if three_d else 4096)
    if three_d:
        N, Q, dims = n ** 3, 27, (n, n, n)
        beta = Wk.tgv3d_beta(n)
        log(f"building {n}^3 Taylor-Green fields")
        rho, u = Wk.taylor_green_3d(n)
        workload = (f"D3Q27 ELBM Taylor-Green vortex {n}^3 periodic, u0=0.05, Re=1600")
    else:
        N, Q, dims = n * n, 9, (n, n, 1)
        beta = Wk.shear_beta(n)
        log(f"building {n}^2 shear-layer fields")
        rho, u = Wk.shear_layer(n)
        workload = (f"D2Q9 ELBM doubly periodic shear layer {n}^2, u0=0.04, kappa=80, "
                    f"delta=0.05, Re=3e4")
    box = (args.lattice, dims)
    diag = elbm.DIAG_COUNTS
    results = {}
    modes = [args.only] if args.only else (["closed"] if args.no_compare
                                           else ["closed", "bgk", "newton"])
    for mode in modes:
        steps = args.steps if mode in ("closed", "bgk") else args.compare_steps
        warm = args.warmup if mode in ("closed", "bgk") else 2
        late_to = args.late_t if (mode == "closed" and not args.only and three_d) else 0
        log(f"{mode}: warmup {warm}, timing {steps} steps"
            + (f", then a window ending at t = {late_to}" if late_to else ""))
        ms, wall, st, late = time_mode(elbm, torch, box, storage, beta, mode, steps, warm, diag,
                                       rho, u, args.arith, late_to=late_to)
        results[mode] = dict(ms=ms, wall=wall, stats=st, steps=steps, late=late)
        log(f"{mode}: {ms:.3f} ms/step, {N / ms / 1e3:.0f} MLUPS"
            + (f"; at t = {late['t_start']}: {late['ms_per_step']:.3f} ms/step" if late else ""))
    # Newton on the closed form's late state (the same state as its late
    # window): the comparison where the flow has developed
    late = results.get("closed", {}).get("late")
    if late and "newton" in results:
        ckpt = late.pop("checkpoint")
        log(f"newton on the state at t = {ckpt[1]}: timing {args.compare_steps} steps")
        ms_n, _, st_n, _ = time_mode(elbm, torch, box, storage, beta, "newton", args.compare_steps,
                                     1, diag, rho, u, args.arith, checkpoint=ckpt)
        results["newton_late"] = dict(ms=ms_n, stats=st_n, steps=args.compare_steps)
        log(f"newton late: {ms_n:.3f} ms/step")
        del ckpt
        torch.cuda.empty_cache()
    elif late:
        late.pop("checkpoint", None)
    del rho, u

    main_mode = args.only or "closed"
    r = results[main_mode]
    ms = r["ms"]
    mlups = N / (ms * 1e-3) / 1e6
    key = f"{args.lattice}_{n}_{storage}_{main_mode}" + ("" if args.arith == "fp64"
                                                         else f"_{args.arith}")
    traffic = measured_traffic(key)
    out = {
        "metric": METRIC,
        "value": round(mlups, 1),
        "unit": "MLUPS",
        "n_gpus": 1,
        "steps": r["steps"],
        "warmup": args.warmup if main_mode in ("closed", "bgk") else 2,
        "ms_per_step": round(ms, 4),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": ARITH[args.arith][0],
        "data": "synthetic (analytic Taylor-Green initial field)",
        "config": {"workload": f"{workload}, {storage.upper()} population storage, "
                               f"{ARITH[args.arith][1]} site arithmetic, {main_mode} alpha",
                   "lattice": args.lattice.upper(), "n": n, "sites": N, "storage": storage,
                   "beta": beta, "alpha_mode": main_mode, "arithmetic": args.arith,
                   "diagnostics": "counts, recorded by the last step of the timed call"},
        "roofline": roofline(elbm, box, storage, main_mode, args.arith, diag, ms, r["steps"],
                             traffic),
    }

    def diag_of(st):
        return {"accept2_fraction": round(st["n_accept2"] / N, 4),
                "alpha_lt2_fraction": round(st["n_alpha_lt2"] / N, 4),
                "alpha_min": st["alpha_min"],
                "fallback_fraction": st["n_fallback"] / N,
                "negative_populations": st["n_negative"],
                "nonfinite_populations": st["n_nonfinite"]}

    st = r["stats"]
    if st:
        out["diagnostics"] = dict(diag_of(st), at_step=st["step"])
    late = r.get("late")
    if late:
        out["late_window"] = {"t_start": late["t_start"], "steps": late["steps"],
                              "ms_per_step": late["ms_per_step"],
                              "mlups": round(N / late["ms_per_step"] / 1e3, 1),
                              "diagnostics": diag_of(late["stats"]) if late["stats"] else None}
    if "newton" in results or "bgk" in results:
        cmp = {}
        if "newton" in results:
            rn = results["newton"]
            stn = rn["stats"]
            cmp["newton_mlups"] = round(N / rn["ms"] / 1e3, 1)
            cmp["closed_over_newton"] = round(rn["ms"] / ms, 2)
            cmp["newton_window"] = (f"t = {stn['t_start']} .. {stn['t_start'] + rn['steps']}"
                                    if stn else None)
            if stn:
                cmp["newton_iters_per_site"] = round(stn["total_iters"] / N, 3)
        if "newton_late" in results and r.get("late"):
            rl = results["newton_late"]
            stl = rl["stats"]
            cmp["late"] = {"t_start": stl["t_start"] if stl else None,
                           "closed_ms": r["late"]["ms_per_step"],
                           "newton_ms": round(rl["ms"], 4),
                           "newton_mlups": round(N / rl["ms"] / 1e3, 1),
                           "closed_over_newton": round(rl["ms"] / r["late"]["ms_per_step"], 2),
                           "newton_iters_per_site": (round(stl["total_iters"] / N, 3)
                                                     if stl else None)}
        if "bgk" in results:
            cmp["bgk_mlups"] = round(N / results["bgk"]["ms"] / 1e3, 1)
            cmp["closed_over_bgk_time"] = round(ms / results["bgk"]["ms"], 3)
        out["comparison"] = cmp
    if args.serving_requests > 0 and not args.only:
        out["serving"] = serving_block(args)
    if not args.no_cpu_baseline and not args.only:
        log("CPU oracle baseline (bounded sample)")
        out["cpu_baseline"] = cpu_baseline(n, beta)
    else:
        out["cpu_baseline"] = None
    print(json.dumps(out), flush=True)
    return 0


if __name__ == "__main__":
    sys.exit(main())
