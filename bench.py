"""Throughput of the signed-particle Wigner branching random walk on one MI355X.

python bench.py [--gpus 1] [--steps K] [--warmup W] [--no-cpu] [--no-forms]

Headline workload: the Gaussian barrier V = 0.3 exp(-x^2/2) with 1e7 initial
signed particles (capacity 2e8), dt = 0.1, annihilation every 10 steps on a
2000 x 512 grid over x in [-200,200), k in [-8,8), density on 2000 bins, sp1
(pair generation).  A timed step is one time step of every particle (clock,
free flight, jumps and offspring families); every 10th step is followed by the
annihilation and the density readout, which are inside the timed region.
value = sum over timed steps of the particles held at the start of the step,
divided by the wall time.  Inputs are resident on the GPU before timing starts.

Roofline: the whole step against HBM, with a model of 34 algorithmic bytes per
particle-step (read x, k, id; write x; the offspring records and the parents'
signs), timed by HIP events around every launch group of up to five steps on
the launch stream inside the timed region.  That is a rate of work, not of
memory: a launch group reads x, k and id once for its steps and moves fewer
bytes.  `measured` is the HBM rate itself, from the bytes that the counters of
the committed profile give for these kernel sources (left out if the sources
have changed since); what bounds the step is issue (the integer products of the
clock words, the jumps' dependent FP64 chains).  The same steps are then run again with events around every kernel, for the per-kernel split
(`kernels`, with the dominant kernel named).

Printed: one JSON line on stdout (everything else goes to stderr).
"""
import argparse
import hashlib
import json
import multiprocessing as mp
import os
import platform
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0   # MI355X HBM3E
ANN_EVERY = 10
STEP_MODEL_BYTES = 34   # algorithmic bytes per particle-step of the 1D sp1 step
# the placement launch's first block closes the steps (tallies, counts, the next plan)
STEP_KERNELS = (("family", "k_walk"), ("place", "k_place"))
TRAFFIC_SOURCES = ("wbrw_walk.hpp", "wbrw_step.hpp", "wbrw_math.hpp", "wbrw_dev.hpp")


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def run_form(P, torch, cfg, steps, warmup, every=ANN_EVERY, use_graph=False, density=True,
             autotune=False, adjoint=None):
    """Runs warmup (and the autotuner), then `steps` timed steps; returns a dict
    of measurements.  adjoint: {"snapshot_every": S} times the differentiation
    form: forward steps with a checkpoint every S steps, then the density and
    its backward pass (the vector-Jacobian kernel) inside the timed region."""
    s = torch.cuda.Stream()
    sim = P.Simulation(cfg, stream=s)
    done = 0
    tuned = None
    snap_every = (adjoint or {}).get("snapshot_every", 0)
    nbins = cfg["density"]["nbins"]
    g = torch.linspace(-1.0, 1.0, nbins, dtype=torch.float64, device="cuda").reshape(1, nbins)
    g = g.expand(sim.B, nbins).contiguous()
    held = {}

    def advance(n):
        # stretches up to the next annihilation or checkpoint, one call each
        nonlocal done
        end = done + n
        while done < end:
            m = end - done
            for q in (every, snap_every):
                if q:
                    m = min(m, q - done % q)
            sim.run(m, every)
            done += m
            if every and done % every == 0 and density and not adjoint:
                sim.density()
            if snap_every and done % snap_every == 0:
                held["snap"] = sim.snapshot()      # the latest checkpoint is kept

    advance(warmup)
    if autotune:
        # tune on a state an annihilation is due on (the binning is timed on
        # it): `every` steps after the last one
        while every and done % every != every - 1:
            advance(1)
        if every:
            sim.step(1)
        tuned = sim.autotune(1)
        done = sim.stats(0)["step"]
        # re-align with the annihilation schedule before timing
        while every and done % every:
            advance(1)
    s.synchronize()

    def timed(n, marks):
        ps0 = sum(sim.stats(b)["particle_steps"] for b in range(sim.B))
        if marks:
            sim.profile(True, steps_only=(marks == "steps"))
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        if use_graph:
            sim.run(n, every, use_graph=True)
        else:
            advance(n)
        if adjoint:
            sim.density()
            held["grad"] = sim.density_vjp(g)
        s.synchronize()
        torch.cuda.synchronize()
        wall = time.perf_counter() - t0
        prof = sim.profile_read() if marks else None
        if marks:
            sim.profile(False)
        return wall, sum(sim.stats(b)["particle_steps"] for b in range(sim.B)) - ps0, prof

    # the timed region: exactly `steps` steps, with two HIP events per launch group
    # (none inside a graph replay)
    wall, ps, step_prof = timed(steps, None if use_graph else "steps")
    # the same number of steps again with HIP events around every kernel
    _, ps_prof, prof = timed(steps, "all")
    stats = [sim.stats(b) for b in range(sim.B)]
    out = {"wall_s": wall, "particle_steps": int(ps), "rate": ps / wall,
           "prof_particle_steps": int(ps_prof), "steps": steps,
           "n_end": int(sum(st["n"] for st in stats)), "profile": prof, "step_profile": step_prof,
           "sim": sim, "tuned": tuned, "sim_launch": sim.launch()}
    return out


def copy_rate(torch):
    """Read+write rate of a plain 1 GiB device-to-device copy on the same GPU
    (torch's copy kernel, HIP events): what a streaming kernel can reach on
    this part in practice, beside the nominal peak."""
    a = torch.empty(1 << 27, dtype=torch.float64, device="cuda")
    b = torch.empty_like(a)
    a.fill_(1.0)
    b.copy_(a)
    torch.cuda.synchronize()
    best = None
    for _ in range(3):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(4):
            b.copy_(a)
        e1.record()
        torch.cuda.synchronize()
        gbs = 4 * 2 * (1 << 30) / (e0.elapsed_time(e1) * 1e-3) / 1e9
        best = gbs if best is None else max(best, gbs)
    del a, b
    torch.cuda.empty_cache()
    return best


def measured_traffic():
    """Per-kernel HBM bytes per particle-step of the step from the committed
    counter summary, only if it was taken on the current kernel sources."""
    path = os.path.join(ROOT, "profiles", "step_traffic_gaussian_barrier_1e7.json")
    if not os.path.exists(path):
        return None
    info = json.load(open(path))
    h = hashlib.sha256()
    for f in TRAFFIC_SOURCES:
        h.update(open(os.path.join(ROOT, "paper_1709_02121_amd", "csrc", f), "rb").read())
    if info.get("source_sha256") != h.hexdigest():
        return None
    return info.get("hbm_bytes_per_particle_step")


def step_roofline(res):
    """Roofline of the whole step: STEP_MODEL_BYTES per particle-step over the
    mean step time of the timed region (HIP events around each launch group),
    with the per-kernel split of the profiled pass."""
    sp = res["step_profile"]
    if not sp or sp["step"][1] == 0:
        return None
    step_ms, nsteps = sp["step"]
    ps_step = res["particle_steps"] / nsteps
    avg_step_s = step_ms * 1e-3 / nsteps
    bytes_step = STEP_MODEL_BYTES * ps_step
    achieved = bytes_step / avg_step_s / 1e9
    prof = res["profile"]
    kern = {}
    total = sum(prof[st][0] for st, _ in STEP_KERNELS)
    for st, name in STEP_KERNELS:
        ms, n = prof[st]
        if n == 0:
            continue
        kern[name] = {"avg_launch_us": round(ms * 1e3 / n, 2), "us_per_step": round(ms * 1e3 / prof["step"][1], 2)
                      if prof["step"][1] else None, "share": round(ms / total, 4)}
    dominant = max(kern, key=lambda k: kern[k]["avg_launch_us"])
    out = {"bound": "issue", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
           "frac": round(achieved / HBM_PEAK_GBS, 4), "traffic": None,
           "scope": "whole step: k_walk and k_place (with the closing block), up to five steps a launch",
           "kernel": dominant, "dominant_kernel": dominant,
           "avg_step_us": round(avg_step_s * 1e6, 2), "steps_timed": nsteps,
           "particle_steps_per_step": int(ps_step), "bytes_per_particle_step": STEP_MODEL_BYTES,
           "bytes_per_step": int(bytes_step),
           "note": "achieved and frac are by the model, which counts every step's reads and writes; a launch of "
                   "several steps makes them once (measured: the HBM rate by the counters)",
           "kernels": kern}
    per = measured_traffic()
    if per:
        out["traffic"] = int(sum(per.values()) * ps_step)
        gbs = out["traffic"] / avg_step_s / 1e9
        out["measured"] = {"GBps": round(gbs, 1), "frac": round(gbs / HBM_PEAK_GBS, 4)}
        out["traffic_per_kernel"] = {k: int(v * ps_step) for k, v in per.items()}
    return out


def _oracle_leg(args):
    """One host process: the oracle on one share of the CPU-baseline sample."""
    n0, steps, offset = args
    import workloads as W
    from oracle import oracle as O
    cfg = W.scaled(W.gaussian_barrier_large("sp1"), N0=n0, instance_offset=offset)
    sim = O.OracleSim(cfg)
    ps = 0
    t0 = time.perf_counter()
    for s in range(steps):
        ps += sim.count()
        sim.step(1)
        if (s + 1) % ANN_EVERY == 0:
            sim.annihilate()
            sim.density()
    return ps, time.perf_counter() - t0


def cpu_model():
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return platform.processor() or "unknown"


def cpu_baseline():
    """The FP64 oracle on the host: one core over the headline workload's
    physics and grid with 1e6 initial particles for 100 steps (annihilation
    and density every 10); then every core of the box's share at once, each
    process running its own instance (own random keys) of 1e6 / P particles,
    the same per-particle work."""
    from oracle import oracle as O
    O.build()
    ps, wall = _oracle_leg((1_000_000, 100, 0))
    out = {"value": round(ps / wall, 1), "unit": "particle-steps/s", "cores": 1, "kind": "oracle",
           "sample": "Gaussian barrier, 2000x512 grid, 1e6 initial particles, 100 steps with "
                     "annihilation + density every 10 (%.3g particle-steps in %.1f s)" % (ps, wall),
           "cpu": cpu_model()}
    P = max(1, min(16, os.cpu_count() or 1))
    if P > 1:
        ctx = mp.get_context("spawn")
        t0 = time.perf_counter()
        with ctx.Pool(P) as pool:
            legs = pool.map(_oracle_leg, [(1_000_000 // P, 100, p) for p in range(P)])
        wall_all = time.perf_counter() - t0
        ps_all = sum(l[0] for l in legs)
        out["all_cores"] = {"value": round(ps_all / wall_all, 1), "cores": P,
                            "sample": f"{P} processes, each 1e6/{P} particles of the same workload "
                                      f"(own instance key), 100 steps; {ps_all:.3g} particle-steps "
                                      f"in {wall_all:.1f} s of wall time"}
    return out


def run_forms(P, torch, W, args):
    """The batched, differentiation, sp2 and 4D forms (--forms selects)."""
    forms = {}
    snap = {"snapshot_every": 50}
    for name, maker, steps, warm, extra in (
            ("sp2", lambda: W.gaussian_barrier_large("sp2"), 50, 10, {}),
            ("batched_256", lambda: W.batched_barriers(), 100, 10,
             {"use_graph": True, "autotune": True}),
            ("fwd_adjoint", lambda: W.differentiation(), 50, 10, {"adjoint": snap}),
            ("fwd_adjoint_x0_deriv_pairs", lambda: W.differentiation(track_tangent=2), 50, 10,
             {"adjoint": snap}),
            ("fwd_adjoint_sp2", lambda: W.differentiation(strategy="sp2"), 50, 10, {"adjoint": snap}),
            ("helium_4d", lambda: W.helium_soft_coulomb(), 10, 0, {})):
        if args.forms != "all" and name not in args.forms.split(","):
            continue
        try:
            torch.cuda.empty_cache()
            r = run_form(P, torch, maker(), steps, warm, **extra)
            r.pop("sim")
            forms[name] = {"value": round(r["rate"], 1), "steps": steps,
                           "particle_steps": r["particle_steps"], "n_end": r["n_end"]}
            if extra.get("adjoint"):
                forms[name]["timed"] = ("forward steps (annihilation every 10, a checkpoint every "
                                        "50 steps), then the density and its backward pass")
            if r["tuned"]:
                forms[name]["autotuned"] = r["tuned"]
            log(f"{name}: {r['rate']:.4g} particle-steps/s")
        except Exception as e:   # report, never hide, a form that failed
            forms[name] = {"error": str(e)[:300]}
            log(f"{name}: FAILED {e}")

    return forms


def long_runs(P, torch, W):
    """Each configuration once at its full length: the 1e7 barrier for 1000
    steps (sp1 and sp2), the 4D model for 400 steps with resampling at the
    scheduled instants and on a particle-count threshold (when it fires and
    the particles left by each resampling, #_P^a), the batched form and the
    differentiation form (forward, a checkpoint every 50 steps, backward) for
    500 steps."""
    out = {}

    def timed(sim, fn):
        ps0 = sum(sim.stats(b)["particle_steps"] for b in range(sim.B))
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        fn()
        sim.synchronize()
        wall = time.perf_counter() - t0
        ps = sum(sim.stats(b)["particle_steps"] for b in range(sim.B)) - ps0
        return {"steps_run": int(sim.stats(0)["step"]), "wall_s": round(wall, 3),
                "value": round(ps / wall, 1), "particle_steps": int(ps),
                "n_end": int(sum(sim.stats(b)["n"] for b in range(sim.B)))}

    for strat in ("sp1", "sp2"):
        torch.cuda.empty_cache()
        sim = P.Simulation(W.gaussian_barrier_large(strat))
        r = timed(sim, lambda: (sim.run(1000, ANN_EVERY, use_graph=True), sim.density()))
        st = sim.stats()
        r.update({"escaped": int(st["escaped"]), "killed": int(st["killed"]),
                  "annihilations": int(st["annihilations"])})
        out[f"gaussian_barrier_1e7_{strat}_1000_steps"] = r
        log(f"long {strat}: {r}")
        del sim

    torch.cuda.empty_cache()
    cap, limit = 1_500_000_000, 600_000_000
    cfg = W.helium_soft_coulomb(capacity=cap)
    sim = P.Simulation(cfg)
    epochs = []

    def run4d():
        last = 0
        for s in range(cfg["steps"]):
            sim.run_adaptive(1, ANN_EVERY, limit)
            st = sim.stats()
            if st["annihilations"] != last:
                epochs.append({"step": int(st["step"]), "n_after": int(st["n"]),
                               "trigger": (int(st["step"]) % ANN_EVERY) != 0})
                last = st["annihilations"]

    r = timed(sim, run4d)
    st = sim.stats()
    r.update({"capacity": cap, "threshold": limit, "annihilations": int(st["annihilations"]),
              "triggered": int(st["triggered"]), "max_depth": int(st["max_depth"]),
              "n_after_resampling": [e["n_after"] for e in epochs],
              "triggered_at_steps": [e["step"] for e in epochs if e["trigger"]],
              "mean_n_after_resampling": round(float(np.mean([e["n_after"] for e in epochs])), 1)
              if epochs else None})
    out["helium_4d_400_steps"] = r
    log(f"long 4d: {r}")
    del sim

    torch.cuda.empty_cache()
    try:
        sim = P.Simulation(W.batched_barriers())
        out["batched_256_500_steps"] = timed(sim, lambda: sim.run(500, ANN_EVERY, use_graph=True))
        del sim
    except Exception as e:
        out["batched_256_500_steps"] = {"error": str(e)[:300]}
    log(f"long batched: {out['batched_256_500_steps']}")

    torch.cuda.empty_cache()
    cfg = W.differentiation()
    sim = P.Simulation(cfg)
    nb = cfg["density"]["nbins"]
    g = torch.linspace(-1.0, 1.0, nb, dtype=torch.float64, device="cuda").reshape(1, nb)
    held = {}

    def fwd_adj():
        for _ in range(0, cfg["steps"], cfg["snapshot_every"]):
            sim.run(cfg["snapshot_every"], ANN_EVERY)
            held["snap"] = sim.snapshot()
        sim.density()
        held["grad"] = sim.density_vjp(g)

    out["fwd_adjoint_500_steps"] = timed(sim, fwd_adj)
    out["fwd_adjoint_500_steps"]["grad"] = [float(v) for v in held["grad"][0].cpu()]
    log(f"long fwd+adjoint: {out['fwd_adjoint_500_steps']}")
    del sim
    return out


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=100)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--no-forms", action="store_true")
    ap.add_argument("--forms", default="all",
                    help="comma-separated forms to run besides the main line (default: all)")
    ap.add_argument("--calibrate", action="store_true",
                    help="first copy 1 GiB device to device (a reference for HBM byte counters)")
    ap.add_argument("--long", action="store_true",
                    help="instead of the timed line, run every configuration once at its full length")
    ap.add_argument("--no-main", action="store_true",
                    help="skip the headline workload (to profile the forms alone); value is then null")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (asked for --gpus {args.gpus}); the multi-GPU "
              "path is a design (histogram merge over RCCL) that this build does not run.",
              file=sys.stderr)
        sys.exit(2)

    # the host baseline first: its worker processes start before this process
    # has touched the GPU
    cpu = None if args.no_cpu else cpu_baseline()
    if cpu:
        log(f"cpu baseline: {cpu['value']:.4g} particle-steps/s on 1 core ({cpu['cpu']})"
            + (f"; {cpu['all_cores']['value']:.4g} on {cpu['all_cores']['cores']}" if "all_cores" in cpu else ""))

    import torch

    import paper_1709_02121_amd as P
    import workloads as W

    if not torch.cuda.is_available():
        log("no GPU visible")
        sys.exit(1)
    P.lib()
    dev = torch.cuda.get_device_properties(0)
    log(f"device: {dev.name}, {dev.multi_processor_count} CUs")

    if args.calibrate:
        a = torch.empty(1 << 27, dtype=torch.float64, device="cuda")
        b = torch.empty_like(a)
        a.fill_(1.0)
        torch.cuda.synchronize()
        b.copy_(a)
        torch.cuda.synchronize()
        log("calibration copy: 1 GiB read + 1 GiB written")
        del a, b
    if args.long:
        try:
            lr = long_runs(P, torch, W)
        except Exception as e:   # report, never hide, a run that failed
            lr = {"error": str(e)[:300]}
            log(f"long runs: FAILED {e}")
        print(json.dumps({"metric": "full-length runs", "value": None, "long_runs": lr}), flush=True)
        return
    if args.no_main:
        forms = run_forms(P, torch, W, args)
        print(json.dumps({"metric": "forms only (profiling run)", "value": None, "forms": forms}), flush=True)
        return
    cfg = W.gaussian_barrier_large("sp1")
    # the default launch shapes: the autotuner keeps them on this workload
    # (its extra steps would only start the timed region on a larger ensemble)
    main_res = run_form(P, torch, cfg, args.steps, args.warmup)
    roof = step_roofline(main_res)
    if roof is not None:
        cr = copy_rate(torch)
        roof["attainable"] = {"what": "plain 1 GiB device copy, read + write, same GPU", "GBps": round(cr, 1)}
        if "measured" in roof:
            roof["attainable"]["frac"] = round(roof["measured"]["GBps"] / cr, 4)
    log(f"sp1 1e7: {main_res['rate']:.4g} particle-steps/s, n_end={main_res['n_end']}, "
        f"profile={ {k: (round(v[0], 3), v[1]) for k, v in main_res['profile'].items()} }")
    if roof:
        log(f"step: {roof['avg_step_us']} us, {roof['achieved']} GB/s by the model ({roof['frac']} of peak), "
            f"measured {roof.get('measured')}, "
            f"dominant {roof['dominant_kernel']}")
    main_res.pop("sim")

    step_ms = sum(main_res["profile"][st][0] for st, _ in STEP_KERNELS)
    forms = {"plain_sp1": {"value": round(main_res["rate"], 1),
                           "step_kernels_only": round(main_res["prof_particle_steps"] / (step_ms * 1e-3), 1)
                           if step_ms > 0 else None,
                           "launch": main_res["sim_launch"]}}
    if not args.no_forms:
        forms.update(run_forms(P, torch, W, args))

    line = {
        "metric": "particle-steps/s at 1 GPU (plain vs batched vs fwd+adjoint) and % HBM roofline",
        "value": round(main_res["rate"], 1),
        "unit": "particle-steps/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(main_res["wall_s"] * 1e3 / args.steps, 4),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64",
        "data": "synthetic",
        "config": {"workload": "gaussian_barrier_1e7_sp1", "N0": 10_000_000, "capacity": 200_000_000,
                   "grid": "2000x512", "dt": 0.1, "annihilate_every": ANN_EVERY,
                   "density_bins": 2000, "strategy": "sp1", "parallelism": "single GPU"},
        "roofline": roof,
        "cpu_baseline": cpu,
        "forms": forms,
    }
    print(json.dumps(line), flush=True)


if __name__ == "__main__":
    main()
