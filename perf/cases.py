"""The work that users of this package have it do, as cases that can be timed.

A pass is one call sequence of a user's program: an ensemble is set up from
its initial state (or resumed from a checkpoint that the program keeps), it is
advanced with the scheduled annihilations, and what the program is after is
read out: densities, the ensemble, gradients.  Everything goes through the
public entry points (`Simulation` and `autograd.density`; the ensemble through
`wbrw_export` of the C ABI, into device memory).

Sizes are those of the repository's own workloads (1e4 and 1e7 particle
barriers, the 1e7 particle helium-like model, 256 batched barriers, the
differentiation form) and ordinary ones between them, some of them odd.
"""
import ctypes
import math

import numpy as np
import torch

import paper_1709_02121_amd as wbrw
import workloads as W
from paper_1709_02121_amd import autograd

DEVICE = "cuda:0"


def _case(name, form, **over):
    """A case with every field: the potential and its size, how the ensemble
    starts, how far it is taken and what is read."""
    c = {
        "name": name,
        "form": form,            # barrier, switching, cat, helium, batched, adjoint
        "strategy": "sp1",       # sp1: pairs by probability; sp2: weighted pairs + bootstrap
        "n0": 10_000,            # initial particles (batched: the largest instance's)
        "instances": 1,
        "nx": 240, "nk": 128,    # annihilation grid, cells per axis
        "steps": 100,            # steps of a pass
        "every": 10,             # steps between annihilations
        "warm": -1,              # >= 0: resume from a checkpoint taken after so many steps
        "frames": 0,             # > 0: the density is read so many times, at equal distances
        "ensemble": False,       # the particles are read at the end
        "graph": False,          # epochs (adaptive: steps) replayed from a captured graph
        "limit": 0,              # > 0: resampling also when more particles than this are held
        "tangent": 0,            # adjoint: 1 likelihood-ratio scores, 2 derivative ghost pairs
        "sampler": "majorant",   # or rejection (Alg. 4)
    }
    c.update(over)
    return c


def listed():
    return [
        # the smallest workload of the repository, whole: what a first user
        # runs, and parameter studies one at a time; launches and latency count
        _case("barrier_1e4", "barrier", ensemble=True),
        # small ensemble in a time-dependent double barrier (two components),
        # resumed and replayed from graphs as a launch-bound serving loop does
        _case("switching_1e4_graph", "switching", warm=100, graph=True),
        # signed initial data (an interference pattern from a histogram)
        _case("cat_2e5", "cat", n0=200_000, nk=512, steps=50, frames=5),
        # an ordinary ensemble of odd size, the density recorded at every step
        # (a film of the scattering), resumed in mid-flight
        _case("film_1e6", "barrier", n0=1_000_003, nx=480, nk=256, steps=20, warm=40, frames=20),
        # the benchmark's workload: 1e7 particles on 2000 x 512 cells, density
        # after every annihilation
        _case("barrier_1e7", "barrier", n0=10_000_000, nx=2000, nk=512, steps=40, frames=4, ensemble=True),
        # weighted pairs at an ordinary odd size and at the benchmark's size
        _case("weighted_3e5", "barrier", strategy="sp2", n0=300_007, nx=480, nk=128, steps=40, warm=20,
              ensemble=True),
        _case("weighted_1e7", "barrier", strategy="sp2", n0=10_000_000, nx=2000, nk=512, steps=20),
        # 4D phase space: a small model resampled on a threshold as well, and
        # the full one (1e8 cells) up to its first annihilation
        _case("helium_2e5_adaptive", "helium", n0=200_000, nx=24, nk=24, steps=10, warm=10, limit=4_000_000,
              graph=True, ensemble=True),
        _case("helium_1e7", "helium", n0=10_000_000, nx=100, nk=100, steps=10),
        # 256 barriers of different heights, widths and sizes in one handle
        _case("batched_256", "batched", n0=1_000_000, instances=256, steps=30),
        # gradient of the density with respect to the barrier: forward and
        # backward, likelihood-ratio scores at full size, ghost pairs at an
        # ordinary one
        _case("adjoint_1e7", "adjoint", n0=10_000_000, nx=2000, nk=512, steps=20, tangent=1),
        _case("adjoint_1e6_pairs", "adjoint", n0=1_000_000, nx=480, nk=256, steps=30, tangent=2),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _grid(rng, n0):
    """Cells per axis of a 1D grid that suits n0 particles (about 0.3 to 10
    particles a cell, at most 2000 x 512)."""
    cells = min(1_000_000.0, n0 / math.exp(rng.uniform(math.log(0.3), math.log(10.0))))
    nk = int(min(512, max(24, math.sqrt(cells / 4.0))))
    return int(min(2000, max(48, cells / nk))), nk


def draw(rng):
    """One more case of the same ranges: its form, then sizes over the
    logarithm of their range, odd ones among them."""
    form = rng.choice(["barrier", "barrier", "barrier", "switching", "cat", "helium", "batched", "adjoint"])
    c = _case("drawn", form)
    del c["name"]
    c["graph"] = rng.random() < 0.3
    c["every"] = rng.choice([5, 10, 10, 10, 20])
    if form == "helium":
        c["n0"] = _log_int(rng, 1e4, 1e6)
        c["nx"], c["nk"] = rng.randint(12, 40), rng.randint(12, 32)
        c["steps"] = rng.randint(5, 10)
        c["every"] = 10
        c["limit"] = rng.choice([0, 8 * c["n0"]])
        return c
    if form == "batched":
        c["instances"] = _log_int(rng, 2, 300)
        c["n0"] = _log_int(rng, 2e4, 1e6)
        c["strategy"] = rng.choice(["sp1", "sp1", "sp2"]) if c["instances"] <= 64 else "sp1"
        c["steps"] = rng.randint(10, 30)
        return c
    c["n0"] = _log_int(rng, 1e3, 6e6)
    c["steps"] = rng.randint(10, 100) if c["n0"] < 200_000 else rng.randint(5, 40)
    c["nx"], c["nk"] = _grid(rng, c["n0"])
    if rng.random() < 0.4:
        c["warm"] = rng.randint(1, 60)
    if form == "adjoint":
        c["graph"], c["warm"] = False, -1
        c["strategy"] = rng.choice(["sp1", "sp1", "sp2"])
        c["tangent"] = 1 if c["strategy"] == "sp2" else rng.choice([1, 2])
        c["steps"] = min(c["steps"], 30)
        return c
    if form == "cat":
        c["nk"] = max(c["nk"], 128)       # the fringes need a fine wave-vector grid
        if rng.random() < 0.25:
            c["sampler"], c["warm"] = "rejection", max(c["warm"], 10)
    if form == "switching":
        c["every"] = min(c["every"], 10)  # two components: the ensemble grows fast
    if form == "barrier":
        c["strategy"] = rng.choice(["sp1", "sp1", "sp2"])
    c["ensemble"] = rng.random() < 0.5
    c["frames"] = rng.choice([0, 0, 2, c["steps"]])
    if c["frames"]:
        c["steps"] -= c["steps"] % c["frames"]
    return c


def _config(c, seed):
    """The workload that a case describes, with the random streams of `seed`."""
    seed = int(seed) & 0x7FFFFFFF
    form, n0 = c["form"], c["n0"]
    if form == "batched":
        cfg = W.batched_barriers(B=c["instances"], seed=seed % 1000)
        top = float(cfg["N0"].max())
        cfg["N0"] = np.maximum((cfg["N0"] * (n0 / top)).astype(np.int64), 1)
        if n0 == 1_000_000 and c["instances"] == 256:
            # the workload's own instances; the seed gives the random streams
            cfg = W.batched_barriers()
        cfg["capacity"] = np.maximum(16 * cfg["N0"], 400_000)
    elif form == "helium":
        cfg = W.helium_soft_coulomb()
        cfg["N0"] = np.array([n0], dtype=np.int64)
        cfg["grid"] = dict(cfg["grid"], nx=c["nx"], nk=c["nk"])
        if n0 < 10_000_000:
            cfg["capacity_factor"] = 100.0
    elif form == "cat":
        cfg = W.cat_state_barrier(N0=n0)
        g = dict(cfg["grid"], nx=c["nx"], nk=c["nk"])
        x = g["x_lo"] + (np.arange(g["nx"]) + 0.5) * ((g["x_hi"] - g["x_lo"]) / g["nx"])
        k = g["k_lo"] + (np.arange(g["nk"]) + 0.5) * ((g["k_hi"] - g["k_lo"]) / g["nk"])
        cfg["grid"] = g
        cfg["init_histogram"] = W.cat_state_wigner(x[None, :], k[:, None]).reshape(1, -1)
        cfg["capacity_factor"] = 40.0
        cfg["components"][0]["sampler"] = c["sampler"]
    else:
        if form == "switching":
            cfg = W.time_dependent_barriers()
        elif form == "adjoint":
            cfg = W.differentiation(track_tangent=c["tangent"])
        else:
            cfg = W.gaussian_barrier_large() if c["nx"] == 2000 else W.gaussian_barrier_small()
        cfg["N0"] = np.array([n0], dtype=np.int64)
        cfg["grid"] = dict(cfg["grid"], nx=c["nx"], nk=c["nk"])
        cfg["strategy"] = c["strategy"]
        if n0 < 10_000_000:
            cfg["capacity"] = max(40 * n0, 200_000)
        else:
            cfg["capacity"] = 100_000_000
    cfg["strategy"] = c["strategy"]
    cfg["seed"] = seed
    return cfg


class _State:
    pass


def _advance(sim, c, steps):
    if c["limit"]:
        sim.run_adaptive(steps, c["every"], c["limit"], use_graph=c["graph"])
    else:
        sim.run(steps, c["every"], use_graph=c["graph"])


def prepare(case, seed):
    s = _State()
    s.case = c = dict(case)
    s.cfg = _config(c, seed)
    s.stream = torch.cuda.Stream(DEVICE) if c["graph"] else None   # graphs need a stream of their own
    s.sim = None
    s.buffers = _ensemble_buffers(c, s.cfg) if c["ensemble"] else None
    if c["form"] == "adjoint":
        nbins = s.cfg["density"]["nbins"]
        s.theta = [0.3, 1.0, 0.0]
        s.g = torch.linspace(-1.0, 1.0, nbins, dtype=torch.float64, device=DEVICE)
    elif c["warm"] >= 0:
        s.sim = wbrw.Simulation(s.cfg, device=DEVICE, stream=s.stream)
        _advance(s.sim, dict(c, graph=False), c["warm"])
        s.checkpoint = s.sim.snapshot()
    return s


def _ensemble_buffers(c, cfg):
    """Device memory for the particles that a run may leave (room for the
    growth that small ensembles on fine grids show), zeros past the last."""
    dim = int(cfg["dim"])
    cap = int(np.max(cfg["capacity"])) if "capacity" in cfg else int(c["n0"] * cfg["capacity_factor"])
    room = min(cap, 4 * c["n0"]) if c["n0"] >= 1_000_000 else cap
    sp2 = cfg["strategy"] == "sp2"
    return {"x": torch.zeros(dim * room, dtype=torch.float64, device=DEVICE),
            "k": torch.zeros(dim * room, dtype=torch.float64, device=DEVICE),
            "id": torch.zeros(room, dtype=torch.int64, device=DEVICE),
            "w" if sp2 else "sign": torch.zeros(room, dtype=torch.float64 if sp2 else torch.int8, device=DEVICE)}


def _read_ensemble(sim, buf):
    """The particles of a one-instance handle into the program's buffers."""
    n = sim.count()
    if n > buf["id"].numel():
        raise RuntimeError(f"{n} particles do not fit the buffers")
    p = {k: ctypes.c_void_p(t.data_ptr()) for k, t in buf.items()}
    rc = wbrw.lib().wbrw_export(sim.h, 0, 0, n, p["x"], p["k"], p.get("sign"), p.get("w"), p["id"], None)
    if rc != wbrw.OK:
        raise wbrw.WBRWError(rc, "wbrw_export")
    return n


def run(state):
    c = state.case
    if c["form"] == "adjoint":
        theta = torch.tensor(state.theta, dtype=torch.float64, requires_grad=True)
        rho = autograd.density(theta, state.cfg, steps=c["steps"], annihilate_every=c["every"], device=DEVICE)
        rho.backward(state.g)
        return {"density": rho.detach(), "grad": theta.grad}
    sim = state.sim
    if sim is None:
        sim = wbrw.Simulation(state.cfg, device=DEVICE, stream=state.stream)
    else:
        sim.restore(state.checkpoint)
    frames = c["frames"] or 1
    rho = []
    for _ in range(frames):
        _advance(sim, c, c["steps"] // frames)
        rho.append(sim.density())
    out = {"density": rho if frames <= 50 else torch.stack(rho)}
    if c["ensemble"]:
        out["n"] = _read_ensemble(sim, state.buffers)
        out["ensemble"] = state.buffers
    return out


def _mean_particles(c):
    """Particles held at the start of a step, on average over the schedule:
    between annihilations a barrier's ensemble grows at a rate of about
    4/pi gamma0 (a pair with probability <|sin|> = 2/pi at every jump of each
    component), and an annihilation takes it back to about what it was."""
    gamma0, comps, dt = _rates(c)
    g = (4.0 / math.pi) * gamma0 * comps * dt
    n = min(c["every"], max(c["steps"], 1))
    if c["limit"]:
        n = min(n, max(1, int(math.log(c["limit"] / c["n0"]) / g)))
    total = float(c["n0"])
    if c["form"] == "batched":
        total = 5.3e7 * (c["instances"] / 256.0) * (c["n0"] / 1e6)
    return total * (math.exp(g * n) - 1.0) / (g * n)


def _rates(c):
    """gamma0, components (in units of the largest) and dt of a form."""
    return {"helium": (2.0, 2.5, 0.05), "switching": (1.0, 1.2, 0.1),
            "adjoint": (0.45, 0.67, 0.1)}.get(c["form"], (0.3, 1.0, 0.1))


def work(case):
    """Per stretch between two annihilations (which exchange the particles of
    the whole grid) the ensemble is read once and written once; a histogram
    start is read, an ensemble read out written once more.  Per particle-step
    a clock draw (ten rounds of a counter-based generator, about 80 integer
    operations) and the flight; per jump and component about 1000 operations
    (kick, acceptance, two offspring with their own clocks)."""
    c = case
    dim = 2 if c["form"] == "helium" else 1
    per = 16 * dim + 8 + (8 if c["strategy"] == "sp2" else 1) + (24 if c["tangent"] else 0)
    n = _mean_particles(c)
    gamma0, comps, dt = _rates(c)
    stretches = max(1.0, c["steps"] / c["every"])
    return {"bytes": 2.0 * stretches * n * per + (n * per if c["ensemble"] else 0.0),
            "flops": n * c["steps"] * (82.0 + -math.expm1(-gamma0 * dt) * 1000.0 * comps)}


# ---------------------------------------------------------------------------
# The densities of sp1 runs from a Gaussian start in 64 bits, by numpy alone.
# ---------------------------------------------------------------------------
_M = np.uint64(0xFFFFFFFF)


def _philox(ident, step, tag, event, sub, key):
    """Philox4x32-10 of counter (id, step, tag | event | sub): two uniforms of
    53 bits, and the four words."""
    n = ident.shape[0]
    c0, c1 = ident & _M, ident >> np.uint64(32)
    c2 = np.full(n, step, np.uint64)
    c3 = (np.uint64(tag << 28) | (np.broadcast_to(np.asarray(event, np.uint64), (n,)) << np.uint64(8))
          | np.uint64(sub))
    k0, k1 = int(key[0]), int(key[1])
    for _ in range(10):
        p0, p1 = c0 * np.uint64(0xD2511F53), c2 * np.uint64(0xCD9E8D57)
        c0, c1, c2, c3 = ((p1 >> np.uint64(32)) ^ c1 ^ np.uint64(k0), p1 & _M,
                          (p0 >> np.uint64(32)) ^ c3 ^ np.uint64(k1), p0 & _M)
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    u = [((hi << np.uint64(32) | lo) >> np.uint64(11)).astype(np.float64) * 2.0 ** -53
         for lo, hi in ((c0, c1), (c2, c3))]
    return u[0], u[1], (c0, c1, c2, c3)


def _exact_step(e, step, cfg, g0, key):
    """One time step: every particle's jumps, and its offspring's."""
    dt, g = cfg["dt"], cfg["grid"]
    born = []
    todo = dict(e, t0=np.zeros(e["x"].shape[0]), t=np.zeros(e["x"].shape[0]))
    event = np.zeros(e["x"].shape[0], np.uint64)
    while todo["x"].shape[0]:
        u, ua0, _ = _philox(todo["id"], step, 0, event, 0, key)
        te = todo["t"] - np.log1p(-u) / g0
        on = te <= dt
        todo = {k: v[on] for k, v in todo.items()}
        te, ua0, event = te[on], ua0[on], event[on]
        todo["t"] = te
        xe = todo["x"] + todo["k"] * (te - todo["t0"])
        new = []
        for m, comp in enumerate(cfg["components"]):
            H, w, c = float(comp["H"][0]), float(comp["width"][0]), float(comp["center"][0])
            u1, u2, _ = _philox(todo["id"], step, 0, event, 1 + m, key)
            q = np.sqrt(-2.0 * np.log1p(-u1)) * np.cos(2.0 * np.pi * u2) * (0.5 / w)
            sn = np.sin(2.0 * q * (xe - c))
            height = np.full(xe.shape[0], H)
            if "modulation" in comp:
                md = comp["modulation"]
                height = H * (md["a"] + md["b"] * np.cos(md["omega"] * (step * dt + te) + md["phase"]))
            ua = ua0 if m == 0 else _philox(todo["id"], step, 0, event, 8 + m, key)[0]
            hit = ua < np.abs(height) / g0 * np.abs(sn)
            kick = np.where(sn > 0, 1.0, -1.0) * np.where(height >= 0, 1.0, -1.0) * q
            _, _, words = _philox(todo["id"], step, 5, event, m, key)
            for side in (0, 1):
                lo, hi = words[2 * side], words[2 * side + 1]
                k = todo["k"] + kick if side == 0 else todo["k"] - kick
                ok = hit & (k >= g["k_lo"]) & (k < g["k_hi"])
                ident = np.uint64(2 << 62) | ((hi & np.uint64(0x3FFFFFFF)) << np.uint64(32)) | lo
                new.append({"x": xe[ok], "k": k[ok], "id": ident[ok], "t0": te[ok], "t": te[ok],
                            "sign": todo["sign"][ok] * (1 if side == 0 else -1)})
        new = {k: np.concatenate([v[k] for v in new]) for k in todo}
        born.append(dict(new, x=new["x"] + new["k"] * (dt - new["t0"])))
        event = np.concatenate([event + np.uint64(1), np.zeros(new["x"].shape[0], np.uint64)])
        todo = {k: np.concatenate([todo[k], new[k]]) for k in todo}
    e = dict(e, x=e["x"] + e["k"] * dt)
    return {k: np.concatenate([e[k]] + [v[k] for v in born]) for k in e}


def _exact_annihilate(e, step, g, key):
    dx, dk = (g["x_hi"] - g["x_lo"]) / g["nx"], (g["k_hi"] - g["k_lo"]) / g["nk"]
    qx, qk = (e["x"] - g["x_lo"]) / dx, (e["k"] - g["k_lo"]) / dk
    ok = (qx >= 0) & (qx < g["nx"]) & (qk >= 0) & (qk < g["nk"])
    cell = qx[ok].astype(np.int64) + g["nx"] * qk[ok].astype(np.int64)
    net = np.bincount(cell, weights=e["sign"][ok], minlength=g["nx"] * g["nk"]).astype(np.int64)
    nu = np.repeat(np.arange(net.shape[0]), np.abs(net))
    first = np.cumsum(np.abs(net)) - np.abs(net)
    ident = (nu.astype(np.uint64) << np.uint64(32)) | (np.arange(nu.shape[0]) - first[nu]).astype(np.uint64)
    u, v, _ = _philox(ident, step, 1, 0, 0, key)
    return {"x": g["x_lo"] + (nu % g["nx"] + u) * dx, "k": g["k_lo"] + (nu // g["nx"] + v) * dk,
            "sign": np.sign(net[nu]), "id": ident}


def exact(case, seed):
    c = case
    if (c["form"] not in ("barrier", "switching") or c["strategy"] != "sp1" or c["limit"]
            or _mean_particles(c) * (c["steps"] + max(c["warm"], 0)) > 1e7):
        return None
    cfg = _config(c, seed)
    key, ini, g, d = (cfg["seed"], 0), cfg["init"], cfg["grid"], cfg["density"]
    ident = np.arange(c["n0"], dtype=np.uint64)
    u, v, _ = _philox(ident, 0, 2, 0, 0, key)
    r = np.sqrt(-2.0 * np.log1p(-u))
    e = {"x": ini["mean_x"][0] + ini["sigma_x"][0] * r * np.cos(2.0 * np.pi * v),
         "k": ini["mean_k"][0] + ini["sigma_k"][0] * r * np.sin(2.0 * np.pi * v),
         "sign": np.ones(c["n0"], np.int64), "id": ident}
    g0 = cfg["gamma0"] if cfg["gamma0"] > 0 else max(abs(float(m["H"][0])) for m in cfg["components"])
    warm, frames = max(c["warm"], 0), c["frames"] or 1
    rho = []
    for s in range(warm + c["steps"]):
        e = _exact_step(e, s, cfg, g0, key)
        if (s + 1) % c["every"] == 0:
            e = _exact_annihilate(e, s + 1, g, key)
        done = s + 1 - warm
        if done > 0 and done % (c["steps"] // frames) == 0:
            dxb = (d["hi"] - d["lo"]) / d["nbins"]
            q = (e["x"] - d["lo"]) / dxb
            ok = (q >= 0) & (q < d["nbins"])
            h = np.bincount(q[ok].astype(np.int64), weights=e["sign"][ok], minlength=d["nbins"])
            rho.append((h / (c["n0"] * dxb)).reshape(1, -1))
    out = {"density": rho if frames <= 50 else np.stack(rho)}
    if c["ensemble"]:
        out["n"] = int(e["x"].shape[0])
        out["ensemble"] = None   # its order and rounding are this package's own
    return out
