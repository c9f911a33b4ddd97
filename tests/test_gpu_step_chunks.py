"""GPU parity where several steps share a launch and where a cell pass sums
neighbours: the lengths of calls around a launch's five steps and the 32 steps
that positions may be behind, families beyond the block's pool, ranges and runs
at the edges of tiles, cells at their boundaries.  Everything is bit-exact
against the FP64 oracle (tolerance 0)."""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import O, P, _exact, assert_same_ensemble, compare, say  # noqa: F401

pytestmark = pytest.mark.gpu


def _compare_all(g, r, cfg, what):
    B = int(cfg["B"])
    compare(g, r, what, B=B)
    if cfg["track_tangent"]:
        for b in range(B):
            _exact(g.particles(b)["D"], r.particles(b)["D"], what + " tangents")
            assert g.count(b, ghost=True) == r.count(b, ghost=True)
            pg, pr = g.particles(b, ghost=True), r.particles(b, ghost=True)
            assert_same_ensemble(pg, pr, what=what + " ghosts")
            _exact(pg["D"], pr["D"], what + " ghost tangents")


@pytest.mark.parametrize("kind", ["sp1", "sp2", "tangent", "pairs", "sp2 tangent", "two components", "4d"])
def test_lengths_of_calls(P, O, kind):  # noqa: F811
    """1 to 12 steps in one call, annihilated after some of them."""
    n0 = np.array([1500])
    cfg = {"sp1": lambda: W.gaussian_barrier_small(N0=n0),
           "sp2": lambda: W.gaussian_barrier_small(N0=n0, strategy="sp2"),
           "tangent": lambda: W.gaussian_barrier_small(N0=n0, gamma0=0.45, track_tangent=1),
           "pairs": lambda: W.gaussian_barrier_small(N0=n0, gamma0=0.45, track_tangent=2),
           "sp2 tangent": lambda: W.gaussian_barrier_small(N0=n0, gamma0=0.45, track_tangent=1, strategy="sp2"),
           "two components": lambda: W.time_dependent_barriers(N0=n0, capacity=60_000),
           "4d": lambda: W.helium_soft_coulomb(N0=n0, grid={"x_lo": -10.0, "x_hi": 10.0, "nx": 12, "k_lo": -4.0,
                                                            "k_hi": 4.0, "nk": 12}, capacity=400_000)}[kind]()
    g, r = P.Simulation(cfg), O.OracleSim(cfg)
    for n in (1, 2, 4, 5, 6, 9, 10, 11, 3, 12)[:5 if kind == "4d" else 10]:
        say(f"lengths of calls: {kind} {n}")
        g.step(n)
        r.step(n)
        _compare_all(g, r, cfg, f"{kind} {n} steps")
        if n > 4:
            g.annihilate()
            r.annihilate()


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("strategy,every", [("sp1", 7), ("sp1", 31), ("sp1", 32), ("sp1", 33), ("sp1", 40), ("sp2", 33)])
def test_positions_behind(P, O, strategy, every, graph):  # noqa: F811
    """Annihilations after up to 40 steps of one call, in one or several tiles
    per instance; replayed graphs between eager calls."""
    cfg = W.batched_barriers(B=9, strategy=strategy, capacity=1_000_000,
                             N0=np.array([63, 64, 65, 0, 1, 2047, 2049, 300, 4100], dtype=np.int64))
    import torch
    kw = {"stream": torch.cuda.Stream()} if graph else {}
    g, r = P.Simulation(cfg, **kw), O.OracleSim(cfg)
    for _ in range(3):
        say(f"positions behind: {strategy} every {every} graph {graph}")
        g.run(every, every, use_graph=graph)
        g.synchronize()
        r.run(every, every)
        compare(g, r, f"every {every}", B=9)
    g.step(3)
    r.step(3)
    compare(g, r, f"every {every}, 3 steps more", B=9)


def _crowded(gdt, kind, n0):
    """Nearly all kicks happen: every particle sits where |sin(2 q x)| is 1, so
    that a jump leaves two offspring where the plans expect 1.27, and a block's
    event parents more of them than its pool of records holds."""
    spike = {"kind": "table", "axis": 0, "table": gdt * 78539.8 * np.ones(4), "q_lo": 0.98, "q_hi": 1.02, "sgn": 1.0,
             "center": 0.0}                     # gamma0 = gdt / dt
    cfg = W.gaussian_barrier_small(N0=np.array([n0]), dt=0.001, capacity=8 * n0 + 600_000, components=[spike],
                                   init={"mean_x": [np.pi / 4, 0.0], "sigma_x": [0.001, 0.001],
                                         "mean_k": [0.0, 0.0], "sigma_k": [0.5, 0.5]})
    if kind in ("sp1", "sp2"):
        cfg["strategy"] = kind
    else:      # tangents need a Gaussian barrier: a wide spectrum, fewer offspring
        cfg["track_tangent"] = {"tangent": 1, "pairs": 2}[kind]
        cfg["components"] = [W._gauss_component(1, 1000.0 * gdt, 1.0, 0.0)]
        cfg["init"]["mean_x"] = [2.0, 0.0]
    return cfg


@pytest.mark.parametrize("kind,gdt,n0,steps", [("sp1", 0.2, 1_250_000, 3), ("sp1", 0.2, 250_000, 5), ("sp1", 0.3, 700_000, 2),
                                               ("sp1", 1.2, 3000, 2),
                                               ("sp2", 1.2, 3000, 2), ("tangent", 2.0, 3000, 2), ("pairs", 1.2, 3000, 1)])
def test_families_beyond_the_pool(P, O, kind, gdt, n0, steps):  # noqa: F811
    """Tiles of which some batch outgrows the pool, in the first step of a
    launch and in later ones, and (250 000: some 230 jumps of five steps in a
    tile, 224 to a batch) in one list of all steps or step by step."""
    cfg = _crowded(gdt, kind, n0)
    g, r = P.Simulation(cfg), O.OracleSim(cfg)
    for n in (steps, 1):
        g.step(n)
        r.step(n)
        say(f"families beyond the pool: {kind} gamma dt = {gdt}, {n} steps, n={r.count()}")
        _compare_all(g, r, cfg, f"{kind} {gdt}")
        g.annihilate()
        r.annihilate()
        _compare_all(g, r, cfg, f"{kind} {gdt} annihilated")


@pytest.mark.parametrize("nx", [240, 1200])
def test_cells_at_their_boundaries(P, O, nx):  # noqa: F811
    """All particles at one position: a cell boundary as computed and its two
    neighbours, inside, at the ends of the grid and outside.  At 1200 cells the
    cell width is not a binary fraction."""
    w = 120.0 / nx
    at = [-60.0 + j * w for j in (0, 1, 3, nx // 3, nx // 2 + 1, nx - 1, nx)] + [0.0, -0.0, 1e-300, -1e-300, 1e9, -1e9]
    say(f"cells at their boundaries: nx = {nx}")
    for x in at:
        for y in (np.nextafter(x, -np.inf), x, np.nextafter(x, np.inf)):
            cfg = W.gaussian_barrier_small(N0=np.array([40]), init={"mean_x": [float(y), 0.0], "sigma_x": [0.0, 0.0],
                                                                   "mean_k": [1.5, 0.0], "sigma_k": [0.5, 0.5]})
            cfg["grid"] = dict(cfg["grid"], nx=nx)
            g, r = P.Simulation(cfg), O.OracleSim(cfg)
            g.annihilate()
            r.annihilate()
            compare(g, r, f"x = {y!r}")


@pytest.mark.parametrize("kind", ["sp1", "sp2", "tangent"])
@pytest.mark.parametrize("n0", [1, 7, 8, 9, 511, 512, 513, 2047, 2048, 2049, 4103])
def test_runs_of_equal_cells(P, O, n0, kind):  # noqa: F811
    """Two cells along x and four along k: runs over threads, wavefronts and
    tiles; mixed signs and classes behind the ordered front."""
    grid = dict(W.gaussian_barrier_small()["grid"], nx=2, nk=4)
    cfg = W.gaussian_barrier_small(N0=np.array([n0]), grid=grid, gamma0=0.45, capacity=40 * n0 + 2000,
                                   strategy="sp2" if kind == "sp2" else "sp1", track_tangent=int(kind == "tangent"))
    say(f"runs of equal cells: {kind} n0={n0}")
    g, r = P.Simulation(cfg), O.OracleSim(cfg)
    for _ in range(2):
        g.annihilate()
        r.annihilate()
        g.step(6)
        r.step(6)
        _compare_all(g, r, cfg, f"runs {n0}")


def test_cell_sums_over_many_annihilations(P):  # noqa: F811
    """1e7 particles, 100 annihilations whose cell passes empty their tables
    many times: every cell's net sign is that of the particles before, counted
    by torch."""
    import ctypes as C

    import torch
    cfg = W.gaussian_barrier_large("sp1")
    g = cfg["grid"]
    dx, dk = (g["x_hi"] - g["x_lo"]) / g["nx"], (g["k_hi"] - g["k_lo"]) / g["nk"]
    s = P.Simulation(cfg)

    def net():
        n = s.count()
        x, k = (torch.empty(n, dtype=torch.float64, device="cuda") for _ in range(2))
        sign = torch.empty(n, dtype=torch.int8, device="cuda")
        torch.cuda.synchronize()
        assert P.lib().wbrw_export(s.h, 0, 0, n, *(C.c_void_p(t.data_ptr()) for t in (x, k, sign)),
                                   None, None, None) == P.OK
        qx, qk = (x - g["x_lo"]) / dx, (k - g["k_lo"]) / dk
        inside = (qx >= 0) & (qx < g["nx"]) & (qk >= 0) & (qk < g["nk"])
        cell = qx.floor().long() + g["nx"] * qk.floor().long()
        return torch.zeros(g["nx"] * g["nk"], dtype=torch.int64, device="cuda").index_add_(
            0, cell[inside], sign[inside].long())

    for ep in range(100):
        s.step(10)
        before = net()
        s.annihilate()
        assert torch.equal(net(), before), f"annihilation {ep}"
    say(f"many annihilations: n={s.count()}")


@pytest.mark.parametrize("graph", [False, True])
def test_dropped_while_its_work_is_under_way(P, O, graph):  # noqa: F811
    """Handles on two streams, each dropped while its work may be under way:
    the next one, on the other stream, must not get its memory."""
    import torch
    cfgs = [W.batched_barriers(B=14, seed=3, capacity=60_000, N0=np.full(14, n, dtype=np.int64)) for n in (4000, 3500)]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    want = []
    for c in cfgs:
        r = O.OracleSim(c)
        r.run(16, 10)
        want.append(r.density())
    got, last = [], None
    for k in (0, 1, 0, 1):
        s = P.Simulation(cfgs[k], stream=streams[k])
        assert s.workspace.data_ptr() != last
        last = s.workspace.data_ptr()
        s.run(16, 10, use_graph=graph)
        got.append((k, s.density()))
        del s
    torch.cuda.synchronize()
    say(f"dropped while its work is under way: graph {graph}")
    for k, d in got:
        assert np.array_equal(d.cpu().numpy(), want[k])
