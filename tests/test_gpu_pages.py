"""GPU parity of ensembles that grow far in one launch: a tile's offspring
fill more pages than the tile lists itself (24) and than one table holds (64),
with room for exactly the particles that the oracle ends with.  What fits the
capacity is not refused, whatever the tiles' shares."""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import O, P, say  # noqa: F401
from test_gpu_step_chunks import _compare_all, _crowded

pytestmark = pytest.mark.gpu


def _grown(O, cfg, steps):  # noqa: F811
    r = O.OracleSim(cfg)
    r.step(steps)
    return r


# growth of e^(2 gamma dt) a step: 25 and 121 times (pages of half a tile, 2 a
# unit of growth); 18 times in two steps of one launch
@pytest.mark.parametrize("kind,gdt,n0,steps", [("sp1", 1.6, 300, 1), ("sp1", 2.4, 150, 1), ("sp2", 1.6, 300, 1),
                                               ("sp1", 0.66, 4000, 2), ("sp1", 1.6, 60, 1)])
def test_offspring_that_just_fit(P, O, kind, gdt, n0, steps):  # noqa: F811
    cfg = _crowded(gdt, kind, n0)
    r = _grown(O, cfg, steps)
    n = r.count()
    say(f"offspring that just fit: {kind} gamma dt = {gdt}, {n0} -> {n}")
    g = P.Simulation(dict(cfg, capacity=n))
    g.step(steps)
    assert g.stats_code()[0] == P.OK
    _compare_all(g, r, cfg, f"{kind} {gdt}")
    # the room is there again for the next launch, and one particle more is refused
    g.annihilate()
    r.annihilate()
    _compare_all(g, r, cfg, f"{kind} {gdt} annihilated")
    g = P.Simulation(dict(cfg, capacity=n - 1))
    g.step(steps)
    assert g.stats_code()[0] == P.ECAPACITY


def test_ghosts_that_just_fit(P, O):  # noqa: F811
    """Ghosts branch by the same rule in pages and tables of their own."""
    cfg = _crowded(2.4, "tangent", 2000)
    cfg["grid"] = dict(cfg["grid"], nk=8192)
    cfg["ghost_capacity"] = 600_000
    r = _grown(O, cfg, 1)
    r.annihilate()
    ng0 = r.count(0, ghost=True)
    r.step(1)
    ng = r.count(0, ghost=True)
    say(f"ghosts that just fit: {ng0} -> {ng}")
    g = P.Simulation(dict(cfg, ghost_capacity=ng))
    g.step(1)
    g.annihilate()
    g.step(1)
    assert g.stats_code()[0] == P.OK
    _compare_all(g, r, cfg, "ghosts")


def test_instances_share_the_tables(P, O):  # noqa: F811
    """Three instances that each need tables, several launches in a row."""
    one = _crowded(1.6, "sp1", 100)
    cfg = dict(one, B=3, N0=np.array([130, 400, 250]), capacity=60_000)
    r = _grown(O, cfg, 1)
    cap = np.array([r.count(b) for b in range(3)])
    say(f"instances share the tables: {cap}")
    g = P.Simulation(dict(cfg, capacity=cap))
    first = g.snapshot()
    for k in range(3):
        g.restore(first)
        g.step(1)
        assert g.stats_code()[0] == P.OK
        _compare_all(g, r, cfg, f"instances {k}")


def test_offspring_beyond_the_event_bits(P, O):  # noqa: F811
    """Tiles of 1216 particles whose offspring pass 4096 before the launch's
    last step: their jumps are read back from memory.  The instance with the
    particles has hardly any of the sample size, which sets its tiles."""
    cfg = _crowded(0.2, "sp1", 3000)
    grid = {"x_lo": np.pi / 4 - 0.004, "x_hi": np.pi / 4 + 0.004, "nx": 8, "k_lo": -8.0, "k_hi": 8.0, "nk": 32}
    hist = np.zeros((2, 32, 8))
    hist[1, 14:18, :] = 75.0 / (100 * 0.001 * 0.5)         # 32 cells of 75 particles
    cfg.update(B=2, N0=np.array([1_000_000, 100]), capacity=np.array([1_000_000, 60_000]), grid=grid,
               init_histogram=hist.reshape(2, -1))
    r = O.OracleSim(cfg)
    g = P.Simulation(cfg)
    r.step(4)
    assert r.count(1) - 2400 > 2 * 4500        # two tiles
    r.step(1)
    g.step(5)
    say(f"offspring beyond the event bits: {r.count(1)}")
    _compare_all(g, r, cfg, "5 steps")


def test_offspring_beyond_the_event_bits_4d(P, O):  # noqa: F811
    """The same in 4D, where a tile of 2500 grows fourfold in a launch and a
    jump has three components."""
    cfg = W.helium_soft_coulomb()
    grid = dict(cfg["grid"], x_lo=5.0, x_hi=20.0, nx=3, k_lo=-16.0, k_hi=16.0, nk=4)
    hist = np.zeros((2, 4, 4, 3, 3))
    hist[1, 1:3, 1:3] = 138.0 / (100 * 5.0 ** 2 * 8.0 ** 2)          # 36 cells of 138 particles
    cfg.update(B=2, N0=np.array([1_000_000, 100]), capacity=np.array([1_000_000, 100_000]), grid=grid,
               init_histogram=hist.reshape(2, -1))
    r = O.OracleSim(cfg)
    g = P.Simulation(cfg)
    n0 = r.count(1)
    r.step(4)
    assert r.count(1) - n0 > 2 * 4500          # two tiles
    r.step(1)
    g.step(5)
    say(f"offspring beyond the event bits, 4d: {n0} -> {r.count(1)}")
    _compare_all(g, r, cfg, "4d 5 steps")
    g.annihilate()
    r.annihilate()
    g.step(2)
    r.step(2)
    _compare_all(g, r, cfg, "4d 2 steps more")
