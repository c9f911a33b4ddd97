"""Handles whose walk grid is tuned on stretches of several steps, or set: the
tiles follow the grid, the results do not."""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import O, P, compare, say  # noqa: F401

pytestmark = pytest.mark.gpu


def test_autotune_on_stretches(P, O):  # noqa: F811
    cfg = W.batched_barriers(B=3, N0=np.array([3000, 100, 25000], dtype=np.int64), capacity=1_000_000)
    g, r = P.Simulation(cfg), O.OracleSim(cfg)
    g.step(3)
    chosen = g.autotune(7)
    n = g.stats()["step"]
    say(f"autotune on stretches: {chosen} after {n} steps")
    assert (n - 3) % 14 == 0 and n > 3
    r.step(n)
    compare(g, r, "autotune", B=3)
    g.run(21, 10)
    r.run(21, 10)
    compare(g, r, "after autotune", B=3)


@pytest.mark.parametrize("kind", ["sp1", "pairs", "4d"])
def test_grids_set_between_steps(P, O, kind):  # noqa: F811
    """Grids of 1, 7, 300 and 2000 blocks on an ensemble that has plans for the
    one before."""
    n0 = np.array([20_000])
    cfg = {"sp1": lambda: W.gaussian_barrier_small(N0=n0, capacity=1_000_000),
           "pairs": lambda: W.gaussian_barrier_small(N0=n0, capacity=1_000_000, gamma0=0.45, track_tangent=2),
           "4d": lambda: W.helium_soft_coulomb(N0=n0, capacity=2_000_000)}[kind]()
    g, r = P.Simulation(cfg), O.OracleSim(cfg)
    d = g.launch()
    for blocks in (1, 7, 300, 2000):
        say(f"grids set between steps: {kind} {blocks}")
        g.set_launch(dict(d, family_blocks=blocks))
        n = 1 if kind == "4d" else 6
        g.step(n)
        r.step(n)
        compare(g, r, f"{kind} {blocks} blocks")
