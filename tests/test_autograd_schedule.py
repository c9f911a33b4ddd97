"""The schedule of the differentiable density: annihilations after the steps
whose number is a multiple of annihilate_every, checkpoints after those that are
one of snapshot_every, for every period that Python's remainder takes."""
import numpy as np
import pytest
import torch

import workloads as W
from paper_1709_02121_amd import autograd


class _Recorder:
    """Takes the calls of a Simulation and writes down what they amount to."""

    log = []

    def __init__(self, cfg, device=None):
        self.done = 0
        _Recorder.log = []

    def step(self, n=1):
        self.done += n

    def annihilate(self):
        self.log.append(("annihilated", self.done))

    def run(self, n, every, use_graph=False):
        assert isinstance(n, int) and isinstance(every, int) and n >= 0 and 0 <= every < 2 ** 31
        for _ in range(n):
            self.step()
            if every and self.done % every == 0:
                self.annihilate()

    def snapshot(self):
        self.log.append(("snapshot", self.done))
        return self.done

    def density(self):
        return torch.zeros((1, 4), dtype=torch.float64)


@pytest.mark.parametrize("every", [0, None, 1, 4, 10, 100, -4, 4.0, 2.5, True, np.int64(4), 2 ** 31, 2 ** 32 + 4,
                                   float("inf"), float("nan")])
@pytest.mark.parametrize("snap", [0, None, 5, 7, -5, 5.0, 2.5, 50, float("inf")])
@pytest.mark.parametrize("steps", [0, -3, 1, 23])
def test_schedule(monkeypatch, every, snap, steps):
    monkeypatch.setattr(autograd, "Simulation", _Recorder)
    want = []
    for s in range(1, steps + 1):
        if every and s % every == 0:
            want.append(("annihilated", s))
        if snap and s % snap == 0:
            want.append(("snapshot", s))
    theta = torch.tensor([0.3, 1.0, 0.0], dtype=torch.float64)
    for checkpoints in (None, []):
        autograd.WBRWDensity.apply(theta, W.differentiation(), steps, every, snap, "cpu", checkpoints)
        kinds = ("annihilated", "snapshot") if checkpoints is not None else ("annihilated",)
        assert _Recorder.log == [w for w in want if w[0] in kinds]
    assert checkpoints == [(s, s) for k, s in want if k == "snapshot"]
