"""Handles on a stream of their own: tensors that cross to and from torch's
current stream.  A spinning kernel holds the current stream back, so that what
should wait for it shows whether it does."""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import P, say  # noqa: F401

pytestmark = pytest.mark.gpu


def _busy(torch):
    torch.cuda._sleep(50_000_000)


def _barrier(P, **over):  # noqa: F811
    import torch
    s = P.Simulation(W.gaussian_barrier_small(N0=np.array([4000]), **over), stream=torch.cuda.Stream())
    s.run(20, 10)
    s.synchronize()
    return s


def test_gradient_of_another_stream(P):  # noqa: F811
    import torch
    s = _barrier(P, gamma0=0.45, track_tangent=1)
    want = s.density_vjp(torch.linspace(-1, 1, 240, dtype=torch.float64, device="cuda")).cpu()
    say("streams: gradient")
    for dtype in (torch.float64, torch.float32):
        g = torch.full((240,), 1e9, dtype=dtype, device="cuda")
        torch.cuda.synchronize()
        _busy(torch)
        g.copy_(torch.linspace(-1, 1, 240, dtype=dtype, device="cuda"))
        got = s.density_vjp(g).cpu()
        assert torch.allclose(got, want, rtol=0, atol=1e-5 if dtype == torch.float32 else 0.0)


def test_buffers_in_use_on_another_stream(P):  # noqa: F811
    """A caller's buffer that the current stream is still to read."""
    import torch
    s = _barrier(P, gamma0=0.45, track_tangent=1)
    say("streams: buffers")
    for call, shape in ((s.density, (1, 240)), (s.density_noalloc, (1, 240)), (s.density_tangent, (1, 3, 240))):
        out = torch.full(shape, 5.0, dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        _busy(torch)
        before = out.clone()
        call(out=out)
        torch.cuda.synchronize()
        assert bool((before == 5.0).all()) and not bool((out == 5.0).all())


def test_snapshots_in_memory_of_another_stream(P):  # noqa: F811
    """A snapshot, its copy and the exported ensemble in memory that the current
    stream (not the default one, which the copies to the host wait for) is
    still to write."""
    import torch
    s = _barrier(P)
    with torch.cuda.stream(torch.cuda.Stream()):
        _snapshots(s)


def _snapshots(s):
    import torch
    snap, part = s.snapshot(), s.particles()
    n = snap.numel()

    def same(now):
        assert s.stats()["step"] == 20
        for f in part:
            assert np.array_equal(now[f], part[f]), f

    held = torch.empty(n, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    say("streams: snapshots")
    _busy(torch)
    held.fill_(7)
    del held                                   # its memory goes to the next snapshot
    again = s.snapshot()
    torch.cuda.synchronize()
    s.step(3)
    s.restore(again)
    same(s.particles())
    copy = torch.empty_like(snap)
    torch.cuda.synchronize()
    _busy(torch)
    copy.copy_(snap)
    s.step(3)
    s.restore(copy)
    same(s.particles())
    held = [torch.empty(part["id"].nbytes, dtype=torch.uint8, device="cuda") for _ in range(4)]
    torch.cuda.synchronize()
    _busy(torch)
    for h in held:
        h.fill_(7)
    del held, h
    same(s.particles())


def test_results_in_use_on_another_stream(P):  # noqa: F811
    """A density that the current stream is still to read, dropped: the next one
    is not written over it."""
    import torch
    s = _barrier(P, gamma0=0.45, track_tangent=1)
    g = torch.ones(240, dtype=torch.float64, device="cuda")
    say("streams: results")
    for call in (s.density, s.density_tangent, lambda: s.density_vjp(g)):
        first = call()
        want = first.cpu()
        torch.cuda.synchronize()
        _busy(torch)
        read = first.clone()
        del first
        s.step(4)
        # (not density_vjp, which waits for the current stream by itself)
        nxt = [s.density(nbins=n) for n in (240, 240, 3)] + [s.density_tangent()]
        torch.cuda.synchronize()
        assert torch.equal(read.cpu(), want)
        del nxt
    pinned = torch.zeros((1, 240), dtype=torch.float64, pin_memory=True)
    want = s.density().cpu()
    s.density(out=pinned)
    torch.cuda.synchronize()
    assert torch.equal(pinned, want)
