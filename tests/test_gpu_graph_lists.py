"""Block lists and HIP graphs: captured launches create objects at every
replay, and a captured enumeration has not run when the capture ends.  On
heaps too large for direct walks, with the lists valid, stale or never built
when the capture begins, replays and eager work in turn against the oracle
(Game of Life) or a second simulation without graphs."""

import numpy as np
import pytest

from inputs import gol_init, spring_mesh
from oracle import GolWorld
from paper_1908_05845_amd.sims import GenerationSim, GolSim, SpringSim

pytestmark = pytest.mark.gpu


def captured(torch, step):
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        step(torch.cuda.current_stream())
    torch.cuda.synchronize()
    return g


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("eager", [0, 3])
@pytest.mark.parametrize("read_before", [False, True])
def test_gol_replays_and_reads(dev, fused, eager, read_before):
    import torch

    W, H = 510, 513
    init = gol_init(W, H, seed=21)
    sim, w = GolSim(W, H, init, fused=fused), GolWorld(W, H, init)
    assert sim.heap.blocks > 8192
    sim.step(1)                             # (a capture of a class's very first device allocation is not covered)
    w.step(1)
    if read_before:
        sim.read()                          # leaves every list valid
    g = captured(torch, lambda s: sim.step(2, stream=s))
    for lap in range(4):
        g.replay()
        torch.cuda.synchronize()
        w.step(2)
        sim.step(eager)
        w.step(eager)
        for got, want in zip(sim.read(), w.read()):
            assert np.array_equal(got, want), lap
    sim.heap.sync()


def test_generation_replays_and_reads(dev):
    import torch

    W, H = 512, 400
    init = gol_init(W, H, seed=5)
    sim, ref = (GenerationSim(W, H, init) for _ in range(2))
    for s in (sim, ref):
        s.step(2)
    sim.read()
    g = captured(torch, lambda s: sim.step(3, stream=s))
    for lap in range(3):
        g.replay()
        torch.cuda.synchronize()
        ref.step(3)
        for got, want in zip(sim.read(), ref.read()):
            assert np.array_equal(got, want), lap


def test_a_captured_enumeration_is_not_taken_for_done(dev):
    """The node list of a new mesh is first built inside the capture; eager
    steps before any replay still visit every node."""
    import torch

    mesh = spring_mesh(120, 90, seed=3)
    sim, ref = (SpringSim(mesh, 1e-4, 0.3) for _ in range(2))
    g = captured(torch, lambda s: sim.step(2, stream=s))
    sim.step(1)
    ref.step(1)
    a, b = sim.read(), ref.read()
    assert np.array_equal(a["x"], b["x"]) and np.any(a["x"] != mesh["x"])
    g.replay()
    torch.cuda.synchronize()
    ref.step(2)
    a, b = sim.read(), ref.read()
    for key in a:
        assert np.array_equal(a[key], b[key]), key
