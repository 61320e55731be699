"""Captured walks: objects created after the capture - by the graph's own
launches, by another graph or by eager calls - are visited by the next replay,
with no eager look at the class in between."""

import numpy as np
import pytest

from inputs import gol_init
from oracle import GolWorld
from paper_1908_05845_amd import smmo
from paper_1908_05845_amd.sims import GolSim
from test_gpu_graph_growth import captured
from test_gpu_heap import cfg, clean

pytestmark = pytest.mark.gpu

CLASSES = {"A": [("x", "f32", 1), ("key", "i32", 1)], "B": [("key", "i32", 1), ("x", "f32", 1)]}


@pytest.mark.parametrize("W,H", [(510, 513), (64, 48)])
@pytest.mark.parametrize("packing", [0, 2])
def test_a_first_device_allocation_inside_the_capture(dev, W, H, packing):
    """Game of Life captured before any birth or death: the list of the living
    is the one that the read left."""
    init = gol_init(W, H, seed=21)
    sim, w = GolSim(W, H, init, cfg=cfg(sparse_packing=packing)), GolWorld(W, H, init)
    sim.read()
    g = captured(lambda st: sim.step(1, stream=st))
    for laps in (2, 1, 3):
        for _ in range(laps):
            g.replay()
        sim.heap.sync()
        w.step(laps)
        for got, want in zip(sim.read(), w.read()):
            assert np.array_equal(got, want)
    clean(sim.heap)


def make(dev, blocks, n):
    import torch

    heap = smmo.Heap(CLASSES, blocks=blocks)
    heap.new("A", n, x=torch.ones(n, device=dev), key=torch.arange(n, dtype=torch.int32, device=dev))
    heap.new("B", 100, key=torch.arange(100, dtype=torch.int32, device=dev))
    heap.gather("A", ["key"])                       # every list valid
    heap.gather("B", ["key"])
    return heap


def values(heap):
    g = heap.gather("A", ["x", "key"])
    o = np.argsort(g["key"].cpu().numpy(), kind="stable")
    return g["key"].cpu().numpy()[o], g["x"].cpu().numpy()[o]


@pytest.mark.parametrize("blocks", [60, 9000])
def test_objects_of_eager_calls(dev, blocks):
    import torch

    heap = make(dev, blocks, 300)
    axpy = smmo.smmo_axpy_args(2.0, 1.0)
    g = captured(lambda st: heap.do("A", "test.axpy", axpy, stream=st))
    n, want = 300, np.ones(300, np.float32)
    for k in (1, 64, 200):
        heap.new("A", k, x=torch.ones(k, device=dev), key=torch.arange(n, n + k, dtype=torch.int32, device=dev))
        n, want = n + k, np.concatenate([want, np.ones(k, np.float32)])
        g.replay()
        g.replay()
        torch.cuda.synchronize()
        want = 2 * (2 * want + 1) + 1
        key, x = values(heap)
        assert np.array_equal(key, np.arange(n)) and np.array_equal(x, want)
    heap.close()


@pytest.mark.parametrize("blocks", [60, 9000])
def test_objects_of_another_graph(dev, blocks):
    """One graph deletes every A, captured first; another has each B create
    objects of A: replayed in turn, nothing of A is ever left."""
    import torch

    heap = make(dev, blocks, 300)
    gone = captured(lambda st: heap.do("A", "test.destroy_if", smmo.smmo_destroy_if_args(1, 0), stream=st))
    spawn = smmo.smmo_spawn_args(heap.cls["A"], 1, 0, 3, 1, 0)
    births = captured(lambda st: heap.do("B", "test.spawn", spawn, stream=st))
    for lap in range(4):
        births.replay()
        gone.replay()
        torch.cuda.synchronize()
    assert heap.stats().device_news == 4 * 300 and heap.stats().live_objects[heap.cls["A"]] == 0
    clean(heap)
    heap.close()
