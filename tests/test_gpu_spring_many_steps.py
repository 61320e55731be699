"""spring.steps of a small mesh for thousands of steps: several launches, none
of which holds the stream for long, with the results of the do-alls."""

import ctypes

import numpy as np
import pytest

from inputs import spring_mesh
from paper_1908_05845_amd.sims import SpringSim
from test_gpu_heap import clean

pytestmark = pytest.mark.gpu

MOST = 4096          # steps of one launch


def test_thousands_of_steps_equal_the_do_alls(dev):
    n = 2 * MOST + 3
    a, b = (SpringSim(spring_mesh(8, 7, seed=3, v_sigma=3.0), 1e-4, 0.1) for _ in range(2))
    a.step(n)
    for _ in range(n):
        b.spring_force()
        b.node_update()
    ra, rb = a.read(), b.read()
    for key in ra:
        assert np.array_equal(ra[key], rb[key]), key
    assert 0 < ra["alive"].sum() < ra["alive"].size
    clean(a.heap)
    a.heap.close()
    b.heap.close()


@pytest.mark.parametrize("n,launches", [(MOST, 1), (MOST + 1, 2), (3 * MOST, 3)])
def test_no_launch_takes_more(dev, n, launches):
    """Counted as the kernel nodes of a graph: the two enumerations, and per
    part the steps and the launch for meshes that have grown."""
    import torch

    sim = SpringSim(spring_mesh(8, 7, seed=3), 1e-4, 0.3)
    sim.step(2)
    sim.heap.sync()
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g):
        sim.step(n, stream=torch.cuda.current_stream())
    nodes = ctypes.c_size_t()
    hip = ctypes.CDLL("libamdhip64.so")
    assert hip.hipGraphGetNodes(ctypes.c_void_p(g.raw_cuda_graph()), None, ctypes.byref(nodes)) == 0
    assert nodes.value == 2 + 2 * launches
    sim.heap.close()
