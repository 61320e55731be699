"""nbody.steps against the two do-alls one after the other, bit for bit: class
sizes with and without the pair form, free slots, a snapshot taken ahead, and
replays of a graph captured before and after the first eager step."""

import numpy as np
import pytest

from inputs import nbody_init
from paper_1908_05845_amd.sims import NbodySim

pytestmark = pytest.mark.gpu

FIELDS = ("x", "y", "vx", "vy", "fx", "fy")


def make(n, eps=1e-3, free=False, dev=None):
    import torch

    sim = NbodySim(nbody_init(n, seed=n), 1.0 / n, eps, 1e-4)
    if free:
        gone = np.unique(np.random.default_rng(1).integers(0, n, n // 3))
        sim.heap.destroy("Body", sim.handles[torch.from_numpy(gone).to(dev)])
    return sim


def same(a, b):
    a, b = a.read(), b.read()
    assert np.array_equal(a["id"], b["id"])
    for f in FIELDS:
        assert np.array_equal(a[f], b[f]), f


@pytest.mark.parametrize("n,free", [(1, False), (700, False), (64 * 12, False), (3001, False), (3001, True),
                                    (20011, True), (64 * 600 + 5, False), (64 * 1536 + 1, False)])
@pytest.mark.parametrize("eps", [1e-3, 0.0])
def test_steps_equal_the_do_alls(dev, n, free, eps):
    a, b = make(n, eps, free, dev), make(n, eps, free, dev)
    for k in (0, 1, 3, -2):
        a.step(k)
        for _ in range(k):
            b.force()
            b.update()
    same(a, b)
    a.heap.close()
    b.heap.close()


def test_a_snapshot_ahead_is_the_first_step_s(dev):
    a, b = make(3001), make(3001)
    for sim in (a, b):
        sim.heap.snapshot("Body")
    a.step(3)
    for _ in range(3):
        b.force()
        b.update()
    same(a, b)
    a.heap.close()
    b.heap.close()


@pytest.mark.parametrize("eager_first", [False, True])
def test_captured(dev, eager_first):
    import torch

    a, b = make(3001), make(3001)
    if eager_first:
        for sim in (a, b):
            sim.step(1)
    else:
        for sim in (a, b):             # lists and modules, no workspace
            sim.update()
    a.heap.sync()
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        a.step(2, stream=torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    for _ in range(3):
        g.replay()
        torch.cuda.synchronize()
        if eager_first:
            b.step(2)
            same(a, b)
    a.heap.sync()
    a.heap.close()
    b.heap.close()


def test_bad_parameters_are_refused(dev):
    from paper_1908_05845_amd import smmo

    a = make(100)
    for bad in ((1.0, -1.0, 1e-4, 2), (float("nan"), 1e-3, 1e-4, 2), (1.0, 1e-3, float("nan"), 2)):
        with pytest.raises(smmo.SmmoError) as e:
            smmo.smmo_parallel_do(a.heap.h, a.cls, a.m_steps, smmo.smmo_nbody_steps_args(*bad), None)
        assert e.value.status == smmo.SMMO_EINVAL
    with pytest.raises(TypeError):
        a.step(1.5)
    a.heap.close()
