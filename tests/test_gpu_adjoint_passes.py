"""The one-pass forward and reverse steps of the differentiable mesh against
its separate spring and node passes: positions, gradients, the springs' forces
and the nodes' adjoint fields bit for bit, over segment lengths and step
counts on both sides of every rule (one slot per tape, one segment, a last
segment of one step), ragged block counts, and nodes without springs; and what
the two methods refuse."""

import numpy as np
import pytest

from inputs import spring_mesh
from paper_1908_05845_amd import smmo
from paper_1908_05845_amd.adjoint import DiffSpringSim

pytestmark = pytest.mark.gpu


def build(mesh, T, every, passes, monkeypatch):
    monkeypatch.setattr(DiffSpringSim, "PASS_NODES", (1 << 30) if passes else 0)
    sim = DiffSpringSim(mesh, 1e-3, T, every)
    assert sim.passes == (passes and min(every, T) >= 2)
    return sim


def outcome(sim, torch, seed):
    g = torch.Generator(device=sim.dev).manual_seed(seed)
    seeds = [torch.randn(sim.N, generator=g, device=sim.dev) for _ in range(4)]
    xT = sim.forward()
    f = sim.heap.gather("Spring", ["id", "fx", "fy"])
    o = torch.argsort(f["id"].long())
    return [xT, f["fx"][o], f["fy"][o], *sim.backward(*seeds)]


@pytest.mark.parametrize("W,H,T,every", [(2, 2, 5, 2), (9, 7, 20, 1), (8, 8, 1, 20), (16, 12, 2, 20), (33, 21, 21, 20),
                                         (30, 22, 40, 20), (40, 31, 60, 7), (64, 64, 9, 3), (200, 131, 30, 10)])
def test_passes_equal_separate_launches(dev, monkeypatch, W, H, T, every):
    import torch

    mesh = spring_mesh(W, H, seed=W + T, v_sigma=0.5)
    a, b = build(mesh, T, every, True, monkeypatch), build(mesh, T, every, False, monkeypatch)
    for stream in (torch.cuda.default_stream(), torch.cuda.Stream()):
        with torch.cuda.stream(stream):
            for x, y in zip(outcome(a, torch, T), outcome(b, torch, T)):
                assert torch.equal(x, y)
            a.restart()
            b.restart()
        torch.cuda.synchronize()


def test_nodes_without_springs(dev, monkeypatch):
    import torch

    mesh = spring_mesh(12, 11, seed=1, v_sigma=0.5)
    mesh = dict(mesh)
    for key in ("x", "y", "vx", "vy", "m"):
        mesh[key] = np.concatenate([mesh[key], np.full(70, 2.0, np.float32)])
    a, b = build(mesh, 25, 10, True, monkeypatch), build(mesh, 25, 10, False, monkeypatch)
    for x, y in zip(outcome(a, torch, 3), outcome(b, torch, 3)):
        assert torch.equal(x, y)


def test_refusals(dev):
    import torch

    sim = DiffSpringSim(spring_mesh(6, 5, seed=1), 1e-3, 6, 3)
    buf = torch.zeros(8 * sim.plane, device=dev)
    at = [buf.data_ptr() + 4 * sim.plane * i for i in range(8)]

    def refused(name, cls="Node", plane=sim.plane, dt=1e-3, x=at[:2], w=(None, None), out=at[4:6], reserved=0):
        args = smmo.smmo_adjoint_pass_args(sim.cn, sim.cs, dt, reserved, plane, *x, *w, *out)
        with pytest.raises(smmo.SmmoError) as e:
            sim.heap.do(cls, name, args)
        assert e.value.status == smmo.SMMO_EINVAL

    for name in ("adjoint.step", "adjoint.reverse"):
        refused(name, cls="Spring")
        refused(name, plane=sim.plane - 64)
        refused(name, dt=float("nan"))
        refused(name, reserved=1)
        refused(name, out=(at[4], None))
        refused(name, out=(at[4], at[4]))
        refused(name, out=at[1:3], w=at[2:4])
    refused("adjoint.step", out=(None, None))
    refused("adjoint.step", x=(at[0], None))
    refused("adjoint.reverse", x=(None, None), w=at[2:4])
    refused("adjoint.reverse", w=(at[2], None))
    refused("adjoint.reverse", w=at[2:4], out=at[3:5])
    sim.heap.sync()
