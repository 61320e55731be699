"""Step counts beyond what an argument struct's 32 bits hold: the drivers hand
them to the library in parts (without a GPU: what they would launch)."""

from types import SimpleNamespace

import pytest

from paper_1908_05845_amd import smmo
from paper_1908_05845_amd.sims import NbodySim, SpringSim


@pytest.mark.parametrize("n", [0, 1, 7, (1 << 32) - 1, 1 << 32, (1 << 32) + 5, 3 * (1 << 32)])
@pytest.mark.parametrize("cls", [SpringSim, NbodySim])
def test_every_step_is_launched(monkeypatch, cls, n):
    sim = cls.__new__(cls)
    sim.heap = SimpleNamespace(h=None, cls={"Spring": 1, "Node": 0})
    sim.cls, sim.m_steps = 0, 0
    sim.args = (smmo.smmo_spring_args(0, 1, 1e-4, 0.3, 0) if cls is SpringSim else
                smmo.smmo_nbody_args(1.0, 1e-3, 1e-4, 0))
    asked = []
    monkeypatch.setattr(smmo, "smmo_parallel_do", lambda h, c, m, args, stream: asked.append(args.steps))
    sim.step(n)
    assert sum(asked) == n and len(asked) <= 4
