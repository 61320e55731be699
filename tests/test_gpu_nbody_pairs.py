"""The pair form of the n-body force (each pair evaluated once) against the
float64 oracle on the same float32 state: class sizes on both sides of every
choice of work-group and segment, with remainders, with free slots inside the
listed blocks, unsoftened with coincident bodies, and in units whose products
of masses and inverse distances leave float32's range long before the force
does.  Tolerance: 1e-5 of each force's conditioning scale, as for the other
n-body tests."""

import numpy as np
import pytest

from inputs import nbody_init
from oracle import nbody_force_at
from paper_1908_05845_amd.sims import NbodySim

pytestmark = pytest.mark.gpu

TOL = 1e-5


def force_at(x, y, m, G, eps, at):
    """The oracle's forces and scales; unsoftened, where the oracle has no
    value for two bodies at one place, the same sums in float64 with such a
    pair (like a body with itself) left out."""
    if eps > 0:
        return nbody_force_at(x, y, m, G, eps, at)
    x, y, m = (a.astype(np.float64) for a in (x, y, m))
    dx, dy = x - x[at, None], y - y[at, None]
    r2 = dx * dx + dy * dy
    w = G * m * m[at, None] * np.where(r2 > 0, r2, np.inf) ** -1.5
    return (w * dx).sum(1), (w * dy).sum(1), np.abs(w * dx).sum(1), np.abs(w * dy).sum(1)


def check(sim, s, keep, G, eps, seed):
    sim.force()
    g = sim.heap.gather("Body", ["id", "force_x", "force_y"])
    sim.heap.sync()
    ids = g["id"].cpu().numpy()
    assert np.array_equal(np.sort(ids), keep)
    f = np.zeros((2, s["x"].size))
    f[0, ids], f[1, ids] = g["force_x"].cpu().numpy(), g["force_y"].cpu().numpy()
    rng = np.random.default_rng(seed)
    at = np.unique(np.concatenate([np.arange(min(200, keep.size)), np.arange(max(0, keep.size - 200), keep.size),
                                   rng.integers(0, keep.size, 400)]))
    ref = force_at(s["x"][keep], s["y"][keep], s["m"][keep], G, eps, at)
    for c in range(2):
        err = np.abs(f[c, keep[at]] - ref[c])
        assert np.all(err <= TOL * ref[2 + c]), float(np.max(err / np.maximum(ref[2 + c], 1e-300)))


@pytest.mark.parametrize("n", [64 * 10, 64 * 11, 64 * 11 + 1, 1217, 5003, 64 * 95, 64 * 95 + 1, 64 * 223 - 1, 64 * 223 + 1,
                               64 * 511, 64 * 511 + 1, 40000, 64 * 1535, 64 * 1535 + 1])
def test_class_sizes(dev, n):
    s = nbody_init(n, seed=n)
    sim = NbodySim(s, 1.0 / n, 1e-3, 1e-4)
    check(sim, s, np.arange(n), float(np.float32(1.0 / n)), float(np.float32(1e-3)), n)
    sim.heap.close()


@pytest.mark.parametrize("n", [3000, 30000])
@pytest.mark.parametrize("eps", [1e-3, 0.0])
def test_free_slots_and_coincident_bodies(dev, n, eps):
    import torch

    s = nbody_init(n, seed=7)
    for a, b in ((3, 5), (10, n - 1), (64, 2000)):       # pairs at one place
        s["x"][a], s["y"][a] = s["x"][b], s["y"][b]
    sim = NbodySim(s, 1.0 / n, eps, 1e-4)
    gone = np.unique(np.random.default_rng(1).integers(0, n, n // 3))
    sim.heap.destroy("Body", sim.handles[torch.from_numpy(gone).to(dev)])
    check(sim, s, np.setdiff1d(np.arange(n), gone), float(np.float32(1.0 / n)), float(np.float32(eps)), 3)
    sim.heap.close()


def test_units_far_from_one(dev):
    """Metres and kilograms: distances of 1e10 to 1e13, masses of 1e20 to 1e30."""
    n = 4000
    rng = np.random.default_rng(2)
    s = nbody_init(n, seed=2)
    s["x"], s["y"] = (5e12 * s["x"]).astype(np.float32), (5e12 * s["y"]).astype(np.float32)
    s["m"] = (10.0 ** rng.uniform(20, 30, n)).astype(np.float32)
    G = float(np.float32(6.674e-11))
    sim = NbodySim(s, G, 1e8, 1.0)
    check(sim, s, np.arange(n), G, float(np.float32(1e8)), 4)
    sim.heap.close()
