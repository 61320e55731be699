"""Captured graphs replayed after their classes have grown: the launches hold
for the lists that they find, not for those that they were captured on."""

import numpy as np
import pytest

from inputs import nbody_init, spring_mesh
from oracle import nbody_force_at
from paper_1908_05845_amd.sims import NbodySim, SpringSim
from test_gpu_heap import clean

pytestmark = pytest.mark.gpu

DT, EPS = 1e-4, 1e-3


def captured(step):
    import torch

    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        step(torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return g


def add_bodies(sim, s, lo, hi):
    import torch

    t = lambda a: torch.from_numpy(np.ascontiguousarray(a[lo:hi])).to(sim.heap.dev)
    sim.heap.new("Body", hi - lo, pos_x=t(s["x"]), pos_y=t(s["y"]), vel_x=t(s["vx"]), vel_y=t(s["vy"]),
                 mass=t(s["m"]), id=torch.arange(lo, hi, dtype=torch.int32, device=sim.heap.dev))


def check_pass(before, after, n, G, moved):
    """One force pass (and move) from `before`: the forces against float64 (the
    tolerance of the other n-body tests), the move against the stored forces to
    four roundings of its terms."""
    assert np.array_equal(before["id"], np.arange(n)) and np.array_equal(after["id"], before["id"])
    at = np.unique(np.concatenate([np.arange(min(n, 200)), np.arange(max(0, n - 400), n)]))
    ref = nbody_force_at(before["x"], before["y"], before["m"], float(np.float32(G)), float(np.float32(EPS)), at)
    for c, f in enumerate(("fx", "fy")):
        err = np.abs(after[f][at] - ref[c])
        assert np.all(err <= 1e-5 * ref[2 + c]), (f, float(np.max(err / ref[2 + c])))
    if not moved:
        assert np.array_equal(after["x"], before["x"]) and np.array_equal(after["vx"], before["vx"])
        return
    dt, u = np.float64(np.float32(DT)), 4 * 2.0 ** -24
    for f, v, x in (("fx", "vx", "x"), ("fy", "vy", "y")):
        dv = after[f].astype(np.float64) / before["m"] * dt
        assert np.all(np.abs(after[v] - (before[v] + dv)) <= u * (np.abs(before[v]) + np.abs(dv))), v
        dx = after[v].astype(np.float64) * dt
        assert np.all(np.abs(after[x] - (before[x] + dx)) <= u * (np.abs(before[x]) + np.abs(dx))), x


# bounds at the capture of 6 blocks (no pair form), 13 and 14 (one group of two
# blocks ends with the list, or after it), 98, 226 and 513 (groups of four), 1537
@pytest.mark.parametrize("blocks", [5, 12, 13, 97, 225, 512, 1536])
@pytest.mark.parametrize("steps", [False, True])
def test_nbody_replays_after_growth(dev, blocks, steps):
    grow = (1, 1, 2, 4, 20)
    n, total = 64 * blocks, 64 * (blocks + sum(grow))
    s, G = nbody_init(total, seed=blocks), 1.0 / total
    s["vx"], s["vy"] = (np.random.default_rng(blocks).normal(size=(2, total)) * 0.1).astype(np.float32)
    sim = NbodySim({k: v[:n] for k, v in s.items()}, G, EPS, DT, extra_blocks=sum(grow) + 4)
    sim.force()                                   # (the workspace is there)
    g = captured((lambda st: sim.step(1, stream=st)) if steps else (lambda st: sim.force(stream=st)))
    for k in grow:
        add_bodies(sim, s, n, n + 64 * k)
        n += 64 * k
        before = sim.read()                       # (the list is built anew)
        g.replay()
        sim.heap.sync()
        check_pass(before, sim.read(), n, G, steps)
    sim.heap.close()


def add_mesh(sim, mesh, n0, s0):
    """A further mesh in the heap of a SpringSim, with ids from n0 and s0 on."""
    import torch

    heap, dev = sim.heap, sim.heap.dev
    f = lambda k: torch.from_numpy(mesh[k]).to(dev)
    N, S = mesh["x"].size, mesh["a"].size
    nodes = heap.new("Node", N, x=f("x"), y=f("y"), vx=f("vx"), vy=f("vy"), m=f("m"),
                     adj=torch.full((8 * N,), -1, dtype=torch.int32, device=dev),
                     id=torch.arange(n0, n0 + N, dtype=torch.int32, device=dev)).clone()
    heap.new("Spring", S, a=nodes[f("a").long()], b=nodes[f("b").long()], k=f("k"), L0=f("L0"),
             slot_a=f("slot_a").to(torch.uint8), slot_b=f("slot_b").to(torch.uint8),
             id=torch.arange(s0, s0 + S, dtype=torch.int32, device=dev))
    heap.do("Spring", "spring.link", sim.args)


def by_id(heap, cname, names):
    g = heap.gather(cname, ["id"] + names)
    o = np.argsort(g["id"].cpu().numpy())
    return {f: g[f].cpu().numpy()[o] for f in ["id"] + names}


# bounds at the capture of 17 and 45 blocks (the smaller form), 32 and 89 (the larger)
@pytest.mark.parametrize("W,H", [(33, 29), (45, 43)])
def test_spring_steps_replays_after_growth(dev, W, H):
    """One launch's worth of blocks at the capture, more at the replays, among
    them springs that break: every array and the heap as the do-alls leave them."""
    first, more = spring_mesh(W, H, seed=3, v_sigma=3.0), spring_mesh(24, 22, seed=9, v_sigma=3.0)
    a, b = (SpringSim(first, 1e-4, 0.05, extra_blocks=200) for _ in range(2))
    g = captured(lambda st: a.step(5, stream=st))
    n, s = first["x"].size, first["a"].size
    for lap in range(4):
        if lap:
            for sim in (a, b):
                add_mesh(sim, more, n, s)
            n, s = n + more["x"].size, s + more["a"].size
        a.heap.gather("Node", ["id"])             # (the lists are built anew)
        a.heap.gather("Spring", ["id"])
        g.replay()
        a.heap.sync()
        for _ in range(5):
            b.spring_force()
            b.node_update()
        for cname, names in (("Node", ["x", "y", "vx", "vy"]), ("Spring", ["fx", "fy"])):
            ra, rb = by_id(a.heap, cname, names), by_id(b.heap, cname, names)
            for f in ra:
                assert np.array_equal(ra[f], rb[f]), (lap, cname, f)
        assert a.heap.stats().free_blocks == b.heap.stats().free_blocks
        assert a.heap.stats().device_deletes == b.heap.stats().device_deletes
        clean(a.heap)
    assert a.heap.stats().device_deletes > 0
    a.heap.close()
    b.heap.close()
