"""The pair form's workspace: taken from the heap's allocator, bounded while a
class grows, given back, and done without where there is none (the allocator
refuses; a graph captured before any force pass)."""

import numpy as np
import pytest

from inputs import nbody_init
from paper_1908_05845_amd import smmo
from paper_1908_05845_amd.sims import NBODY_CLASSES
from test_gpu_graph_growth import DT, EPS, captured, check_pass

pytestmark = pytest.mark.gpu


class Bodies:
    """An n-body simulation whose class grows, on a heap whose memory comes from
    the allocator set."""

    def __init__(self, s, n, G, blocks):
        self.heap = smmo.Heap(NBODY_CLASSES, blocks=blocks, from_allocator=True)
        self.s, self.n = s, 0
        self.cls = self.heap.cls["Body"]
        self.args = smmo.smmo_nbody_args(G, EPS, DT, 0)
        self.grow(n)

    def grow(self, k):
        import torch

        lo, hi, s = self.n, self.n + k, self.s
        t = lambda a: torch.from_numpy(np.ascontiguousarray(a[lo:hi])).to(self.heap.dev)
        self.heap.new("Body", k, pos_x=t(s["x"]), pos_y=t(s["y"]), vel_x=t(s["vx"]), vel_y=t(s["vy"]),
                      mass=t(s["m"]), id=torch.arange(lo, hi, dtype=torch.int32, device=self.heap.dev))
        self.n = hi

    def force(self, stream=None):
        self.heap.do("Body", "nbody.force", self.args, stream)

    def step(self, n, stream=None):
        a = self.args
        self.heap.do("Body", "nbody.steps", smmo.smmo_nbody_steps_args(a.G, a.eps, a.dt, n), stream)

    def read(self):
        g = self.heap.gather("Body")
        o = np.argsort(g["id"].cpu().numpy())
        names = dict(x="pos_x", y="pos_y", vx="vel_x", vy="vel_y", fx="force_x", fy="force_y", m="mass", id="id")
        return {k: g[f].cpu().numpy()[o] for k, f in names.items()}


class Counted(smmo.TorchDeviceAllocator):
    """Refuses all but the first `most` requests; remembers what is out."""

    def __init__(self, most=1 << 30):
        super().__init__()
        self.most, self.sizes, self.peak = most, {}, 0

    def alloc(self, nbytes):
        if self.allocs >= self.most:
            return 0
        p = super().alloc(nbytes)
        self.sizes[p] = nbytes
        self.peak = max(self.peak, sum(self.sizes.values()))
        return p

    def release(self, ptr, nbytes):
        assert self.sizes.pop(ptr) == nbytes
        super().release(ptr, nbytes)


@pytest.fixture
def counted():
    made = []

    def make(most=1 << 30):
        a = Counted(most)
        smmo.smmo_set_allocator(a.alloc, a.release)
        made.append(a)
        return a

    yield make
    smmo.smmo_set_allocator(None)


# what the largest class that takes the pair form needs: 1,536 blocks in groups
# of 256 bodies and segments of 1,024: 384 rows of 98,304 sums of 8 bytes
LARGEST = 384 * 98304 * 8


def total(blocks):
    s = nbody_init(64 * blocks, seed=blocks)
    return s, 1.0 / (64 * blocks)


def test_growth_is_bounded_and_given_back(dev, counted):
    a = counted()
    s, G = total(1540)
    sim = Bodies(s, 64 * 20, G, 1560)
    base = a.peak
    for blocks in (60, 100, 300, 520, 700, 900, 1100, 1300, 1400, 1500, 1530):
        sim.grow(64 * blocks - sim.n)
        sim.force()
        held = sum(a.sizes.values()) - base
        assert held <= LARGEST, (blocks, held)    # the one in use, no larger than any class needs
    before = sim.read()
    sim.force()
    sim.heap.sync()
    check_pass(before, sim.read(), sim.n, G, False)
    sim.heap.close()
    assert not a.sizes and a.allocs == a.releases


def test_graphs_keep_theirs(dev, counted):
    a = counted()
    s, G = total(400)
    sim = Bodies(s, 64 * 60, G, 420)
    sim.force()
    g = captured(lambda st: sim.step(1, stream=st))
    for blocks in (70, 150, 300):                 # the plan of the capture, then larger ones
        sim.grow(64 * blocks - sim.n)
        sim.force()
        before = sim.read()
        g.replay()
        sim.heap.sync()
        check_pass(before, sim.read(), sim.n, G, True)
    sim.heap.close()
    assert not a.sizes and a.allocs == a.releases


@pytest.mark.parametrize("blocks", [20, 600])
def test_a_refused_workspace(dev, counted, blocks):
    a = counted(1)                                # the heap's own buffer and nothing else
    s, G = total(blocks)
    sim = Bodies(s, 64 * blocks, G, blocks + 8)
    for moved in (False, True):
        before = sim.read()
        sim.step(1) if moved else sim.force()
        sim.heap.sync()
        check_pass(before, sim.read(), sim.n, G, moved)
    sim.heap.close()
    assert a.allocs == a.releases == 1


@pytest.mark.parametrize("blocks", [20, 600])
def test_captured_before_any_force_pass(dev, counted, blocks):
    """No workspace may be taken under capture: the graph's two steps are those
    of the two do-alls, each checked against float64 on the state before it."""
    a = counted()
    s, G = total(blocks)
    sim, ref = (Bodies(s, 64 * blocks, G, blocks + 8) for _ in range(2))
    for b in (sim, ref):
        b.heap.do("Body", "nbody.update", b.args)  # the list and the modules, no workspace
    one = captured(lambda st: sim.step(1, stream=st))
    two = captured(lambda st: ref.step(2, stream=st))
    assert a.allocs == 2
    for _ in range(2):
        for lap in range(2):
            before = sim.read()
            one.replay()
            sim.heap.sync()
            check_pass(before, sim.read(), sim.n, G, True)
        two.replay()
        ref.heap.sync()
        x, y = sim.read(), ref.read()
        for f in x:
            assert np.array_equal(x[f], y[f]), f
    sim.heap.close()
    ref.heap.close()
