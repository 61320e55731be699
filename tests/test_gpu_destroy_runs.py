"""smmo_destroy in two launches (slots, then block states) and the ordered
bulk claim that takes the freed blocks again, against a plain model of the
live set and the block-state invariants.

Runs of neighbouring handles around the length from which a wavefront makes
one release of them; objects named twice and handles of another class in any
of them; heaps of two, three and more than 1,024 containers' levels."""

import numpy as np
import pytest

from paper_1908_05845_amd import smmo
from test_gpu_heap import clean, keys_of

pytestmark = pytest.mark.gpu

CLASSES = {"A": [("x", "f32", 1), ("key", "i32", 1)], "B": [("key", "i32", 1), ("x", "f32", 1)]}


def make(dev, blocks, n):
    import torch

    heap = smmo.Heap(CLASSES, blocks=blocks)
    b = heap.new("B", 100, key=torch.arange(100, dtype=torch.int32, device=dev)).clone()
    hd = heap.new("A", n, key=torch.arange(n, dtype=torch.int32, device=dev)).clone()
    return heap, hd, b


@pytest.mark.parametrize("run", [1, 7, 8, 9, 33, 64])
@pytest.mark.parametrize("blocks,n", [(40, 2001), (5000, 300001)])
def test_runs_of_handles(dev, blocks, n, run):
    import torch

    heap, hd, b = make(dev, blocks, n)
    rng = np.random.default_rng(run)
    runs = [np.arange(i, min(i + run, n)) for i in range(0, n, run)]
    rng.shuffle(runs)
    order = np.concatenate(runs)
    cut = order.size // 3
    live = np.arange(n)
    for part in (order[:cut], order[cut:]):
        heap.destroy("A", hd[torch.from_numpy(part).to(dev)])
        heap.sync()
        live = np.setdiff1d(live, part)
        assert np.array_equal(keys_of(heap), live)
        clean(heap)
    st = heap.stats()
    assert st.free_blocks == st.total_blocks - 2 and st.device_deletes == n
    assert keys_of(heap, "B").size == 100
    heap.close()


@pytest.mark.parametrize("run", [1, 8, 64])
def test_bad_handles_among_good_ones(dev, run):
    """An object named twice (in one run, and far apart), a handle of another
    class, one beyond the heap and one of a deleted object: the error is
    reported, the objects that the handles name are gone, once."""
    import torch

    heap, hd, b = make(dev, 200, 6000)
    gone0 = np.arange(640, 650)
    heap.destroy("A", hd[torch.from_numpy(gone0).to(dev)])
    h = hd.cpu().numpy()
    runs = [np.arange(i, i + run) for i in range(0, 1280, 2 * run)]
    pick = np.setdiff1d(np.concatenate(runs), gone0)
    handles = np.concatenate([h[pick], h[pick[:1]], h[pick[-run:]]])
    handles = np.concatenate([handles, h[pick[:1]], b.cpu().numpy()[:1], np.array([200 << 6], h.dtype), h[gone0[:1]]])
    # one wavefront's worth, so that no part of it is skipped for the error of another
    for part in np.array_split(handles, (handles.size + 63) // 64):
        heap.destroy("A", torch.from_numpy(part).to(dev))
        try:
            heap.sync()
        except smmo.SmmoError as e:
            assert e.status == smmo.SMMO_EDEVICE
            smmo.smmo_clear_error(heap.h)
    live = np.setdiff1d(np.arange(6000), np.concatenate([pick, gone0]))
    assert np.array_equal(keys_of(heap), live)
    assert heap.stats().device_deletes == 6000 - live.size
    assert keys_of(heap, "B").size == 100
    clean(heap)
    with pytest.raises(smmo.SmmoError):
        heap.destroy("A", b[:1])
        heap.sync()
    smmo.smmo_clear_error(heap.h)
    heap.close()


@pytest.mark.parametrize("n", [64, 64 * 64 + 1, 64 * 70001 + 17])
def test_bulk_claim_over_holes(dev, n):
    """The ordered claim takes the lowest free blocks: after every third block
    was freed, new objects fill the holes first, in order."""
    import torch

    blocks = 2 * ((n + 63) // 64) + 8
    heap, hd, b = make(dev, blocks, n)
    key = torch.arange(n, device=dev)
    hole = (key // 64) % 3 == 1
    heap.destroy("A", hd[hole])
    m = int(hole.sum()) + 64 * 5 + 3
    holes = np.unique((hd[hole] >> 6).cpu().numpy())
    new = heap.new("A", m, key=torch.arange(n, n + m, dtype=torch.int32, device=dev))
    took = np.unique((new >> 6).cpu().numpy())
    assert np.array_equal(new.cpu().numpy()[:: 64] >> 6, took)      # ascending
    assert np.array_equal(took[: holes.size], holes)
    heap.sync()
    want = np.concatenate([np.flatnonzero(~hole.cpu().numpy()), np.arange(n, n + m)])
    assert np.array_equal(keys_of(heap), want)
    clean(heap)
    heap.close()
