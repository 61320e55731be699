"""Block lists at the edges of the enumeration's work-groups: 64 containers of
64 blocks each, in block order up to 1,024 containers, 256 a work-group beyond
16,384.  Against a plain model: which objects a gather returns (in no order),
that a packed walk visits each object once, and a snapshot the objects that
were there when it was taken."""

import numpy as np
import pytest

from paper_1908_05845_amd import smmo
from test_gpu_heap import cfg, clean

pytestmark = pytest.mark.gpu

CLASSES = {"A": [("x", "f32", 1), ("key", "i32", 1)], "B": [("key", "i32", 1)]}

EDGES = [1, 63, 64, 65, 64 * 64 - 1, 64 * 64, 64 * 64 + 1, 65536, 65537, 64 * 16384, 64 * 16384 + 1]


@pytest.mark.parametrize("packing", [0, 2])
@pytest.mark.parametrize("blocks", EDGES)
def test_lists_at_the_edges(dev, blocks, packing):
    import torch

    print("blocks %d packing %d" % (blocks, packing), flush=True)
    heap = smmo.Heap(CLASSES, blocks=blocks, cfg=cfg(sparse_packing=packing, bulk_ordered=0))
    rng = np.random.default_rng(blocks)
    # blocks from the first to the last of the heap in use: full heaps where
    # that is cheap, else filler objects of class B between A's
    n = 64 * blocks if blocks <= 65 else 0
    ids = np.arange(blocks)
    if n == 0:
        some = np.unique(np.concatenate([rng.choice(blocks, 700), ids[:70], ids[-70:], [4095, 4096] if blocks > 4097 else []])).astype(np.int64)
        fill = torch.zeros(64 * blocks, dtype=torch.int32, device=dev)
        b = heap.new("B", 64 * blocks, key=fill).clone()
        at = torch.zeros(blocks, dtype=torch.bool, device=dev)
        at[torch.from_numpy(some).to(dev)] = True
        heap.destroy("B", b[at[(b >> 6).long()]])
        ids, n = some, 64 * some.size
    hd = heap.new("A", n, x=torch.zeros(n, device=dev), key=torch.arange(n, dtype=torch.int32, device=dev)).clone()
    h = hd.cpu().numpy()
    assert np.array_equal(np.unique(h >> 6), ids)
    # leave blocks with 1 .. 64 objects
    keep = rng.random(n) < np.repeat(rng.random(n // 64), 64)
    keep[0] = keep[-1] = True
    if not keep.all():
        heap.destroy("A", hd[torch.from_numpy(~keep).to(dev)])

    def rows():
        g = heap.gather("A", ["x", "key"], capacity=n + 2000)
        return g["_handle"].cpu().numpy(), g["key"].cpu().numpy(), g["x"].cpu().numpy()

    got, key, _ = rows()
    assert np.array_equal(np.sort(got), np.sort(h[keep]))
    # a walk (packed if packing is 2) visits each object once
    heap.do("A", "test.axpy", smmo.smmo_axpy_args(1.0, 1.0))
    heap.do("A", "test.axpy", smmo.smmo_axpy_args(1.0, 1.0))
    _, _, x = rows()
    assert np.array_equal(x, np.full(x.size, 2.0, np.float32))
    # a snapshot lists what was there before new objects came into the holes
    new = min(int((~keep).sum()), 1000)
    heap.snapshot("A")
    if new:
        heap.new("A", new, x=torch.zeros(new, device=dev),
                 key=torch.arange(n, n + new, dtype=torch.int32, device=dev))
    heap.do("A", "test.axpy", smmo.smmo_axpy_args(1.0, 1.0))
    _, key, x = rows()
    assert np.array_equal(np.sort(key), np.concatenate([np.flatnonzero(keep), np.arange(n, n + new)]))
    assert np.array_equal(x, np.where(key < n, 3.0, 0.0).astype(np.float32))
    clean(heap)
    heap.close()


def test_an_empty_class(dev):
    heap = smmo.Heap(CLASSES, blocks=200)
    g = heap.gather("A", ["key"])
    assert g["key"].numel() == 0
    heap.do("A", "test.axpy", smmo.smmo_axpy_args(1.0, 1.0))
    clean(heap)
    heap.close()
