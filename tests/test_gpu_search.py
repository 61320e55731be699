"""Searches of the block bitmaps on heaps of one to four levels: objects made
by the device allocator next to a class that holds most blocks, deleted and
made again, with and without bitmap rotation, against the live set, distinct
handles and the block-state invariants."""

import numpy as np
import pytest

from paper_1908_05845_amd import smmo
from test_gpu_heap import cfg, clean, keys_of

pytestmark = pytest.mark.gpu

CLASSES = {"A": [("key", "i32", 1)], "B": [("key", "i32", 1)]}


@pytest.mark.parametrize("rotation", [0, 1])
@pytest.mark.parametrize("blocks", [1, 63, 64, 65, 4095, 4097, 270000])
def test_device_allocation_between_other_blocks(dev, blocks, rotation):
    import torch

    if rotation == 0 and blocks > 4097:
        pytest.skip("without rotation every search starts at one block: slow by design on a large heap")
    heap = smmo.Heap(CLASSES, blocks=blocks, cfg=cfg(bulk_ordered=0, rotation=rotation))
    # without rotation every request queues at one block: fewer of them
    room = 64 * blocks if rotation else min(64 * blocks, 30000)
    nb = room // 2 if blocks > 1 else 0
    if nb:
        heap.new("B", nb, key=torch.arange(nb, dtype=torch.int32, device=dev))
    n = room // 4 + 1
    hd = heap.new("A", n, key=torch.arange(n, dtype=torch.int32, device=dev)).clone()
    heap.sync()
    assert torch.unique(hd).numel() == n
    clean(heap)
    heap.destroy("A", hd[::2])
    m = n // 3
    heap.new("A", m, key=torch.arange(n, n + m, dtype=torch.int32, device=dev))
    heap.sync()
    want = np.concatenate([np.arange(n)[1::2], np.arange(n, n + m)]).astype(np.int32)
    assert np.array_equal(keys_of(heap), want)
    assert heap.gather("B")["_count"] == nb
    clean(heap)
    heap.close()
