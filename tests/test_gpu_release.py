"""Deletion of handles in any order: the lanes of a wavefront release all
their blocks side by side.  Against a plain model of the live set and the
block-state invariants; handles in creation order (one block a wavefront),
strided (each lane its own block) and shuffled, in batches that leave blocks
full, partly filled and empty; an object named twice by one wavefront."""

import numpy as np
import pytest

from paper_1908_05845_amd import smmo
from test_gpu_heap import clean, keys_of

pytestmark = pytest.mark.gpu

CLASSES = {"A": [("x", "f32", 1), ("key", "i32", 1)], "B": [("key", "i32", 1), ("x", "f32", 1)]}


@pytest.mark.parametrize("n", [1, 64, 65, 4096, 5003, 70000])
@pytest.mark.parametrize("order", ["created", "strided", "shuffled"])
def test_destroy_in_any_order(dev, n, order):
    import torch

    heap = smmo.Heap(CLASSES, blocks=2 * ((n + 63) // 64) + 4)
    rng = np.random.default_rng(n)
    for lap in range(2):                    # the second lap reuses freed blocks
        hd = heap.new("A", n, key=torch.arange(n, dtype=torch.int32, device=dev)).clone()
        perm = {"created": np.arange(n), "strided": np.argsort(np.arange(n) % 64, kind="stable"),
                "shuffled": rng.permutation(n)}[order]
        left = set(range(n))
        before = heap.stats()
        for part in np.array_split(perm, 3):
            if part.size:
                heap.destroy("A", hd[torch.from_numpy(part).to(dev)])
            left -= set(part.tolist())
            heap.sync()
            assert np.array_equal(keys_of(heap), np.array(sorted(left), np.int32))
            clean(heap)
        st = heap.stats()
        assert st.free_blocks == st.total_blocks and st.device_deletes - before.device_deletes == n
    heap.close()


def test_an_object_named_twice_is_released_once(dev):
    import torch

    heap = smmo.Heap(CLASSES, blocks=16)
    hd = heap.new("A", 300, key=torch.arange(300, dtype=torch.int32, device=dev)).clone()
    pick = torch.tensor([5, 70, 5, 140, 299], device=dev)
    heap.destroy("A", hd[pick])
    with pytest.raises(smmo.SmmoError) as e:
        heap.sync()
    assert e.value.status == smmo.SMMO_EDEVICE
    smmo.smmo_clear_error(heap.h)
    want = np.setdiff1d(np.arange(300), [5, 70, 140, 299]).astype(np.int32)
    assert np.array_equal(keys_of(heap), want)
    assert heap.stats().device_deletes == 4
    clean(heap)
    heap.close()
