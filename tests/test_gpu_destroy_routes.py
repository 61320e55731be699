"""smmo_destroy: on a heap that has failed already, after an error of its own,
and on each of its routes (a few handles; many of them; handles that are few
beside a class of many blocks)."""

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


def fails(heap):
    with pytest.raises(smmo.SmmoError) as e:
        heap.sync()
    assert e.value.status == smmo.SMMO_EDEVICE


@pytest.mark.parametrize("n", [1, 64, 4000])
def test_a_failed_heap_is_left_alone(dev, n):
    """A block's last object is taken out of its bitmap behind the library's
    back, so that bringing the block states in line would show: after an error
    no destroy touches anything; once the error is cleared the next one does."""
    import torch

    heap, hd, b = make(dev, 200, 64 * 100 + 37)
    words = heap.buf[heap.base - heap.buf.data_ptr():]
    words = words[: words.numel() // 8 * 8].view(torch.int64)
    at = torch.nonzero(words == (1 << 37) - 1).flatten()
    assert at.numel() == 1                        # the last block's bitmap
    heap.destroy("A", b[:1])
    fails(heap)
    words[at] = 0
    free = heap.stats().free_blocks
    for _ in range(2):
        heap.destroy("A", hd[:n])
        fails(heap)
        st = heap.stats()
        assert st.free_blocks == free and st.device_deletes == 0
    smmo.smmo_clear_error(heap.h)
    heap.destroy("A", hd[:4000])
    heap.sync()
    st = heap.stats()
    assert st.device_deletes == 4000 and st.free_blocks == free + 62 + 1
    assert np.array_equal(keys_of(heap), np.arange(4000, 6400))
    clean(heap)
    heap.close()


@pytest.mark.parametrize("n", [128, 4000])
def test_an_error_of_the_call_itself(dev, n):
    """A bad handle among good ones: what the call has deleted before the error
    was seen is brought in line, and only by that call."""
    import torch

    heap, hd, b = make(dev, 200, 64 * 100)
    h = torch.cat([hd[:n], b[:1]])
    heap.destroy("A", h)
    fails(heap)
    st = heap.stats()
    assert st.live_objects[heap.cls["A"]] == 6400 - st.device_deletes
    clean(heap)
    heap.destroy("A", hd[n:])
    fails(heap)
    assert heap.stats().device_deletes == st.device_deletes
    smmo.smmo_clear_error(heap.h)
    heap.destroy("A", hd[n:])
    heap.sync()
    assert heap.stats().device_deletes == st.device_deletes + 6400 - n
    clean(heap)
    heap.close()


# classes of 100, 1,600 and 20,000 blocks; requests on both sides of 16 handles
@pytest.mark.parametrize("n", [6400 - 3, 64 * 1600 - 3, 64 * 20000 - 3])
@pytest.mark.parametrize("shuffled", [False, True])
def test_requests_of_all_sizes(dev, n, shuffled):
    heap, hd, b = make(dev, (n + 63) // 64 + 8, n)
    requests(dev, heap, hd, n, shuffled, (1, 2, 15, 16, 17, 63, 64, 65, 255, 257, 1000, 4096, 5000, 20000, 70000, n))
    heap.close()


@pytest.mark.parametrize("shuffled", [False, True])
def test_few_handles_of_a_class_of_many_blocks(dev, shuffled):
    """A class whose bound of blocks is past the line (it grows with every
    parallel_new): requests on both sides of one handle in 32 blocks, with
    objects named twice by lanes of one and of different wavefronts."""
    import torch

    half = 1 << 18
    heap = smmo.Heap({"A": [("key", "i32", 1)]}, blocks=2 * half + 64)
    for _ in range(2):
        hd = heap.new("A", 64 * half, key=torch.zeros(64 * half, dtype=torch.int32, device=dev))
        heap.destroy("A", hd.clone())
    n = 200003
    hd = heap.new("A", n, key=torch.arange(n, dtype=torch.int32, device=dev)).clone()
    gone = requests(dev, heap, hd, n, shuffled, (17, 64, 65, 1000, 4096, 16384, 16386, 16387, 30000))
    left = np.flatnonzero(~gone)
    twice = np.concatenate([left[:300], left[100:101], left[:200:7]])
    heap.destroy("A", hd[torch.from_numpy(twice).to(dev)])
    fails(heap)
    smmo.smmo_clear_error(heap.h)
    assert np.isin(left[300:], keys_of(heap)).all()         # nothing but what was named is gone
    assert heap.stats().live_objects[0] == 2 * 64 * half + n - heap.stats().device_deletes
    clean(heap)
    heap.close()


def requests(dev, heap, hd, n, shuffled, sizes):
    import torch

    order = np.random.default_rng(n).permutation(n) if shuffled else np.arange(n)
    lo, gone, before = 0, np.zeros(n, bool), heap.stats().device_deletes
    for k in sizes:
        part = order[lo:lo + k]
        if not part.size:
            break
        lo += k
        heap.destroy("A", hd[torch.from_numpy(part).to(dev)])
        gone[part] = True
        assert np.array_equal(keys_of(heap), np.flatnonzero(~gone)), k
        clean(heap)
    assert heap.stats().device_deletes - before == gone.sum()
    # a deleted object's handle, now bad
    heap.destroy("A", hd[torch.from_numpy(order[:1]).to(dev)])
    fails(heap)
    smmo.smmo_clear_error(heap.h)
    clean(heap)
    return gone
