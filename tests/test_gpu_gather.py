"""smmo_gather_soa against the arrays the objects were created from: sizes
around a wavefront's block, a work-group's share of the block list and its
1,024-entry pass over it; holes left by deletions; inner arrays whose rows
take 16-byte stores and destinations that do not allow them; capacities below
the number of objects.  Copies are exact, so the comparison is too."""

import numpy as np
import pytest

from paper_1908_05845_amd import smmo

pytestmark = pytest.mark.gpu

FIELDS = [("key", "i32", 1), ("w", "f32", 4), ("v", "u32", 3), ("t", "u8", 1), ("s", "u8", 2), ("z", "f32", 8)]
CLASSES = {"A": FIELDS, "B": [("key", "i32", 1)]}


def values(n, torch, dev, seed):
    g = torch.Generator(device=dev).manual_seed(seed)
    word = lambda m: torch.randint(-2 ** 31, 2 ** 31, (m,), generator=g, device=dev, dtype=torch.int64).int()
    byte = lambda m: torch.randint(0, 256, (m,), generator=g, device=dev, dtype=torch.uint8)
    return {"key": torch.arange(n, dtype=torch.int32, device=dev), "w": word(4 * n).view(torch.float32), "v": word(3 * n),
            "t": byte(n), "s": byte(2 * n), "z": word(8 * n).view(torch.float32)}


@pytest.mark.parametrize("n,keep,shift", [(1, 1, 0), (63, 1, 1), (64, 2, 0), (65, 1, 0), (1024, 3, 2), (1025, 1, 3),
                                          (64 * 511, 1, 0), (64 * 8192 + 17, 5, 0), (64 * 8209 + 1, 1, 1)])
def test_gather_returns_every_live_object(dev, n, keep, shift):
    """keep: every keep-th object survives; shift: words by which the
    destinations are moved off a 16-byte boundary."""
    import torch

    heap = smmo.Heap(CLASSES, blocks=(n + 63) // 64 + 8)
    heap.new("B", 70, key=torch.arange(70, dtype=torch.int32, device=dev))
    vals = values(n, torch, dev, n)
    handles = heap.new("A", n, **vals).clone()
    ids = np.arange(n)
    if keep > 1:
        heap.destroy("A", handles[torch.arange(n, device=dev) % keep != 0])
        ids = ids[ids % keep == 0]
    names = [f[0] for f in FIELDS]
    for capacity in (n, max(1, len(ids) // 2)):
        out, ptr = {}, []
        for f, dt, cnt in FIELDS:
            size = 1 if dt == "u8" else 4
            buf = torch.zeros(capacity * cnt * size + 4 * shift + 16, dtype=torch.uint8, device=dev)
            out[f] = buf[4 * shift:4 * shift + capacity * cnt * size]
            ptr.append(out[f].data_ptr())
        hd = torch.zeros(capacity, dtype=torch.int32, device=dev)
        count = torch.full((1,), -1, dtype=torch.int32, device=dev)
        smmo.smmo_gather_soa(heap.h, heap.cls["A"], [heap.fields["A"][f][0] for f in names], ptr, hd, capacity, count)
        heap.sync()
        assert int(count.item()) == len(ids)
        got = min(capacity, len(ids))
        key = out["key"].view(torch.int32)[:got].cpu().numpy()
        assert len(np.unique(key)) == got and np.isin(key, ids).all()
        assert np.array_equal(hd[:got].cpu().numpy(), handles.cpu().numpy()[key])
        for f, dt, cnt in FIELDS:
            size = 1 if dt == "u8" else 4
            want = vals[f].view(torch.uint8).reshape(n, cnt * size).cpu().numpy()[key]
            assert np.array_equal(out[f].reshape(capacity, cnt * size)[:got].cpu().numpy(), want), f
    assert heap.gather("B")["_count"] == 70
    heap.close()


def test_gather_passes_over_long_shares(dev):
    """More list entries per work-group than it takes in one pass: 1,024."""
    import torch

    n = 64 * (512 * 1024 + 700) + 5
    heap = smmo.Heap({"C": [("key", "i32", 1)]}, blocks=n // 64 + 2)
    heap.new("C", n, key=torch.arange(n, dtype=torch.int32, device=dev))
    for _ in range(2):                     # the second starts from the counter the first left
        g = heap.gather("C")
        assert g["_count"] == n
        assert torch.equal(torch.sort(g["key"])[0], torch.arange(n, dtype=torch.int32, device=dev))
    heap.close()
