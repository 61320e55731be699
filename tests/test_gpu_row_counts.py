"""Neighbour counts of the cellular automata on boards whose blocks hold runs
of a row (64 consecutive cells), hold none, or both: widths around 64 and its
multiples, boards of one and two rows, cells created out of order.  Against
the sum of the eight shifted boards."""

import numpy as np
import pytest

from paper_1908_05845_amd import smmo
from paper_1908_05845_amd.sims import GENERATION_CLASSES, GOL_CLASSES

pytestmark = pytest.mark.gpu

BOARDS = [(1, 130), (2, 100), (63, 7), (64, 1), (64, 2), (64, 5), (65, 64), (66, 66), (127, 4), (128, 1), (128, 5),
          (129, 128), (192, 3), (4096, 2), (5000, 3)]


def neighbours(v):
    return sum(np.roll(v, (dy, dx), (0, 1)) for dy in (-1, 0, 1) for dx in (-1, 0, 1) if (dy, dx) != (0, 0))


def counts(dev, classes, W, H, init, ids, args_of, method, group):
    import torch

    n = W * H
    heap = smmo.Heap(classes, blocks=3 * ((n + 63) // 64) + 4)
    hd = heap.new("Cell", n, state=torch.from_numpy(init[ids]).to(dev), cell_id=torch.from_numpy(ids).to(dev)).clone()
    cells = torch.empty_like(hd)
    cells[torch.from_numpy(ids).to(dev).long()] = hd
    c, a = heap.cls["Cell"], heap.cls["Alive"]
    smmo.smmo_set_launch(heap.h, smmo.smmo_method_id(method), c, 0, 0, group)
    heap.do("Cell", method, args_of(c, a, cells.data_ptr()))
    g = heap.gather("Cell", ["cell_id", "count"], capacity=n)
    out = np.full(n, -1, np.int32)
    out[g["cell_id"].cpu().numpy()] = g["count"].cpu().numpy()
    heap.sync()
    heap.close()
    return out


@pytest.mark.parametrize("order", ["created", "shuffled", "pairs"])
@pytest.mark.parametrize("W,H", BOARDS)
def test_counts(dev, W, H, order):
    n = W * H
    rng = np.random.default_rng(n)
    ids = np.arange(n, dtype=np.int32)
    if order == "shuffled":
        rng.shuffle(ids)
    elif order == "pairs":                  # every other stretch of 64 in reverse
        ids = np.concatenate([p if i % 2 else p[::-1] for i, p in enumerate(np.split(ids, range(64, n, 64)))])
        ids = np.ascontiguousarray(ids)
    live = rng.integers(0, 2, n).astype(np.uint8)
    want = neighbours(live.reshape(H, W).astype(np.int32)).ravel()
    dying = np.where(live == 1, 1, rng.integers(0, 2, n) * 7).astype(np.uint8)      # only 1 counts
    for group in (1, 2, 4):
        got = counts(dev, GOL_CLASSES, W, H, live, ids,
                     lambda c, a, p: smmo.smmo_gol_args(c, a, p, W, H), "gol.cell_count", group)
        assert np.array_equal(got, want), group
        got = counts(dev, GENERATION_CLASSES, W, H, dying, ids,
                     lambda c, a, p: smmo.smmo_generation_args(c, a, W, H, 0, 0, 9, 0, p), "generation.cell_count",
                     group)
        assert np.array_equal(got, want), group


def test_a_cell_outside_the_heap_is_reported(dev):
    import torch

    W, H = 128, 4
    n = W * H
    heap = smmo.Heap(GOL_CLASSES, blocks=64)
    hd = heap.new("Cell", n, cell_id=torch.arange(n, dtype=torch.int32, device=dev)).clone()
    hd[200] = 64 << 6
    heap.do("Cell", "gol.cell_count", smmo.smmo_gol_args(heap.cls["Cell"], heap.cls["Alive"], hd.data_ptr(), W, H))
    with pytest.raises(smmo.SmmoError) as e:
        heap.sync()
    assert e.value.status == smmo.SMMO_EDEVICE
    smmo.smmo_clear_error(heap.h)
    heap.close()
