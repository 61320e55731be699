"""The step counts that the simulation drivers hand to the library: those of
range(), which the drivers looped over."""

import numpy as np
import pytest

from paper_1908_05845_amd.sims import _count


def test_counts():
    for n in (0, 1, 7, -1, -5, np.int64(3), np.int32(-2), True):
        assert _count(n) == len(range(n))
    for bad in (1.0, 2.5, "3", None):
        with pytest.raises(TypeError):
            _count(bad)
