"""The counting path's slots, each lane finding its item by the beginnings
marked in the window: items of one pair, of whole rows and of a band's every
tile, views of one column and of one row of tiles, items without pairs between
them, and partitions and windows that end inside an item; keys, values, ranges
and offsets against the oracle."""
import math

import numpy as np
import pytest

import scenes as S
from test_gpu_binning import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 64, 257, 1025, 2600])
@pytest.mark.parametrize("sizes", [[(256, 256)], [(8, 2000), (2000, 8)], [(264, 256), (40, 33), (256, 248)]],
                         ids=["1024 tiles", "one column, one row", "bands"])
def test_slots(n, sizes):
    rng = np.random.default_rng(400 + n)
    g = S.gaussians(n, math.log(0.02), 0.3, 410 + n)
    g["scales"] *= np.where(rng.random(n) < 0.15, 60.0, rng.choice([0.2, 1.0, 8.0], n)).astype(np.float32)[:, None]
    off = rng.random(n) < 0.3
    off[0] = False
    g["means"][off] *= 9.0   # many off the detector
    _check(g, [0.4 + 1.1 * k for k in range(len(sizes))], sizes, 8, f"slots: {n} items, {sizes}")
