"""Tile lists by counting at every partition size its rule picks (256 to 2048
items, with one or more items per thread of the ranking kernel), at both
table sizes (up to 1024 and up to 4096 tiles per view): keys, values, ranges
and offsets against the oracle."""
import math

import pytest

import scenes as S
from test_gpu_binning import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,sizes,tile", [
    (1, [(64, 48)], 16),                        # one item
    (257, [(64, 48), (20, 90)], 16),            # a partition and one item more
    (8193, [(256, 256)], 16),                   # 33 partitions of 256 items
    (70_000, [(96, 96)] * 3, 16),               # 512 items
    (150_000, [(96, 96)] * 3, 16),              # 1024 items
    (550_000, [(96, 96), (40, 64)], 16),        # 2048 items
    (60_001, [(512, 500)], 8),                  # more than 1024 tiles: 256 items
    (150_000, [(512, 500)] * 2, 8),             # 1024 items
    (530_000, [(512, 512), (64, 64)], 8),       # 2048 items, 4096 tiles
])
def test_partition_sizes(n, sizes, tile):
    g = S.gaussians(n, math.log(0.3 * n ** (-1 / 3)), 0.3, 600 + n % 97)
    _check(g, [0.3 + 0.7 * k for k in range(len(sizes))], sizes, tile, f"{n} items a view, {sizes}, tile {tile}")
