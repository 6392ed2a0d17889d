"""Tile lists by counting where a view has more tiles than one workgroup's
counters, in bands of tile rows, and the views beyond that path (emission and
the radix sort of the pairs): keys, values, ranges and offsets against the
oracle."""
import math

import pytest

import scenes as S
from test_gpu_binning import _check

pytestmark = pytest.mark.gpu


def _scene(n, seed, s0=0.4):
    return S.gaussians(n, math.log(s0 * n ** (-1 / 3)), 0.4, seed)


@pytest.mark.parametrize("n,sizes,tile", [
    (9000, [(264, 256)], 8),                  # 33 tiles a row: bands of 31 rows, the last of one
    (30_000, [(512, 512), (100, 90)], 8),     # 4 bands beside a view of one
    (5000, [(520, 1000)], 8),                 # 8125 tiles, counted by the sort's launch
    (9000, [(1100, 700), (2000, 33)], 8),     # bands of 7 and of 4 rows
    (200_000, [(1024, 1024), (1030, 600)], 16),   # partitions of 2048 items
    (9000, [(8192, 40), (30, 500)], 8),       # 1024 tiles a row: a band per row
    (9000, [(8200, 24)], 8),                  # 1025 tiles a row: the radix path
    (2000, [(2200, 2100)], 8),                # 72 325 tiles: the radix path
    (300_000, [(1200, 1100)] * 2, 8),         # more ranking workgroups than the rule allows: the radix path
    (2000, [(2000, 2000)], 8),                # 62 500 tiles in 63 bands
])
def test_bands(n, sizes, tile):
    _check(_scene(n, 310 + n % 83), [0.3 + 0.8 * k for k in range(len(sizes))], sizes, tile, f"{n} items, {sizes}")


def test_rectangles_over_many_bands():
    g = _scene(3000, 321)
    g["scales"][:60] *= 12.0     # rectangles over every band, wider than a packed one
    _check(g, [0.4, 2.0], [(640, 600), (64, 600)], 8, "large footprints")
