"""The one-workgroup item sort of small views and the list counting in its
launch, at the edges of their ranges: keys, values, ranges and offsets
against the oracle."""
import math

import numpy as np
import pytest

import scenes as S
from test_gpu_binning import _check

pytestmark = pytest.mark.gpu


def _scene(n, seed):
    return S.gaussians(n, math.log(0.4 * n ** (-1 / 3)), 0.3, seed)


@pytest.mark.parametrize("n,sizes,tile", [
    (63, [(40, 24)] * 3, 16),
    (4096, [(64, 64)] * 2, 16),           # 4 items a thread, full
    (4097, [(64, 64)], 16),               # 8 items a thread, lists counted separately
    (8192, [(128, 120)], 16),             # the largest view
    (8193, [(128, 120)], 16),             # one more: the radix passes
    (4000, [(64, 48)] * 17, 16),          # 68 000 items: sorted per view, counted separately
    (2000, [(505, 512), (30, 20)], 8),    # 8 partitions of the counts of 4096 tiles
    (4096, [(505, 512)], 8),              # larger partitions, so that the counts fit
    (4096, [(1023, 1)], 8),               # an odd number of tiles in one row
])
def test_edges(n, sizes, tile):
    _check(_scene(n, 700 + n % 89), [0.2 + 0.8 * k for k in range(len(sizes))], sizes, tile, f"{n} items, {sizes}")


@pytest.mark.parametrize("n", [700, 6000])
def test_equal_depths_keep_the_index_order(n):
    g = _scene(n, 801)
    # azimuth 0: the depth depends on x alone; four depths, one of them of half the items
    g["means"][:, 0] = np.random.default_rng(8).choice(np.array([0.25, 0.25, -0.5, 0.125, 0.75], np.float32), n)
    _check(g, [0.0], [(96, 64)], 16, f"{n} items on four planes")


def test_one_depth_and_no_item_kept():
    g = _scene(300, 802)
    g["means"][:, 0] = 0.5
    _check(g, [0.0], [(64, 64)], 16, "one depth")
    import torch
    import paper_2403_04116_amd as P
    g["opacity"][:] = 1e-6    # all culled
    cams = P.cameras([0.0], [(64, 64)], S.L_SO, S.L_SD, S.DETECTOR_SIDE)
    frame = P.Frame(300, cams, P.settings())
    gt = {k: torch.from_numpy(v).cuda() for k, v in g.items()}
    image, final_t, n_contrib = frame.forward(gt)
    torch.cuda.synchronize()
    assert frame.status() == 0 and frame.n_pairs() == 0
    assert not image.any() and bool((final_t == 1).all()) and not n_contrib.any()
