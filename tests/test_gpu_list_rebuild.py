"""xg_bin_sort repeated on one preprocess where a view has more tiles than the
counting path takes (pairs emitted and radix sorted by tile), for every form of
the item sort: each build gives the oracle's lists.  (A 1100 x 1100 view at 8 x 8
tiles with a few thousand Gaussians is counted in bands; the sizes here and the
last ones of test_gpu_bands.py take the pair sort.)  The Gaussians are ordered
farthest first, so that the depth range of the first 256 items decides."""
import math

import numpy as np
import pytest

import oracle as O
import scenes as S
from _gpu import note, oracle_cams

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,sizes,tile", [
    (2500, [(2200, 2100)], 8),            # 72 325 tiles; a view sorted by one workgroup, 4 items a thread
    (7000, [(8200, 24)], 8),              # 1025 tiles a row; 8 items a thread
    (9000, [(8200, 24)], 8),              # radix passes of the items
    (300_000, [(1200, 1100)] * 2, 8),     # too many ranking workgroups
])
def test_repeated_builds_of_the_pair_sort(n, sizes, tile):
    import torch
    import paper_2403_04116_amd as P
    from paper_2403_04116_amd import _lib as X
    angles = [0.3 + 0.8 * k for k in range(len(sizes))]
    g = S.gaussians(n, math.log(0.4 * n ** (-1 / 3)), 0.4, 91)
    st = O.Settings(tile=tile)
    cams = oracle_cams(angles, sizes)
    order = np.argsort(-O.project(g, cams[0], st)["depth_bits"].astype(np.int64), kind="stable")
    g = {k: np.ascontiguousarray(v[order]) for k, v in g.items()}
    pr = O.pairs(g, cams, st)
    frame = P.Frame(n, P.cameras(angles, sizes, S.L_SO, S.L_SD, S.DETECTOR_SIDE), P.settings(tile=tile),
                    pair_capacity=pr["keys"].size + 1)
    gt = {k: torch.from_numpy(v).cuda() for k, v in g.items()}
    note(f"rebuild {n} {sizes}")
    frame.preprocess_sort(gt)
    for again in range(3):
        keys, vals, ranges = (t.cpu().numpy() for t in frame.sorted_pairs())
        assert frame.status() == 0
        np.testing.assert_array_equal(keys.view(np.uint64), pr["keys"], err_msg=f"build {again}")
        np.testing.assert_array_equal(vals.view(np.uint32), pr["values"], err_msg=f"build {again}")
        np.testing.assert_array_equal(ranges.view(np.uint32).reshape(-1), np.asarray(pr["ranges"]).reshape(-1))
        X.xg_bin_sort(frame.frame, int(torch.cuda.current_stream().cuda_stream))
