"""A list build leaves its workspace ready for another: xg_bin_sort repeated
on one preprocess, and a workspace that rendered other scenes before, give
the lists of a fresh workspace, on every item-sort path."""
import math

import pytest

import scenes as S
from _gpu import note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,sizes,tile", [
    (900, [(64, 48)] * 2, 16),            # one workgroup a view, lists counted with it
    (6000, [(64, 48)], 16),               # one workgroup a view
    (9000, [(200, 120), (64, 64)], 16),   # radix passes, depth range folded by the histogram launch
    (9000, [(1100, 1100)], 8),            # radix passes of items and pairs
    (700_000, [(48, 48)] * 3, 16),        # radix passes with their clearing launch
])
def test_repeated_builds(n, sizes, tile):
    import torch
    import paper_2403_04116_amd as P
    from paper_2403_04116_amd import _lib as X
    cams = P.cameras([0.3 + 0.8 * k for k in range(len(sizes))], sizes, S.L_SO, S.L_SD, S.DETECTOR_SIDE)
    scene = [{k: torch.from_numpy(v).cuda() for k, v in S.gaussians(n, math.log(0.4 * n ** (-1 / 3)), 0.3, s).items()}
             for s in (41, 42)]
    scene[1]["means"] *= 0.5      # another depth range
    frame = P.Frame(n, cams, P.settings(tile=tile))
    note(f"repeat {n} {sizes}")
    fresh = []
    for g in scene:
        f = P.Frame(n, cams, P.settings(tile=tile))
        f.fit_capacity(g)
        fresh.append([t.clone() for t in f.sorted_pairs()])
        frame.set_capacity(max(frame.capacity, f.capacity))
    for k in (0, 1, 0):
        frame.preprocess_sort(scene[k])
        for again in range(3):
            got = frame.sorted_pairs()
            assert frame.status() == 0
            for a, b in zip(got, fresh[k]):
                assert torch.equal(a, b), (k, again)
            s = int(torch.cuda.current_stream().cuda_stream)
            if tile == 16:        # (the pair sort's path folds its scan's words: once a preprocess)
                X.xg_bin_sort(frame.frame, s)
