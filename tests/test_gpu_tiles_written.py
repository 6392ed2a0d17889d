"""Every pixel of every view is written by one forward launch, whatever order
the tiles are dealt in: contiguous blocks, chunks with left-over pieces, frames
of millions of pairs and frames of many tiles."""
import math

import pytest

import scenes as S
from _gpu import note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,sizes,tile", [
    (6000, [(512, 512)], 16),                                     # edge rows light, centre rows heavy
    (6000, [(9, 9)], 8),                                          # fewer tiles than XCDs
    (200_000, [(512, 512)] * 8, 16),                              # contiguous, a view per XCD
    (200_000, [(1000, 700)], 8),                                  # one view, left-over piece
    (100_000, [(128, 128)] * 9 + [(512, 500)] * 5, 16),           # heaviest first
    (100_000, [(512, 500)] * 5 + [(128, 128)] * 9, 16),           # heaviest last
    (300, [(512, 512)] * 90, 16),                                 # 92 160 tiles of few entries
    (3000, [(1600, 1400)] * 5 + [(40, 40)] * 60, 8),              # 176 500 tiles
])
def test_every_pixel_is_written(n, sizes, tile):
    import torch
    import paper_2403_04116_amd as P
    note(f"written {n} {len(sizes)} views tile {tile}")
    g = {k: torch.from_numpy(v).cuda() for k, v in S.gaussians(n, math.log(0.5 * n ** (-1 / 3)), 0.4, 93).items()}
    cams = P.cameras([0.05 * k for k in range(len(sizes))], sizes, S.L_SO, S.L_SD, S.DETECTOR_SIDE)
    frame = P.Frame(n, cams, P.settings(tile=tile))
    frame.fit_capacity(g)
    out = [torch.full((frame.total_pixels,), float("nan"), device="cuda") for _ in range(2)]
    out.append(torch.full((frame.total_pixels,), -7, dtype=torch.int32, device="cuda"))
    frame.render_fwd(g, out)
    assert torch.isfinite(out[0]).all() and torch.isfinite(out[1]).all()
    assert (out[2] >= 0).all() and (out[2] > 0).any()
