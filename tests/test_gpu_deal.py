"""The order in which the blend launches take the tiles, where contiguous
blocks of tiles per XCD would hold very different amounts of work and the
tiles are dealt in chunks: every tile is rendered once, so each view equals,
bit for bit, the same view rendered in a frame of its own."""
import math

import numpy as np
import pytest

import scenes as S
from _gpu import note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes,tile", [
    ([(128, 128)] * 5 + [(512, 480)] * 3, 16),      # the longest lists first, chunks and left-over pieces
    ([(512, 512)], 16),                             # one view: edge rows light, centre rows heavy
    ([(33, 65), (700, 20), (20, 333), (1, 1)], 8),  # odd sizes, fewer tiles than a round of chunks
    ([(9, 9)], 8),                                  # fewer tiles than XCDs
    ([(1600, 1400), (40, 40)], 8),                  # above 2048 groups of 16 tiles
])
def test_every_tile_is_rendered_once(sizes, tile):
    import torch
    import paper_2403_04116_amd as P
    n = 6000
    g = {k: torch.from_numpy(v).cuda() for k, v in S.gaussians(n, math.log(0.04), 0.4, 77).items()}
    cams = P.cameras([0.4 + 0.3 * k for k in range(len(sizes))], sizes, S.L_SO, S.L_SD, S.DETECTOR_SIDE)

    def render(cs):
        frame = P.Frame(n, cs, P.settings(tile=tile))
        frame.fit_capacity(g)
        out = [torch.full((frame.total_pixels,), float("nan"), device="cuda") for _ in range(2)]
        out.append(torch.full((frame.total_pixels,), -7, dtype=torch.int32, device="cuda"))
        frame.render_fwd(g, out)
        torch.cuda.synchronize()
        return [frame.split(t) for t in out]

    note(f"deal {sizes} tile {tile}")
    together = render(cams)
    for v, cam in enumerate(cams):
        alone = render([cam])
        for a, b in zip(together, alone):
            np.testing.assert_array_equal(a[v].cpu().numpy(), b[0].cpu().numpy())
