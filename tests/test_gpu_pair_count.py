"""The pair count of a frame with more pairs than an int32 holds reads the
largest int32 (status XG_ECAPACITY, empty lists), whichever launch counts."""
import math

import pytest

import scenes as S
from _gpu import note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2048, 2049])   # counted in the item sort's launch; by the lists' own
def test_pair_count_above_int32(n):
    import torch
    import paper_2403_04116_amd as P
    note(f"pair count, {n} items a view")
    views = 32
    # alpha_min 0: every rectangle is the whole view, 36 864 tiles
    cams = P.cameras([0.1 * k for k in range(views)], [(1536, 1536)] * views, S.L_SO, S.L_SD, S.DETECTOR_SIDE)
    frame = P.Frame(n, cams, P.settings(tile=8, alpha_min=0.0))
    g = {k: torch.from_numpy(v).cuda() for k, v in S.gaussians(n, math.log(0.05), 0.3, 92).items()}
    frame.preprocess_sort(g)
    torch.cuda.synchronize()
    assert n * views * 36864 > 0x7fffffff
    assert frame.status() == P._lib.XG_ECAPACITY
    assert frame.n_pairs() == 0x7fffffff
    assert not frame.ws_tensor(frame.layout.ranges, torch.int32, 2 * frame.total_tiles).any().item()
