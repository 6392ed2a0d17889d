"""Walk lists filled up with the empty entry to groups of four: lists of every
length around a group and a batch, for each tile size, with alpha_min = 0
(where an entry of alpha 0 would count as a contributor) and with the default
settings, forward, backward, stored transmittances and work counts against the
oracle at the parity tolerance."""
import math

import numpy as np
import pytest

import oracle as O
import scenes as S
from _gpu import check_counts, compare_forward, compare_grads, gpu_run, grad_upstream, note, oracle_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("n", [1, 3, 4, 5, 63, 64, 65])
@pytest.mark.parametrize("kw", [{"alpha_min": 0.0, "t_min": 0.0}, {}], ids=["all", "default"])
def test_list_lengths(tile, n, kw):
    g = S.gaussians(n, math.log(0.3), 0.3, 700 + n)
    g["means"] *= 0.3
    g["opacity"] = np.minimum(g["opacity"], 0.6).astype(np.float32)
    angles, sizes = [0.4, 3.0], [(19, 9), (40, 33)]
    label = f"list pad: tile {tile}, {n} entries, {kw}"
    ref = oracle_run(g, angles, sizes, tile=tile, **kw)
    up = np.random.default_rng(9).normal(size=sum(w * h for w, h in sizes)).astype(np.float32)
    up = grad_upstream(up, ref)
    note(label)
    gpu = gpu_run(g, angles, sizes, tile=tile, lds=64, upstream=up, **kw)
    m = compare_forward(gpu, ref, label=label)
    rg = O.backward(g, ref["cams"], ref["st"], up, binned=(ref["pairs"]["values"], ref["pairs"]["ranges"]),
                    flip=m.flip)
    compare_grads(gpu["grads"], rg)
    check_counts(gpu["frame"].render_counts().cpu().numpy(), ref, g, m, label=label)
