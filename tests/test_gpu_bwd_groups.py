"""Backward gradient sums at the edges of their grouping (4 list entries a
group, 8 a read of the list, a batch at a time): lists of every short length,
entries without contributors inside a group, and a list one entry longer
than a batch, against the oracle's adjoint at the parity tolerance."""
import math

import numpy as np
import pytest

import oracle as O
import scenes as S
from _gpu import compare_forward, compare_grads, gpu_run, grad_upstream, note, oracle_run

pytestmark = pytest.mark.gpu


def _check(g, sizes, tile, lds, label):
    angles = [0.3 + 0.9 * k for k in range(len(sizes))]
    ref = oracle_run(g, angles, sizes, tile=tile)
    up = np.random.default_rng(5).normal(size=sum(w * h for w, h in sizes)).astype(np.float32)
    up = grad_upstream(up, ref)
    note(f"{label}: GPU")
    gpu = gpu_run(g, angles, sizes, tile=tile, lds=lds, upstream=up)
    m = compare_forward(gpu, ref, label=label)
    rg = O.backward(g, ref["cams"], ref["st"], up, binned=(ref["pairs"]["values"], ref["pairs"]["ranges"]),
                    flip=m.flip)
    compare_grads(gpu["grads"], rg)


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 7, 8, 9, 65])
def test_short_lists(n):
    g = S.gaussians(n, math.log(0.3), 0.3, 900 + n)
    g["means"] *= 0.3
    _check(g, [(8, 8), (11, 5)], 8, 64, f"{n} entries")


def test_entries_without_contributors():
    # opacities around alpha_min: many listed entries reach it at no pixel
    g = S.gaussians(60, math.log(0.25), 0.5, 950)
    g["opacity"] = np.random.default_rng(6).choice(np.array([0.0045, 0.006, 0.5], np.float32), 60)
    _check(g, [(40, 24)], 16, 64, "faint entries")
