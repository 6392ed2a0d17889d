"""The blend without rectangle test and alpha clamp, taken by 8 x 8 and 16 x 16
tiles for records marked as needing neither, against 32 x 32 tiles, which
always test: images and transmittances bit for bit, and the gradients that are
plain sums of the backward's terms (opacity, intensity) up to the order of
those sums; the others pass through the inverse covariance, which for
footprints this thin multiplies that difference by its condition number.  Opacities around every limit of the rule, footprints from far
below a pixel to the whole detector, and the settings it depends on."""
import math

import numpy as np
import pytest

import scenes as S
from _gpu import note

pytestmark = pytest.mark.gpu


def _scene(n, seed, amin):
    rng = np.random.default_rng(seed)
    g = S.gaussians(n, math.log(0.05), 0.3, seed)
    g["scales"] = np.exp(rng.uniform(math.log(1e-4), math.log(0.6), (n, 3))).astype(np.float32)
    edge = np.array([1.0, 0.99, 0.9801, 0.98, 0.9799, 0.96, 0.4951, 0.495, 0.49, max(amin, 1e-3) * 1.001], np.float32)
    pick = rng.random(n) < 0.5
    g["opacity"] = np.where(pick, rng.choice(edge, n), g["opacity"]).astype(np.float32)
    g["means"] *= 1.3     # some centres past the detector's edges
    return g


@pytest.mark.parametrize("lowpass,amin,amax,tmin", [
    (0.3, 1 / 255, 0.99, 1e-4), (0.0, 1 / 255, 0.99, 1e-4), (0.3, 0.1, 0.99, 1e-4), (0.3, 1 / 255, 0.5, 1e-4),
    (0.3, 0.0, 0.99, 1e-4), (0.3, 1 / 255, 0.99, 0.0)])
def test_equals_tested_blend(lowpass, amin, amax, tmin):
    import torch
    import paper_2403_04116_amd as P
    n, sizes = 900, [(129, 97), (64, 64), (500, 40)]
    angles = [0.2, 1.7, 4.0]
    cams = P.cameras(angles, sizes, S.L_SO, S.L_SD, S.DETECTOR_SIDE)
    g = {k: torch.from_numpy(v).cuda() for k, v in _scene(n, 71, amin).items()}
    out = {}
    for tile in (32, 16, 8):
        note(f"plain blend: tile {tile}, lowpass {lowpass}, alpha_min {amin}, alpha_max {amax}, t_min {tmin}")
        frame = P.Frame(n, cams, P.settings(tile=tile, lowpass=lowpass, alpha_min=amin, alpha_max=amax, t_min=tmin))
        frame.fit_capacity(g)
        image, final_t, n_contrib = frame.render_fwd(g)
        up = torch.from_numpy(np.random.default_rng(3).normal(size=image.numel()).astype(np.float32)).cuda()
        grads = frame.backward(g, up, final_t, n_contrib)
        torch.cuda.synchronize()
        out[tile] = image, final_t, grads
    for tile in (16, 8):
        assert torch.equal(out[tile][0], out[32][0]) and torch.equal(out[tile][1], out[32][1])
        for k in ("opacity", "intensity"):
            a, b = out[tile][2][k].double(), out[32][2][k].double()
            # float32 sums of the same terms in another order
            assert ((a - b).norm() <= 1e-5 * b.norm()).item(), k
