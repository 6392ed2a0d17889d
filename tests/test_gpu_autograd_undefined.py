"""A gradient that a later node leaves undefined reaches the renderer's
backward as none, and gives zero gradients; a render that would wait for the
status word is refused while its stream is being captured."""
import math

import pytest

import scenes as S
from _gpu import KEYS, note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("both", [False, True])
def test_undefined_image_gradient(both):
    import torch
    import paper_2403_04116_amd as P

    class Cut(torch.autograd.Function):
        @staticmethod
        def forward(ctx, x):
            return x.clone()

        @staticmethod
        def backward(ctx, grad):
            return None

    note(f"undefined gradient, beside a defined one: {both}")
    g = S.gaussians(300, math.log(0.1), 0.3, 77)
    cams = P.cameras([0.4], [(40, 24)], S.L_SO, S.L_SD, S.DETECTOR_SIDE)
    frame = P.Frame(300, cams, P.settings(), device="cuda")
    leaves = {k: torch.from_numpy(g[k]).cuda().requires_grad_() for k in KEYS}
    image = P.render(leaves, frame)
    loss = Cut.apply(image).sum()
    if both:
        loss = loss + image.sum()
    loss.backward()
    torch.cuda.synchronize()
    assert leaves["intensity"].grad.abs().sum().item() > 0 if both else \
        all(leaves[k].grad.abs().sum().item() == 0 for k in KEYS)


def test_render_is_refused_under_capture():
    import torch
    import paper_2403_04116_amd as P
    note("render under capture")
    g = S.gaussians(300, math.log(0.1), 0.3, 78)
    cams = P.cameras([0.4], [(40, 24)], S.L_SO, S.L_SD, S.DETECTOR_SIDE)
    frame = P.Frame(300, cams, P.settings(), device="cuda")
    t = {k: torch.from_numpy(g[k]).cuda() for k in KEYS}
    image = P.render(t, frame)
    torch.cuda.synchronize()
    with pytest.raises(RuntimeError):
        with torch.cuda.graph(torch.cuda.CUDAGraph()):
            P.render(t, frame)
    torch.cuda.synchronize()
    assert torch.equal(P.render(t, frame), image)
