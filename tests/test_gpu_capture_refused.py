"""A render refused because its stream is being captured leaves the frame as it
was: the backward of an earlier forward still runs, under autograd and called
directly, and gives the gradients it gives without the refusal."""
import math

import pytest

import scenes as S
from _gpu import KEYS, note

pytestmark = pytest.mark.gpu


def _frame():
    import torch
    import paper_2403_04116_amd as P
    g = {k: torch.from_numpy(v).cuda() for k, v in S.gaussians(400, math.log(0.1), 0.3, 79).items()}
    cams = P.cameras([0.4], [(40, 24)], S.L_SO, S.L_SD, S.DETECTOR_SIDE)
    return g, P.Frame(400, cams, P.settings(), device="cuda")


def _refused(call):
    import torch
    torch.cuda.synchronize()
    with pytest.raises(RuntimeError):
        with torch.cuda.graph(torch.cuda.CUDAGraph()):
            call()
    torch.cuda.synchronize()


def _close(a, b):
    # the same sums, their atomics in another order
    assert (a - b).norm().item() <= 1e-5 * b.norm().item()


def test_autograd_backward_after_a_refusal():
    import torch
    import paper_2403_04116_amd as P
    note("refused render between forward and backward")
    g, frame = _frame()
    grads = []
    for refuse in (False, True):
        leaves = {k: g[k].clone().requires_grad_() for k in KEYS}
        image = P.render(leaves, frame)
        if refuse:
            _refused(lambda: P.render(g, frame))
        (image ** 2).sum().backward()
        grads.append([leaves[k].grad for k in KEYS])
    for a, b in zip(*grads):
        _close(b, a)


@pytest.mark.parametrize("what", ["render", "fit_capacity"])
def test_repeated_backward_after_a_refusal(what):
    import paper_2403_04116_amd as P
    note(f"refused {what} between two backwards")
    g, frame = _frame()
    frame.fit_capacity(g)
    image, final_t, n_contrib = frame.render_fwd(g)
    first = frame.backward(g, image, final_t, n_contrib)
    _refused(lambda: P.render(g, frame) if what == "render" else frame.fit_capacity(g))
    second = frame.backward(g, image, final_t, n_contrib)
    for k in KEYS:
        _close(second[k], first[k])
