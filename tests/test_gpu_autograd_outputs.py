"""MatchFunction where only some of its outputs carry a gradient: the same
gradients as the adjoint called with zeros for the rest."""
import pytest
import torch

import parity
import synth
from paper_2412_12392_amd import MatchFunction, match_backward, params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("use", ["p", "xhat", "both"])
def test_gradients_of_some_outputs(use):
    t = parity.pair_tensors(synth.make_pair(37, 53, 61, conf=True))
    Xi, Xj = t["Xii"].requires_grad_(True), t["Xji"].requires_grad_(True)
    p, xhat, idx, valid, theta = MatchFunction.apply(Xi, Xj, t["Dii"], t["Dji"], t["Qii"], t["Qji"], None, params())
    assert not (idx.requires_grad or valid.requires_grad or theta.requires_grad)
    g = torch.Generator(device="cuda").manual_seed(7)
    gp = torch.randn(p.shape, generator=g, device="cuda") if use != "xhat" else None
    gx = torch.randn(xhat.shape, generator=g, device="cuda") if use != "p" else None
    outs = [(o, w) for o, w in ((p, gp), (xhat, gx)) if w is not None]
    got = torch.autograd.grad([o for o, _ in outs], (Xi, Xj), [w for _, w in outs])
    ref = match_backward(Xi.detach(), Xj.detach(), p.detach(), valid, torch.zeros_like(p) if gp is None else gp,
                         torch.zeros_like(xhat) if gx is None else gx)
    # dXji is written by one thread per entry; dXii is summed in the order of its
    # atomics, a few float32 roundings of at most some ten terms apart.
    assert torch.equal(got[1], ref[1])
    assert (got[0] - ref[0]).norm() <= 1e-6 * ref[0].norm()
