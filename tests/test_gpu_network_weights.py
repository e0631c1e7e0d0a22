"""New single-network weights between a forward and its adjoint: the adjoint's network derivative
is that of the new weights at the forward's fields. With a mass cotangent alone the gradient
passes through nothing else that depends on the weights, so it equals, bit for bit, the one
of a forward with the new weights."""
import gc

import numpy as np
import pytest
import torch

import synth
from paper_1805_02247_amd import _lib as L
from paper_1805_02247_amd import api, cosmo
from _gpu import DEV, require_gpu, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,mixed", [(8, False), (16, False), (32, False), (64, False), (32, True), (64, True)])
def test_adjoint_after_new_weights(H, mixed):
    require_gpu()
    say(f"network weights H={H} mixed={mixed}")
    n, box, B = 16, 60.0, 2
    power = cosmo.linear_power(0.8, 0.2)
    pm = api.PMContext(api.Config(batch=B, n_part=n, n_mesh=n, n_out=n, n_steps=2, mlp_hidden=H,
                                  box=box, precision=L.PMR_MIXED if mixed else L.PMR_FP32), DEV)
    pm.set_prior(torch.from_numpy(cosmo.prior_inv_variance(n, box, power)))
    old, new = ({k: torch.from_numpy(v) for k, v in synth.mlp_weights(seed, H).items()}
                for seed in (1, 2))
    pm.set_mlp(old)
    pm.set_target(torch.ones(B, n ** 3, device=DEV))
    pm.set_loss(api.LossParams())
    s = torch.from_numpy(np.stack([cosmo.modes_from_white_noise(synth.white_noise(b, n), box, power)
                                   .reshape(-1) for b in range(B)])).to(DEV)
    mbar = torch.randn(B, n ** 3, device=DEV, generator=torch.Generator(device=DEV).manual_seed(H))
    zero = torch.zeros(B, dtype=torch.float64, device=DEV)

    def after(w):
        pm.set_mlp(w)
        pm.forward(s)
        return torch.view_as_real(pm.adjoint(zero, mbar)).clone()

    ref = {"old": after(old), "new": after(new)}
    assert not torch.equal(ref["old"], ref["new"])
    pm.set_mlp(old)
    pm.forward(s)
    pm.set_mlp(new)
    assert torch.equal(torch.view_as_real(pm.adjoint(zero, mbar)), ref["new"])
    assert torch.equal(torch.view_as_real(pm.adjoint(zero, mbar)), ref["new"])
    gc.collect()  # nothing of earlier tests goes away during the capture
    # a captured adjoint: the weights of the moment of each replay
    grad = torch.empty(B, pm.n_modes, dtype=torch.complex64, device=DEV)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        pm.adjoint(zero, mbar, out=grad)
    for name, w in (("new", new), ("old", old), ("new", new), ("old", old)):
        pm.set_mlp(w)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(torch.view_as_real(grad), ref[name])
