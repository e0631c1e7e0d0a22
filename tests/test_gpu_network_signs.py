"""The single network's adjoint from the forward's stored outputs and ReLU signs: every hidden
width and precision against FP64 autograd, on a mesh whose gradient passes through the
network alone (mass cotangent only), and twice from one forward."""
import numpy as np
import pytest
import torch

import synth
from paper_1805_02247_amd import _lib as L
from paper_1805_02247_amd import api, cosmo
from _gpu import DEV, rel_l2, require_gpu, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,mixed", [(8, False), (16, False), (32, False), (64, False), (32, True), (64, True)])
@pytest.mark.parametrize("B", [1, 3])
def test_density_adjoint_through_the_network(H, mixed, B):
    require_gpu()
    say(f"network signs H={H} mixed={mixed} B={B}")
    n, box = 16, 60.0
    power = cosmo.linear_power(0.8, 0.2)
    pm = api.PMContext(api.Config(batch=B, n_part=n, n_mesh=n, n_out=n, n_steps=2, mlp_hidden=H,
                                  box=box, precision=L.PMR_MIXED if mixed else L.PMR_FP32), DEV)
    pm.set_prior(torch.from_numpy(cosmo.prior_inv_variance(n, box, power)))
    w = synth.mlp_weights(H, H)
    pm.set_mlp({k: torch.from_numpy(v) for k, v in w.items()})
    pm.set_target(torch.ones(B, n ** 3, device=DEV))
    pm.set_loss(api.LossParams())
    s = np.stack([cosmo.modes_from_white_noise(synth.white_noise(H + b, n), box, power).reshape(-1)
                  for b in range(B)])
    mass, _ = pm.forward(torch.from_numpy(s).to(DEV))
    g = torch.Generator(device=DEV)
    g.manual_seed(H)
    mbar = torch.randn(B, n ** 3, generator=g, device=DEV)
    zero = torch.zeros(B, dtype=torch.float64, device=DEV)
    first = pm.adjoint(zero, mbar)
    got = pm.debug("dbar_f").double()
    assert torch.equal(torch.view_as_real(first), torch.view_as_real(pm.adjoint(zero, mbar)))
    # FP64 autograd from the library's own final density
    d = pm.debug("delta_f").double().reshape(B, n, n, n).requires_grad_()
    k = 2 * np.pi / box * torch.fft.fftfreq(n, 1.0 / n, dtype=torch.float64, device=DEV)
    kz = 2 * np.pi / box * torch.arange(n // 2 + 1, dtype=torch.float64, device=DEV)
    k2 = k[:, None, None] ** 2 + k[None, :, None] ** 2 + kz ** 2
    f = [torch.fft.irfftn(torch.fft.rfftn(d, dim=(1, 2, 3)) * torch.exp(-0.5 * k2 * R * R),
                          s=(n, n, n), dim=(1, 2, 3)) for R in (1.0, 2.0)]
    v = torch.stack([d, f[0], f[0] - f[1]]).reshape(3, -1)
    t = {q: torch.from_numpy(x).to(DEV).double() for q, x in w.items()}
    h = torch.relu(t["W1"] @ v + t["b1"][:, None])
    h = torch.relu(t["W2"] @ h + t["b2"][:, None])
    m = torch.nn.functional.softplus((t["W3"] @ h + t["b3"][:, None])[0])
    m = m.reshape(B, -1)
    tol = 2e-2 if mixed else 1e-5  # BF16 products (2^-8 each); FP32 sums of up to 64 terms
    assert rel_l2(mass.cpu().numpy(), m.detach().cpu().numpy()) < tol
    ref, = torch.autograd.grad((m * mbar.double()).sum(), d)
    # a unit whose input is within rounding of zero may take its other side: rare in FP32,
    # one in some hundred with BF16 products
    assert rel_l2(got.cpu().numpy(), ref.reshape(B, -1).cpu().numpy()) < (1e-1 if mixed else 1e-3)
