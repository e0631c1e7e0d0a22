"""The paints give bitwise the same rows however many wavefronts share a chunking group: the
share depends on the launch's total rows, so the same item is painted alone and in batches."""
import numpy as np
import pytest
import torch

import synth
from oracle import mesh as M
from paper_1805_02247_amd import _lib as L
from paper_1805_02247_amd import api, cosmo
from _gpu import DEV, rel_l2, require_gpu, say

pytestmark = pytest.mark.gpu


def _positions(seed, npart, box):
    """Half uniform, half in blobs of which one straddles the wrapped row (y = 0)."""
    P = npart ** 3
    r = np.random.default_rng(seed)
    x = r.uniform(0, box, (3, P))
    c = r.uniform(0, box, (3, 8))
    c[1, 0] = 0.0
    x[:, :P // 2] = (c[:, r.integers(0, 8, P // 2)] + r.normal(0, box / 100, (3, P // 2))) % box
    return x[:, r.permutation(P)]


@pytest.mark.parametrize("npart,nm,batches", [(16, 16, (1, 7)), (32, 32, (1, 5, 64)), (64, 64, (1, 3, 32)),
                                              (32, 64, (1, 16)), (128, 128, (1, 2, 4)),
                                              (64, 256, (1, 2))])
def test_density_is_the_same_alone_and_in_a_batch(npart, nm, batches):
    require_gpu()
    say(f"paint share: np={npart} nm={nm} batches {batches}")
    box, mass = 50.0, (nm / npart) ** 3
    x = _positions(npart + nm, npart, box)
    ref = None
    for B in batches:
        xt = torch.from_numpy(x).to(DEV).expand(B, 3, npart ** 3).contiguous()
        d = api.cic_paint(xt, *api.cic_sort(xt, nm, box), nm, box, mass, 0.0)
        if ref is None:
            ref = d[0].clone()
            assert rel_l2(ref.cpu().numpy().reshape(nm, nm, nm),
                          M.cic_paint(x, nm, box, np.full(npart ** 3, mass))) < 1e-6
        assert all(torch.equal(d[b], ref) for b in range(B))


@pytest.mark.parametrize("npart,nm,big", [(16, 32, 9), (32, 32, 40), (64, 64, 8)])
def test_gradient_is_the_same_alone_and_in_a_batch(npart, nm, big):
    require_gpu()
    say(f"paint share in the gradient: np={npart} nm={nm} batch {big}")
    box = 2.0 * npart
    power = cosmo.linear_power(0.8, 0.2)
    s = cosmo.modes_from_white_noise(synth.white_noise(npart, npart), box, power).reshape(-1)
    out = []
    for B in (1, big):
        pm = api.PMContext(api.Config(batch=B, n_part=npart, n_mesh=nm, n_out=npart, n_steps=4,
                                      box=box, loss_kind=L.PMR_LOSS_DENSITY_L2), DEV)
        pm.set_prior(torch.from_numpy(cosmo.prior_inv_variance(npart, box, power)))
        pm.set_target(torch.zeros(B, npart ** 3, device=DEV))
        pm.set_loss(api.LossParams())
        mass, _ = pm.forward(torch.from_numpy(np.stack([s] * B)).to(DEV))
        out.append((mass, pm.adjoint(torch.ones(B, dtype=torch.float64, device=DEV))))
    for b in range(big):
        assert torch.equal(out[1][0][b], out[0][0][0])
        assert torch.equal(out[1][1][b].view(torch.float32), out[0][1][0].view(torch.float32))
