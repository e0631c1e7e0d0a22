"""The stand-alone inverse transform leaves its input as it is and takes every layout a
complex64 tensor can have; transforms of several fields equal those of one."""
import pytest
import torch

from paper_1805_02247_amd import api
from _gpu import DEV, rel_l2, require_gpu, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,B", [(16, 3), (32, 1), (64, 2), (128, 1), (128, 3), (256, 1), (512, 1)])
def test_inverse_keeps_its_input(n, B):
    require_gpu()
    say(f"fft inputs n={n} B={B}")
    g = torch.Generator(device=DEV)
    g.manual_seed(n + B)
    x = torch.randn(B, n, n, n, generator=g, device=DEV)
    h = n // 2 + 1
    X = torch.fft.rfftn(x.double(), dim=(1, 2, 3)).to(torch.complex64)
    kept = X.clone()
    y = api.fft_c2r(X)
    assert torch.equal(torch.view_as_real(X), torch.view_as_real(kept))
    assert rel_l2(y.cpu().numpy(), x.cpu().numpy()) < 2e-6
    # one complex value off the allocation's alignment, strided, and a lazy conjugate
    flat = torch.empty(X.numel() + 1, dtype=torch.complex64, device=DEV)
    flat[1:] = X.reshape(-1)
    assert torch.equal(api.fft_c2r(flat[1:].reshape(B, n, n, h)), y)
    wide = torch.zeros(B, n, n, h + 3, dtype=torch.complex64, device=DEV)
    wide[..., :h] = X
    assert torch.equal(api.fft_c2r(wide[..., :h]), y)
    assert torch.equal(api.fft_c2r(X.conj().resolve_conj().conj()), y)
    # each field alone, both directions
    S = api.fft_r2c(x)
    for b in range(B):
        assert torch.equal(api.fft_c2r(X[b:b + 1])[0], y[b])
        one = api.fft_r2c(x[b:b + 1])[0]
        assert torch.equal(torch.view_as_real(one), torch.view_as_real(S[b]))


def test_bad_sizes_are_refused_as_before():
    require_gpu()
    for shape in ((0, 16, 16, 9), (1, 12, 12, 7)):
        with pytest.raises(api.L.PmrError):
            api.fft_c2r(torch.zeros(*shape, dtype=torch.complex64, device=DEV))


@pytest.mark.parametrize("n,B", [(32, 1), (32, 3), (64, 1), (64, 2), (128, 2)])
def test_plane_force_equals_the_separate_passes(n, B):
    """kz windows switch the plane-by-plane force off: bitwise the same gradient."""
    require_gpu()
    say(f"plane force n={n} B={B}")
    import numpy as np

    import synth
    from paper_1805_02247_amd import cosmo
    box = 2.0 * n
    power = cosmo.linear_power(0.8, 0.2)
    s = np.stack([cosmo.modes_from_white_noise(synth.white_noise(n + b, n), box, power).reshape(-1)
                  for b in range(B)])
    pm = api.PMContext(api.Config(batch=B, n_part=n, n_mesh=n, n_out=n, n_steps=3, box=box,
                                  loss_kind=api.L.PMR_LOSS_DENSITY_L2), DEV)
    pm.set_prior(torch.from_numpy(cosmo.prior_inv_variance(n, box, power)))
    pm.set_target(torch.zeros(B, n ** 3, device=DEV))
    pm.set_loss(api.LossParams())
    out = []
    saved = api.fft_get_slab(n)
    try:
        for slab in (0, 16):
            api.fft_set_slab(n, slab)
            mass, _ = pm.forward(torch.from_numpy(s).to(DEV))
            out.append((pm.debug("force", 2), mass,
                        torch.view_as_real(pm.adjoint(torch.ones(B, dtype=torch.float64,
                                                                 device=DEV)))))
    finally:
        api.fft_set_slab(n, saved)
    for a, b in zip(*out):
        assert torch.equal(a, b)
