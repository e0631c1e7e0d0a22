"""The plane-by-plane y and z transforms stand in for strided passes with the same butterflies
only: whatever tiles are set, the force and the gradient have the same bits with kz windows
(which switch the planes off) and without, and one item's do not depend on the batch. And the
strided y pass of every tile shape, where the model runs it up to 128^3, against FP64."""
import numpy as np
import pytest
import torch

import paper_1805_02247_amd as P
import synth
from oracle import model as OM
from paper_1805_02247_amd import api, cosmo
from paper_1805_02247_amd.tune import candidates
from _gpu import DEV, rel_l2, require_gpu, say

pytestmark = pytest.mark.gpu

BOX = 100.0


def _context(n, B, steps):
    power = cosmo.linear_power(0.8, 0.2)
    pm = api.PMContext(api.Config(batch=B, n_part=n, n_mesh=n, n_out=n, n_steps=steps, box=BOX,
                                  loss_kind=api.L.PMR_LOSS_DENSITY_L2), DEV)
    pm.set_prior(torch.from_numpy(cosmo.prior_inv_variance(n, BOX, power)))
    pm.set_target(torch.zeros(B, n ** 3, device=DEV))
    pm.set_loss(api.LossParams())
    s = np.stack([cosmo.modes_from_white_noise(synth.white_noise(n + b, n), BOX, power).reshape(-1)
                  for b in range(B)])
    return pm, torch.from_numpy(s).to(DEV)


def _run(pm, s, B):
    mass, _ = pm.forward(s)
    grad = pm.adjoint(torch.ones(B, dtype=torch.float64, device=DEV))
    return [pm.debug("force", 1).reshape(B, -1), mass.clone(), torch.view_as_real(grad).clone()]


# 16 columns and 256 threads take every staging; the library's own default is staging 0
@pytest.mark.parametrize("n", [16, 32, 64, 128])
@pytest.mark.parametrize("y", [0, 1, 2])
@pytest.mark.parametrize("x", [0, 1, 2])
def test_windows_and_batch_leave_the_bits(n, y, x):
    require_gpu()
    say(f"plane plans n={n} y staging {y} x staging {x}")
    tiles = {P.PMR_FFT_YPASS: y, P.PMR_FFT_XPASS: x, P.PMR_FFT_XPASS_MULTI: x}
    saved = {p: P.fft_get_tile(n, p) for p in tiles}
    slab = P.fft_get_slab(n)
    two, s = _context(n, 2, 2)
    one, _ = _context(n, 1, 2)
    try:
        for p, st in tiles.items():
            P.fft_set_tile(n, p, 16, 256, st)
        P.fft_set_slab(n, 0)
        whole, single = _run(two, s, 2), _run(one, s[:1], 1)
        P.fft_set_slab(n, 16)
        windows = _run(two, s, 2)
    finally:
        P.fft_set_slab(n, slab)
        for p, t in saved.items():
            P.fft_set_tile(n, p, *t)
    for a, b, c in zip(whole, windows, single):
        assert torch.equal(a, b)
        assert torch.equal(a[:1], c)


@pytest.mark.parametrize("n", [64, 128])
def test_strided_y_pass_of_every_tile(n):
    """kz windows keep the planes off, so every y pass of the force is the strided one. The
    oracle's force of the library's own positions; the tolerance is the one of the force meshes
    of the smaller meshes."""
    require_gpu()
    pm, s = _context(n, 1, 1)
    saved, slab = P.fft_get_tile(n, P.PMR_FFT_YPASS), P.fft_get_slab(n)
    ref = None
    try:
        P.fft_set_slab(n, 16)
        for c in candidates(n):
            P.fft_set_tile(n, P.PMR_FFT_YPASS, *c)
            pm.forward(s)
            F = pm.debug("force", 0).cpu().numpy()[0]
            if ref is None:
                ocfg = OM.Config(BOX, n, n, n, 1, loss_kind=OM.LOSS_DENSITY_L2)
                x = pm.debug("x", 0).cpu().numpy()[0].astype(np.float64)
                ref = OM.force_meshes(ocfg, OM.density(ocfg, x, n))
            e = max(rel_l2(F[:, a], ref[a].ravel()) for a in range(3))
            say(f"  n={n} y {c}: {e:.2e}")
            assert e <= 2e-6
    finally:
        P.fft_set_slab(n, slab)
        P.fft_set_tile(n, P.PMR_FFT_YPASS, *saved)
