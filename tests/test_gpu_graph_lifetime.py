"""Captured graphs go away with their owners, not when the garbage collector comes by, which is
kept from running during a capture (a graph destroyed there aborts the process)."""
import gc
import weakref

import numpy as np
import pytest
import torch

import synth
from paper_1805_02247_amd import _lib as L
from paper_1805_02247_amd import api, cosmo
from paper_1805_02247_amd import recon as R
from _gpu import DEV, require_gpu, say

pytestmark = pytest.mark.gpu


def _context():
    n, box = 16, 100.0
    power = cosmo.linear_power(0.8, 0.2)
    pm = api.PMContext(api.Config(batch=1, n_part=n, n_mesh=n, n_out=n, n_steps=2, box=box,
                                  loss_kind=L.PMR_LOSS_DENSITY_L2), DEV)
    pm.set_prior(torch.from_numpy(cosmo.prior_inv_variance(n, box, power)))
    pm.set_target(torch.zeros(1, n ** 3, device=DEV))
    pm.set_loss(api.LossParams())
    s = cosmo.modes_from_white_noise(synth.white_noise(1, n), box, power).astype(np.complex64)
    return pm, torch.from_numpy(s).reshape(1, -1).to(DEV)


class _Watched(api.GradientGraph):
    def _enqueue(self):
        self.seen = getattr(self, "seen", []) + [(torch.cuda.is_current_stream_capturing(),
                                                  gc.isenabled())]
        super()._enqueue()


@pytest.mark.parametrize("enabled", [True, False])
def test_no_collection_while_capturing(enabled):
    require_gpu()
    say(f"graph capture, collector enabled: {enabled}")
    pm, modes = _context()
    was = gc.isenabled()
    try:
        (gc.enable if enabled else gc.disable)()
        G = _Watched(pm, modes)
        assert gc.isenabled() == enabled
    finally:
        (gc.enable if was else gc.disable)()
    assert (True, False) in G.seen and (True, True) not in G.seen


def test_device_optimiser_is_in_no_cycle():
    require_gpu()
    say("device L-BFGS: lifetime")
    pm, modes = _context()
    was = gc.isenabled()
    gc.disable()
    try:
        D = R.DeviceLBFGS(pm, modes, api.LossParams(), max_iter=2)
        D.stage(modes, api.LossParams())
        torch.cuda.synchronize()
        dead = weakref.ref(D), weakref.ref(D.graph), weakref.ref(D.S)
        graph = D.graph
        del D
        assert dead[0]() is None and dead[2]() is not None  # the graph keeps what it works on
        del graph
        assert all(r() is None for r in dead)
    finally:
        if was:
            gc.enable()
