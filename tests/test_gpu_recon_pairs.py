"""The L-BFGS direction at the history lengths where its form changes: none, one and two pairs
(the Gram matrix on the vector units), up to 15 (on the matrix units), more, or buffers of more
slots (the recursion launch by launch)."""
import ctypes
import math

import numpy as np
import pytest
import torch

import synth
from paper_1805_02247_amd import _lib as L
from paper_1805_02247_amd import api, cosmo
from paper_1805_02247_amd import recon as R
from _gpu import DEV, rel_l2, require_gpu, say

pytestmark = pytest.mark.gpu


def _history(n, m, seed):
    r = np.random.default_rng(seed)
    S = r.standard_normal((m, n)).astype(np.float32)
    Y = (S * np.exp(0.3 * r.standard_normal((m, n)))).astype(np.float32)
    return S, Y, r.standard_normal(n).astype(np.float32), [int(v) for v in r.permutation(m)]


def _direction64(S, Y, g, order):
    S8, Y8, q = S.astype(np.float64), Y.astype(np.float64), g.astype(np.float64)
    al = {}
    for i in order:
        al[i] = S8[i] @ q / (S8[i] @ Y8[i])
        q = q - al[i] * Y8[i]
    if order:
        q = q * ((S8[order[0]] @ Y8[order[0]]) / (Y8[order[0]] @ Y8[order[0]]))
    for i in order[::-1]:
        q = q + (al[i] - Y8[i] @ q / (S8[i] @ Y8[i])) * S8[i]
    return -q


# n: below a wavefront's 64 elements, not a multiple of 4 (no 16-byte loads), several blocks;
# the last digit moves every vector off its 16-byte alignment by that many floats
@pytest.mark.parametrize("n,m,count,off", [
    (61, 15, 15, 0), (4099, 15, 15, 0), (61, 16, 15, 0), (4100, 16, 15, 2), (61, 16, 16, 0),
    (4099, 16, 16, 0), (4099, 17, 15, 0), (61, 17, 16, 0), (4100, 11, 3, 0), (4099, 14, 13, 0),
    (5, 4, 1, 0), (2047, 16, 2, 0), (4100, 2, 2, 1), (300001, 3, 1, 0), (8192, 3, 0, 3), (262148, 2, 1, 0)])
def test_direction(n, m, count, off):
    require_gpu()
    say(f"direction n={n} m={m} count={count} off={off}")
    S, Y, g, order = _history(n, m, n + m)
    order = order[:count]
    ref = _direction64(S, Y, g, order)
    sy = (S.astype(np.float64) * Y).sum(1)
    yy = (Y.astype(np.float64) ** 2).sum(1)

    def dev(x):
        t = torch.empty(x.size + off, dtype=torch.float32, device=DEV)[off:]
        t.copy_(torch.from_numpy(x.reshape(-1)))
        return t.reshape(x.shape)

    tS, tY, tg = dev(S), dev(Y), dev(g)
    tsy, tyy = torch.from_numpy(sy).to(DEV), torch.from_numpy(yy).to(DEV)
    d, again = torch.empty_like(tg), torch.empty_like(tg)
    v = R.VecOps(n, m, DEV)
    v.direction(tg, d, order, tS, tY, tsy, tyy)
    v.direction(tg, again, order, tS, tY, tsy, tyy)
    assert torch.equal(d, again)
    if count == 0:
        assert torch.equal(d, -tg)
    # one rounding per element and FP64 inner products, amplified by cancellation along the
    # history (the bound of the directions of other lengths)
    assert rel_l2(d.cpu().numpy(), ref) < (2 * count + 2) * 2e-6


# 15: the longest history in the Gram form (16 slots on the host), 16 and more: launch by launch
@pytest.mark.parametrize("m", [1, 2, 14, 15, 16, 20])
def test_both_drivers_take_the_same_steps(m):
    """Enough iterations to fill and turn over the history; the losses and the modes are the same
    bit for bit."""
    require_gpu()
    n, box, iters = 16, 100.0, m + 6
    say(f"L-BFGS drivers: m={m}")
    power = cosmo.linear_power(0.8, 0.2)
    modes = [torch.from_numpy(cosmo.modes_from_white_noise(synth.white_noise(q, n), box, power)
                              .astype(np.complex64)).reshape(1, -1).to(DEV) for q in (1, 2)]

    def context():
        pm = api.PMContext(api.Config(batch=1, n_part=n, n_mesh=n, n_out=n, n_steps=2, box=box,
                                      loss_kind=L.PMR_LOSS_DENSITY_L2), DEV)
        pm.set_prior(torch.from_numpy(cosmo.prior_inv_variance(n, box, power)))
        pm.set_target(torch.zeros(1, n ** 3, device=DEV))
        pm.set_loss(api.LossParams())
        pm.forward(modes[0], want_mass=False)
        pm.set_target(pm.debug("delta_f").reshape(1, -1).clone())
        return pm

    a, b = modes[1].clone(), modes[1].clone()
    host = R.minimize(context(), a, max_iter=iters, m=m, rel_tol=0.0)
    D = R.DeviceLBFGS(context(), b, api.LossParams(), m=m, max_iter=iters)
    dev = D.stage(b, api.LossParams(), rel_tol=0.0)
    say(f"  {host.iters} iterations, {host.evals} evaluations, {host.reason}")
    assert host.iters == iters and host.reason == "max_iter"
    assert (dev.losses, dev.iters, dev.evals, dev.reason) == (host.losses, host.iters, host.evals,
                                                              host.reason)
    assert torch.equal(torch.view_as_real(a), torch.view_as_real(b))


def test_update_with_a_shorter_history_than_the_state_holds():
    """The caller's m is below the state's, which the header forbids and no call can see: a
    descent direction from the newest 15 pairs, and nothing outside the buffers."""
    require_gpu()
    say("L-BFGS update: m below the state's")
    n, m, guard = 200, 20, 512
    lib = L.lib()
    f32 = dict(dtype=torch.float32, device=DEV)
    f64 = dict(dtype=torch.float64, device=DEV)
    diag = torch.logspace(0.0, 1.5, n, **f32)
    x, xt, g, gt, d = (torch.ones(n, **f32) for _ in range(5))
    S, Y = torch.zeros(m + 1, n, **f32), torch.zeros(m + 1, n, **f32)
    sy, yy = torch.zeros(m + 1, **f64), torch.zeros(m + 1, **f64)
    words = int(lib.pmr_vec_work_bytes(n, 0)) // 8
    work = torch.full((words + guard,), 7.0, **f64)
    state = torch.zeros(int(lib.pmr_lbfgs_state_bytes(100)) // 8, **f64)
    loss = torch.zeros(1, **f64)

    def evaluate(at, grad):
        grad.copy_(diag * at + 0.1 * at ** 3)
        loss[0] = (0.5 * diag * at ** 2 + 0.025 * at ** 4).double().sum()

    def held():
        raw = state.view(torch.uint8)[:ctypes.sizeof(L.PmrLbfgsState)].cpu().numpy().tobytes()
        return L.PmrLbfgsState.from_buffer_copy(raw)

    evaluate(x, g)
    prm = L.PmrLbfgsParams(m=m, max_iter=100, max_halvings=30, c1=1e-4, curvature_eps=0.0,
                           rel_tol=0.0, stop_below=-math.inf)
    p, s = api._ptr, api._stream()
    L.check(lib.pmr_lbfgs_init(n, ctypes.byref(prm), p(state), p(loss), p(g), p(d), p(S), p(Y), p(sy),
                               p(yy), p(work), s))
    for k in range(60):
        L.check(lib.pmr_lbfgs_trial(n, p(state), p(x), p(d), p(xt), s))
        evaluate(xt, gt)
        short = held().count >= 17
        L.check(lib.pmr_lbfgs_update(n, 10 if short else m, p(state), p(loss), p(x), p(g), p(xt),
                                     p(gt), p(d), p(S), p(Y), p(sy), p(yy), p(work), s))
        torch.cuda.synchronize()
        if short and held().accepted:
            break
    st = held()
    assert st.count >= 17 and st.accepted and st.status == 1
    assert torch.isfinite(d).all() and float((g.double() @ d.double())) < 0.0
    assert torch.equal(work[words:], torch.full((guard,), 7.0, **f64))
    order = list(st.order[:15])
    ref = _direction64(S.cpu().numpy(), Y.cpu().numpy(), g.cpu().numpy(), order)
    assert rel_l2(d.cpu().numpy(), ref) < 32 * 2e-6
