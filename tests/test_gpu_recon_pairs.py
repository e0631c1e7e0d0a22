"""The L-BFGS direction at the history lengths where its form changes: none, one and two pairs
(the Gram matrix on the vector units), up to 15 (on the matrix units), more, or buffers of more
slots (the recursion launch by launch)."""
import numpy as np
import pytest
import torch

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
