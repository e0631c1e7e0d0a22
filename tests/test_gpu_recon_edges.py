"""Edges of the reconstruction kernels: binned spectra at the smallest and odd-shaped sizes and
with non-finite modes, and the two-loop direction at every history length's ends."""
import numpy as np
import pytest
import torch

from oracle import stats as ST
from paper_1805_02247_amd import recon as R
from _gpu import DEV, rel_l2, require_gpu, say

pytestmark = pytest.mark.gpu


def _spectra(n, seed):
    r = np.random.default_rng(seed)
    return [(r.standard_normal((n, n, n // 2 + 1)) + 1j * r.standard_normal((n, n, n // 2 + 1)))
            .astype(np.complex64) for _ in range(2)]


# n = 2, 4: fewer rows than a workgroup; 128: kz rows of one wavefront and one lane; nbins from one
# shell to more than hold a mode (n / 2 sqrt(3)).
@pytest.mark.parametrize("n,nbins", [(2, 1), (2, 4), (4, 8), (8, 3), (64, 56), (64, 128), (128, 111)])
def test_power_bins_edges(n, nbins):
    require_gpu()
    say(f"power bins n={n} nbins={nbins}")
    a, b = _spectra(n, n + nbins)
    ta, tb = torch.from_numpy(a).to(DEV), torch.from_numpy(b).to(DEV)
    got = R.power_bins(ta, tb, n, 90.0, nbins).cpu().numpy()
    ref = np.stack(ST.power_bins(a.astype(np.complex128), b.astype(np.complex128), 90.0, nbins))
    assert np.array_equal(got[0], ref[0])
    # FP64 sums of up to n^3 terms that may cancel in the cross power
    scale = np.sqrt(ref[1] * ref[2])
    assert np.all(np.abs(got[1:] - ref[1:]) <= 1e-12 * np.maximum(scale, 1e-300) + 0.0 * ref[1:])
    assert np.array_equal(got, R.power_bins(ta, tb, n, 90.0, nbins).cpu().numpy())


def test_power_bins_keep_a_bad_mode_in_its_shell():
    require_gpu()
    n, nbins = 32, 28
    a, b = _spectra(n, 5)
    clean = R.power_bins(torch.from_numpy(a).to(DEV), torch.from_numpy(b).to(DEV), n, 50.0, nbins)
    a[0, 0, 0] = np.nan  # k = 0 is excluded
    a[3, n - 4, 0] = np.inf  # |m| = 5
    got = R.power_bins(torch.from_numpy(a).to(DEV), torch.from_numpy(b).to(DEV), n, 50.0, nbins)
    keep = torch.arange(nbins, device=DEV) != 5
    assert torch.equal(got[:, keep], clean[:, keep])
    assert not torch.isfinite(got[1, 5]) and torch.equal(got[2], clean[2])


@pytest.mark.parametrize("n,m,count", [(1, 1, 1), (63, 2, 0), (255, 3, 3), (2048, 5, 1), (2049, 64, 64),
                                       (100003, 7, 6), (2100000, 2, 2)])
def test_direction_against_the_64_bit_recursion(n, m, count):
    require_gpu()
    say(f"direction n={n} m={m} count={count}")
    r = np.random.default_rng(n + m)
    S = r.standard_normal((m, n)).astype(np.float32)
    Y = (S * np.exp(0.3 * r.standard_normal((m, n)))).astype(np.float32)
    g = r.standard_normal(n).astype(np.float32)
    order = [int(v) for v in r.permutation(m)[:count]]
    S8, Y8, q = S.astype(np.float64), Y.astype(np.float64), g.astype(np.float64)
    sy, yy = (S8 * Y8).sum(1), (Y8 * Y8).sum(1)
    al = {}
    for i in order:
        al[i] = S8[i] @ q / sy[i]
        q = q - al[i] * Y8[i]
    if order:
        q = q * (sy[order[0]] / yy[order[0]])
    for i in order[::-1]:
        q = q + (al[i] - Y8[i] @ q / sy[i]) * S8[i]
    v = R.VecOps(n, m, DEV)
    t = [torch.from_numpy(x).to(DEV) for x in (g, S, Y, sy, yy)]
    d, d2 = torch.empty_like(t[0]), torch.empty_like(t[0])
    v.direction(t[0], d, order, *t[1:])
    v.direction(t[0], d2, order, *t[1:])
    assert torch.equal(d, d2)
    if count == 0:
        assert torch.equal(d, -t[0])
    # 2 count + 2 roundings per element, amplified by cancellation along the history; a single
    # element (n = 1) cancels to its rounding
    scale = 1.0 if n > 1 else max(np.abs(g[0]) / max(np.abs(q[0]), 1e-300), 1.0)
    assert rel_l2(d.cpu().numpy(), -q) < (2 * count + 2) * 2e-6 * scale
