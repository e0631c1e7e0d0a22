"""The cell sort at the edges of its tiers, scans and lane networks, bit for bit against the
oracle's (key, id) order."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import mesh as M
from paper_1805_02247_amd import _lib as L
from paper_1805_02247_amd import api
from _gpu import DEV, require_gpu, say

pytestmark = pytest.mark.gpu


def _check(x, nm, box, keys, ids, rows):
    B = x.shape[0]
    k = np.concatenate([b * nm ** 3 + M.cell_keys(x[b], nm, box) for b in range(B)])
    order = M.sort_order(k)
    assert np.array_equal(keys.cpu().numpy().view(np.uint32), k[order].astype(np.uint32))
    assert np.array_equal(ids.cpu().numpy().view(np.uint32), order.astype(np.uint32))
    row = np.searchsorted(k[order] // nm, np.arange(B * nm * nm + 1), side="left")
    assert np.array_equal(rows.cpu().numpy().view(np.uint32), row.astype(np.uint32))


# 32^3 particles on a 16^3 mesh: 128 per row on average, so a segment is half a row. Rows of
# the given lengths, the rest of the particles spread over the other rows.
@pytest.mark.parametrize("lengths", [(1, 2, 31, 32, 33, 63, 64, 65), (127, 128, 129, 191, 192),
                                     (255, 256, 257, 511, 512, 513), (4095, 4096, 4097, 9000)])
@pytest.mark.parametrize("one_half", [True, False])
def test_segment_lengths_at_the_tier_edges(lengths, one_half):
    require_gpu()
    say(f"sort tiers: lengths {lengths}, in one half row: {one_half}")
    npart, nm, box = 32, 16, 16.0
    P = npart ** 3
    r = np.random.default_rng(len(lengths) + one_half)
    cell = np.empty((3, P), dtype=np.int64)
    at = 0
    for i, n in enumerate(lengths):
        cell[0, at:at + n], cell[1, at:at + n] = i, (5 * i) % nm
        cell[2, at:at + n] = r.integers(0, 8 if one_half else 16, n)
        at += n
    cell[0, at:] = r.integers(len(lengths), nm, P - at)
    cell[1, at:] = r.integers(0, nm, P - at)
    cell[2, at:] = r.integers(0, nm, P - at)
    x = (cell + r.uniform(0.0, 0.999, (3, P)))[:, r.permutation(P)][None]
    keys, ids, rows = api.cic_sort(torch.from_numpy(x).to(DEV), nm, box)
    _check(x, nm, box, keys, ids, rows)


# 16^3 particles: a row count below one scan tile, the most rows the one-launch scan takes
# (512^2), and twice as many (three launches); and a scratch buffer that is only 4-byte aligned.
@pytest.mark.parametrize("B,nm,shift", [(1, 16, 0), (3, 16, 0), (1, 512, 0), (2, 512, 0), (1, 64, 4)])
def test_scan_paths(B, nm, shift):
    require_gpu()
    say(f"sort scans: B={B} nm={nm} scratch offset {shift}")
    npart, box = 16, 100.0
    total = B * npart ** 3
    x = np.random.default_rng(nm + B).uniform(0.0, box, (B, 3, npart ** 3))
    xt = torch.from_numpy(x).to(DEV)
    need = int(L.lib().pmr_sort_scratch_bytes(total, nm, B))
    scratch = torch.full((need + 64,), 255, dtype=torch.uint8, device=DEV)
    out = [torch.empty(n, dtype=torch.int32, device=DEV) for n in (total, total, B * nm * nm + 1)]
    L.check(L.lib().pmr_cic_sort(npart, nm, B, box, api._ptr(xt), *[api._ptr(t) for t in out],
                                 ctypes.c_void_p(scratch.data_ptr() + shift), need,
                                 api._stream()))
    torch.cuda.synchronize()
    assert int((scratch[need + shift:] != 255).sum()) == 0
    _check(x, nm, box, *out)


# 2^25 segments, the most that the kernels writing the keys count, and twice as many (a pass of
# its own), against torch's stable sort of the same integer keys.
@pytest.mark.parametrize("B", [8192, 16384])
def test_both_ways_to_count(B):
    require_gpu()
    say(f"sort counts: B={B}")
    npart, nm, box = 16, 64, 64.0  # one cell per unit length: the corner is the integer part
    g = torch.Generator(device=DEV).manual_seed(B)
    x = torch.rand(B, 3, npart ** 3, dtype=torch.float64, device=DEV, generator=g) * box
    keys, ids, rows = api.cic_sort(x, nm, box)
    k = x[:, 0].long().mul_(nm).add_(x[:, 1].long()).mul_(nm).add_(x[:, 2].long())
    k += torch.arange(B, device=DEV)[:, None] * nm ** 3
    k, order = torch.sort(k.reshape(-1), stable=True)
    assert torch.equal(keys.long() & 0xFFFFFFFF, k)
    assert torch.equal(ids.long() & 0xFFFFFFFF, order)
    row = torch.searchsorted(k // nm, torch.arange(B * nm * nm + 1, device=DEV))
    assert torch.equal(rows.long() & 0xFFFFFFFF, row)
