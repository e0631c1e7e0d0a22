"""The cell sort of clustered particles, whose long rows are neighbours, on meshes with more rows
than the long tier's workgroups test at once, against torch's stable sort of the same keys."""
import pytest
import torch

from paper_1805_02247_amd import api
from _gpu import DEV, require_gpu, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("npart,nm,B,sigma", [(64, 256, 1, 0.02), (64, 128, 4, 0.02), (128, 256, 1, 0.1)])
def test_long_rows_side_by_side(npart, nm, B, sigma):
    require_gpu()
    say(f"clustered sort: {B} x {npart}^3 on {nm}^3, sigma {sigma}")
    g = torch.Generator(device=DEV).manual_seed(npart + nm)
    P = npart ** 3
    x = 0.5 + sigma * torch.randn(B, 3, P, dtype=torch.float64, device=DEV, generator=g)
    x = (x % 1.0) * nm  # one cell per unit length: the corner is the integer part
    keys, ids, rows = api.cic_sort(x, nm, float(nm))
    k = x[:, 0].long().mul_(nm).add_(x[:, 1].long()).mul_(nm).add_(x[:, 2].long())
    k += torch.arange(B, device=DEV)[:, None] * nm ** 3
    k, order = torch.sort(k.reshape(-1), stable=True)
    assert torch.equal(keys.long() & 0xFFFFFFFF, k)
    assert torch.equal(ids.long(), order)
    row = torch.searchsorted(k // nm, torch.arange(B * nm * nm + 1, device=DEV))
    assert torch.equal(rows.long(), row)
