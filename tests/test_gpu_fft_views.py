"""The stand-alone inverse transform of a tensor whose memory holds other values than it stands
for: lazily negated, conjugated, and both."""
import pytest
import torch

from paper_1805_02247_amd import api
from _gpu import DEV, require_gpu, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("neg", [False, True])
@pytest.mark.parametrize("conj", [False, True])
def test_lazy_views(neg, conj):
    require_gpu()
    say(f"c2r of a view: negated {neg}, conjugated {conj}")
    n = 16
    g = torch.Generator(device=DEV).manual_seed(3)
    X = torch.randn(2, n, n, n // 2 + 1, dtype=torch.complex64, device=DEV, generator=g)
    view = torch._neg_view(X) if neg else X
    view = view.conj() if conj else view
    assert (view.is_neg(), view.is_conj()) == (neg, conj)
    assert torch.equal(api.fft_c2r(view), api.fft_c2r(view.clone()))
