"""The paint of the last row of a mesh of 2^32 cells in all, the most it takes: the keys of its
last cells are also those of lanes without a particle."""
import pytest
import torch

from paper_1805_02247_amd import api
from _gpu import DEV, require_gpu, say

pytestmark = pytest.mark.gpu


# The last valid lane of the row's only chunk is `lane`, in cell iz = 62 - lane: with one particle
# per cell before it (alone), or with the whole run in that cell (together).
@pytest.mark.parametrize("lane,together", [(0, False), (1, False), (20, True), (62, True)])
def test_mass_of_the_last_item(lane, together):
    require_gpu()
    say(f"paint last cells: lane={lane} together={together}")
    npart, nm, B, P = 16, 64, 16384, 16 ** 3
    box = float(nm)
    x = torch.full((B, 3, P), 0.5, dtype=torch.float64, device=DEV)
    # the last item: lane + 1 particles in row (63, 63), the others far from it
    last = x[-1]
    last[0], last[1], last[2] = 20.25, 20.5, 20.75
    iz = 62 - lane
    last[:2, :lane + 1] = 63.25
    cells = torch.full((lane + 1,), float(iz), dtype=torch.float64, device=DEV)
    if not together:
        cells -= torch.arange(lane, -1, -1, dtype=torch.float64, device=DEV)
    last[2, :lane + 1] = cells + 0.25
    keys, ids, rows = api.cic_sort(x, nm, box)
    assert int(keys[-1].item()) & 0xFFFFFFFF == 0xFFFFFFFF - lane - 1
    out = api.cic_paint(x, keys, ids, rows, nm, box).reshape(B, -1)
    total = out[-1].double().sum().item()
    say(f"  mass {total}")
    # weights are multiples of 1/64 and the cells' sums are small: exact in FP32
    assert total == P
    assert out[0].double().sum().item() == P
