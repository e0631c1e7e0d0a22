"""Host-side checks of the inverse transform with a work buffer: nothing is launched where the
buffer is missing, misaligned or overlaps the input."""
import ctypes

import pytest

from paper_1805_02247_amd import _lib as L

P = ctypes.c_void_p


@pytest.mark.parametrize("n,batch", [(16, 1), (16, 3), (64, 2)])
def test_work_buffer(n, batch):
    lib = L.lib()
    inp = batch * n * n * (n // 2 + 1) * 8
    need = lib.pmr_fft_c2r_work_bytes(n, batch)
    assert need >= inp
    base, out = 1 << 34, P(1 << 40)  # never dereferenced: every call below is refused
    for work in (None, base + (1 << 30) + 8):
        assert lib.pmr_fft_c2r_work(n, batch, P(base), P(work), out, None) == -1
    for work in (base, base + 16, base + (inp - 1) // 16 * 16, base - need + 16):
        assert lib.pmr_fft_c2r_work(n, batch, P(base), P(work), out, None) == -1
