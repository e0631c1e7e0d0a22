"""The autotuner offers only choices that its workload can tell apart."""
import paper_1805_02247_amd as P
from paper_1805_02247_amd import tune


def test_stand_alone_transforms():
    for n in (32, 64, 128, 256):
        assert tune.fft_candidates(n, "x") == tune.candidates(n)
    assert tune.fft_candidates(256, "y") == tune.candidates(256)
    for n in (32, 64, 128):
        cur = P.fft_get_tile(n, P.PMR_FFT_YPASS)
        got = tune.fft_candidates(n, "y")
        assert got and {c[:2] for c in got} == {cur[:2]}
        assert {c[2] for c in got} == {c[2] for c in tune.candidates(n) if c[:2] == cur[:2]}


def test_paint_rows():
    assert tune.paint_candidates(64, 3) == tune.paint_candidates(512, 1) == (1, 2, 4, 8, 16)
    assert tune.paint_candidates(128, 3) == tune.paint_candidates(512, 3) == (1, 2)
