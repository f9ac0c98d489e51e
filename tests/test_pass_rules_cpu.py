"""Dispatch rules of the row passes without a GPU."""

import ctypes

import pytest


@pytest.mark.parametrize("nw,j,last", [
    (4, 1, 128), (4, 64, 128),                       # 4 slices of the rows
    (4, 65, 64), (4, 128, 64), (8, 129, 64), (8, 256, 64),   # 2 slices
    (8, 65, 128), (8, 128, 128),
    (8, 257, 32), (8, 320, 32),                      # 1 slice
    (16, 129, 96), (16, 192, 96),                    # 16 wavefronts, 3 and 5 chunks: 4 and 2 slices
    (16, 257, 48), (16, 320, 48), (16, 321, 40), (16, 512, 40),
])
def test_reducing_passes_count_the_sums_a_lane_adds(nw, j, last):
    """Passes reduce up to 32 sums per lane (with 16 wavefronts 24 up to 320 columns,
    20 beyond) of the pass before: its workgroups over the slices that the kernel makes of them, a power
    of two."""
    from paper_1805_05821_amd import foa

    f = foa.lib._ZN3foa12pass_reducesEiii
    f.argtypes, f.restype = [ctypes.c_int] * 3, ctypes.c_bool
    assert f(nw, 1, j) and f(nw, last, j) and not f(nw, last + 1, j) and not f(nw, 1024, j)
