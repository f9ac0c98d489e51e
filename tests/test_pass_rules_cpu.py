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


def test_sweep_tiles_cover_the_basis():
    """One-reduction sweeps: whatever the columns, the rows and the option ls_nw, the
    tile holds every final column; an FP64 basis takes 8 wavefronts of two-column
    groups at 33-64 columns, at 97-128 from 1024 panels and beyond from 8192."""
    from paper_1805_05821_amd import foa

    nw, qw = foa.lib._ZN3foa5ls_nwEbiil, foa.lib._ZN3foa5ls_qwEbiil
    for f in (nw, qw):
        f.argtypes = [ctypes.c_bool, ctypes.c_int, ctypes.c_int, ctypes.c_int64]
        f.restype = ctypes.c_int
    for P in (1, 1023, 1024, 8191, 8192, 1 << 20):
        for q in range(0, 257):
            w, g = nw(True, q, 0, P), qw(True, q, 0, P)
            rows = 33 <= q <= 64 or (97 <= q <= 128 and P >= 1024) or (q > 128 and P >= 8192)
            assert w == (8 if rows else 4)
            assert g * w * (2 if rows else 4) >= q and g in ((4, 8, 16) if rows else (1, 2, 6, 8, 10, 12, 14, 16))
        for opt in (0, 8, 16):
            for q in range(0, 513):
                w, g = nw(False, q, opt, P), qw(False, q, opt, P)
                assert w == (16 if opt == 16 and 128 < q <= 256 else (4 if q <= 256 else 8))
                assert g * w * 4 >= q
