"""The buffer range of the blocked passes (foa_block.hip, load_xs) without a GPU:
at both ends of what the host lets through, rows that exist are inside the
range, and the offset of the others is not (there the load returns 0)."""

import ctypes

import pytest

BPK, PANEL = 4, 64


@pytest.fixture(scope="module")
def lib():
    from paper_1805_05821_amd import foa

    ok = foa.lib._ZN3foa14block_range_okEli
    ok.argtypes, ok.restype = [ctypes.c_int64, ctypes.c_int], ctypes.c_bool
    rng = foa.lib._ZN3foa13block_x_rangeElii
    rng.argtypes, rng.restype = [ctypes.c_int64, ctypes.c_int, ctypes.c_int], ctypes.c_uint32
    return ok, rng


@pytest.mark.parametrize("es", [4, 8])
@pytest.mark.parametrize("rows", [32, 64])
def test_masked_rows_are_out_of_range(lib, es, rows):
    ok, x_range = lib
    last = max(ld for ld in range(2 ** 32 // (BPK * es) - 200, 2 ** 32 // (BPK * es) + 10) if ok(ld, es))
    assert not ok(last + 1, es) and not ok(2 * last, es)
    half = 2 ** 31 // ((BPK - 1) * es)  # where the range passes 2^31
    for ld in (1, 1000, half - 100, half - 1, half, half + 1, half + 100, 95_000_000 * 8 // es, last - 1, last):
        assert ok(ld, es)
        mask = x_range(ld, rows, es)  # the range, and the offset of rows past the end
        assert mask == ((BPK - 1) * ld + rows) * es  # nothing lost to 32 bits
        assert mask + es <= 2 ** 32  # an access there does not wrap
        for k in range(BPK):
            assert (k * ld + rows - 1) * es + es <= mask
