"""The split bf16 products of the FP32 mode reconstruction (foa_modes.hip,
k_modes_split) without a GPU: the bound on what the six products leave out, the
bound that the GPU test sets on a column's error (and that it rejects a kernel
that lacks one of the six), and the rule that sends products there."""

import ctypes

import numpy as np
import pytest

EPS = 2.0 ** -24
TERMS = [(1, 1), (1, 2), (2, 1), (1, 3), (2, 2), (3, 1)]  # (piece of b, piece of w)


def bf16(v):
    """Float32 values rounded to bf16 (nearest even), as float32."""
    u = np.ascontiguousarray(v, dtype=np.float32).view(np.uint32).astype(np.uint64)
    u = (u + 0x7FFF + ((u >> 16) & 1)) & 0xFFFF0000
    return u.astype(np.uint32).view(np.float32)


def pieces(v):
    v = np.asarray(v, dtype=np.float32)
    p1 = bf16(v)
    p2 = bf16(v - p1)
    p3 = bf16(v - p1 - p2)
    assert np.array_equal(p1.astype(np.float64) + p2 + p3, v.astype(np.float64))
    return [p.astype(np.float64) for p in (p1, p2, p3)]


def test_left_out_products_are_below_half_an_ulp():
    """|b w - six products| <= 2^-24 |b w| over significands in [1, 2): Gaussian
    and uniform ones, and those at the far ends of the second and third piece."""
    rng = np.random.default_rng(24)
    ends = [s * (1.0 + i * 2.0 ** -7 + t * 2.0 ** -8 + u * 2.0 ** -16 + d * 2.0 ** -17 + e * 2.0 ** -23)
            for i in (0, 1, 2, 64, 126) for t in (-1, 0, 1) for u in (-1, 0, 1) for d in (-1, 0, 1) for e in (-1, 0, 1)
            for s in (1, -1)]
    ends = np.unique(np.array(ends, dtype=np.float32))
    near = (1.0 + rng.integers(0, 1 << 17, 2000) * 2.0 ** -23).astype(np.float32)
    wide = rng.standard_normal(2000).astype(np.float32)
    v = np.concatenate([ends, near, wide])
    b, w = pieces(v), pieces(v)
    worst = 0.0
    for i in range(len(v)):
        six = sum(b[p - 1][i] * w[q - 1] for p, q in TERMS)
        exact = float(v[i]) * v.astype(np.float64)
        worst = max(worst, float(np.max(np.abs(six - exact) / np.abs(exact))))
    assert worst <= EPS
    assert worst > 0.5 * EPS  # the values above come near the bound


@pytest.mark.parametrize("m", [32, 52, 160, 257])
def test_column_bound_separates_the_six_products(m):
    """sqrt(m) 2^-24 (the bound of test_mode_split_error): met by the six
    products with room for the accumulation's roundings, exceeded when any of the
    smallest three is missing."""
    rng = np.random.default_rng(m)
    n = 4096
    W = np.linalg.qr(rng.standard_normal((n, m)))[0].astype(np.float32)
    B = rng.standard_normal((m, 8))
    B = (B / np.linalg.norm(B, axis=0)).astype(np.float32)
    ref = W.astype(np.float64) @ B.astype(np.float64)
    bp, wp = pieces(B), pieces(W)

    def err(terms):
        s = sum(wp[q - 1] @ bp[p - 1] for p, q in terms)
        return np.max(np.linalg.norm(s - ref, axis=0) / np.linalg.norm(ref, axis=0))

    bound = np.sqrt(m) * EPS
    assert err(TERMS) <= 0.5 * EPS
    for i in range(3, 6):
        assert err(TERMS[:i] + TERMS[i + 1:]) > 1.5 * bound, TERMS[i]


@pytest.fixture(scope="module")
def lib():
    from paper_1805_05821_amd import foa

    return foa.lib


def test_split_rule(lib):
    """From 2^31 multiply-adds and 48 basis columns on."""
    pays = getattr(lib, "_ZN3foa16modes_split_paysElii")
    pays.argtypes, pays.restype = [ctypes.c_int64, ctypes.c_int, ctypes.c_int], ctypes.c_bool
    assert pays(1 << 19, 64, 64) and not pays((1 << 19) - 1, 64, 64)
    assert not pays(1 << 40, 47, 47) and not pays(1 << 40, 1, 1) and not pays(1 << 40, 2, 2)
    assert pays(1 << 31, 48, 1)


def test_split_range(lib):
    """Coefficients the split takes: every basis column's largest in [2^-60, 2^60]
    (a column without a coefficient leaves its values unbounded), none beyond."""
    ok = getattr(lib, "_ZN3foa14modes_split_okEPKfiim")
    ok.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_int, ctypes.c_size_t]
    ok.restype = ctypes.c_bool
    k, r, ld = 5, 3, 32
    base = np.zeros((k, ld), dtype=np.float32)
    base[:, :r] = np.random.default_rng(5).standard_normal((k, r))

    def check(row):
        B = base.copy()
        B[2, :r] = row
        return ok(B.ctypes.data, k, r, ld)

    assert check([1.0, 0.0, 0.0]) and check([2.0 ** 60, 2.0 ** -140, 0.0]) and check([0.0, -(2.0 ** -60), 0.0])
    assert not check([0.0, 0.0, 0.0])
    assert not check([2.0 ** 61, 1.0, 1.0]) and not check([2.0 ** -61, 0.0, 2.0 ** -90])
    assert not check([np.nan, 1.0, 1.0]) and not check([np.inf, 1.0, 1.0])
