"""Blocked form (foa_push_blocked, 4 snapshots per sweep of the basis) through
the C ABI: against the blocked oracle (same algorithm, different summation
order), against the sequential oracle within the O(eps kappa) bounds, and the
fallbacks (breakdown, non-finite snapshots, the snapshots of a call that do
not fill a block); an FP64 basis above 256 columns in column windows."""

import numpy as np
import pytest

import datagen
import oracle
import oracle.blocked as ob
from gpu_helpers import EPS32, EPS64, announce, kappa_of, rel
from pins import match_eigs

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _name_case(request):
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    announce(request.node.nodeid)
    yield


def _noisy(n, N, name="noisy_2p20x200"):
    w = datagen.get_workload(name).with_n(n).with_N(N)
    X, lam, b = datagen.snapshots_numpy(w, dtype="float64")
    return X


def _run_blocked(X, prec, tol=-1.0, split=None, snap_dtype=None):
    """Blocked pushes of the columns of X; split: list of (kind, count) with
    kind "b" (blocked) or "s" (single pushes), in order."""
    import torch

    from paper_1805_05821_amd.stream import FOAStream

    n, N = X.shape
    dt = snap_dtype or torch.float64
    Xd = torch.from_numpy(np.ascontiguousarray(X.T)).to(device="cuda", dtype=dt)
    s = FOAStream(n, N, prec=prec, breakdown_tol=tol, ws_fill=0xFF)
    k = 0
    for kind, cnt in (split or [("b", N)]):
        if kind == "b":
            s.push_blocked(Xd[k:k + cnt])
        else:
            s.push_all(Xd[k:k + cnt])
        k += cnt
    from paper_1805_05821_amd import foa as F

    try:
        st, q = s.sync()
    except F.FOAError as e:
        st = e.code
    H, B, q, m = s.state()
    V = s.basis(q).cpu().numpy().T if q > 0 else np.zeros((n, 0))
    return dict(status=st, q=q, m=m, H=H, beta=B, V=V, stream=s)


def _compare(g, ref, c, eps, name):
    q = ref.q
    assert g["q"] == q, (g["q"], q)
    m = q - 1
    kap = kappa_of(ref.beta[:m, :m])
    tol = c * eps * kap * q
    eH = rel(g["H"][:q, :m], ref.H[:q, :m])
    eB = rel(g["beta"][:q, :q], ref.beta[:q, :q])
    orth = np.linalg.norm(np.eye(q) - g["V"].T @ g["V"], 2)
    announce(f"{name}: q={q} kappa={kap:.2e} relH={eH:.2e} relB={eB:.2e} orth={orth:.2e} tol={tol:.2e}")
    assert eH <= tol and eB <= tol
    return kap, orth


@pytest.mark.parametrize("n,N", [(3037, 61), (20000, 121), (64 * 37 + 5, 45)])
def test_blocked_f64_matches_blocked_oracle(n, N):
    X = _noisy(n, N)
    g = _run_blocked(X, "f64")
    ref = ob.foa_blocked(X)
    kap, orth = _compare(g, ref, 10.0, EPS64, "vs blocked oracle")
    assert orth <= 10 * np.sqrt(g["q"]) * EPS64
    seq = oracle.foa_batch(X)
    _compare(g, seq, 10.0, EPS64, "vs sequential oracle")
    g["stream"].close()


@pytest.mark.parametrize("n,N", [(5000, 61), (5000, 300), (5000, 500), (20000, 500)])
def test_blocked_f32_within_bound(n, N):
    """FP32 basis: ||H32 - H64|| <= 10 eps32 kappa and orthogonality.  N = 300
    reaches the 12-group column tile (257-384 columns), N = 500 the widest;
    from about 300 columns on, these noise-floor snapshots need the third
    projection at these n (two projections leave ||I - V^T V|| about 47)."""
    X = _noisy(n, N, "noisy_2p24x500")
    g = _run_blocked(X, "f32")
    seq = oracle.foa_batch(X)
    q = seq.q
    m = q - 1
    kap = kappa_of(seq.beta[:m, :m])
    eH = np.linalg.norm(g["H"][:m, :m] - seq.H[:m, :m], 2) / np.linalg.norm(seq.H[:m, :m], 2)
    orth = np.linalg.norm(np.eye(q) - g["V"].T @ g["V"], 2)
    announce(f"f32 blocked n={n} N={N}: q={g['q']} kappa={kap:.2e} relH2={eH:.2e} (bound {10 * EPS32 * kap:.2e}) "
             f"orth={orth:.2e}")
    assert g["q"] == q
    assert eH <= 10 * EPS32 * kap
    assert orth <= 10 * np.sqrt(q) * EPS32
    g["stream"].close()


@pytest.mark.parametrize("n,N", [(3000, 300), (64 * 33 + 17, 512)])
def test_blocked_f64_column_windows(n, N):
    """FP64 basis beyond 256 columns: the row passes go over column windows
    of at most 256 (the second window from 1 to 252 columns; N = 512 fills
    the capacity).  Against the blocked and the sequential oracle."""
    X = _noisy(n, N)
    g = _run_blocked(X, "f64")
    ref = ob.foa_blocked(X)
    kap, orth = _compare(g, ref, 10.0, EPS64, f"f64 windows N={N} vs blocked oracle")
    assert orth <= 10 * np.sqrt(g["q"]) * EPS64
    seq = oracle.foa_batch(X)
    _compare(g, seq, 10.0, EPS64, f"f64 windows N={N} vs sequential oracle")
    g["stream"].close()


def test_blocked_f64_windows_third_projection(monkeypatch):
    """FP64 basis, rank-250 snapshots plus relative noise 1e-15 and no
    breakdown rule (tol 0): the snapshots past the rank sit at the FP64 noise
    floor and the blocked oracle takes the third projection in about ten of
    the blocks from j = 256 on (which ones depends on the host's rounding),
    i.e. through the column windows.  The oracle's basis keeps
    ||I - V^T V||_2 about 2e-13 with it and 1.3e-10 without it, so the bound
    1e-12 holds only if the gated passes run over both windows.  The leading
    200 columns of H_bar (fixed by the first 201 snapshots) against the
    blocked oracle within 10 m eps kappa_2; the factorisation X = V beta
    within 100 eps."""
    import dataclasses

    base = datagen.get_workload("exact_rank_4096x64")
    w = dataclasses.replace(base, pairs=125, noise=1e-15, kappa_max=None).with_n(2000).with_N(300)
    X, lam, b = datagen.snapshots_numpy(w, dtype="float64")
    g = _run_blocked(X, "f64", tol=0.0)
    fired = []
    test = ob.third_projection_needed

    def record(R1, R2, Z, unit):
        t = test(R1, R2, Z, unit)
        if t:
            fired.append(R1.shape[0])
        return t

    monkeypatch.setattr(ob, "third_projection_needed", record)
    ref = ob.foa_blocked(X, tol=0.0)
    announce(f"oracle third projections at j = {fired}")
    assert len(fired) >= 5 and sum(j > 256 for j in fired) >= 4
    assert g["q"] == ref.q == 300
    V, B = g["V"], g["beta"][:300, :300]
    orth = np.linalg.norm(np.eye(300) - V.T @ V, 2)
    res = np.linalg.norm(X - V @ B) / np.linalg.norm(X)
    m0 = 200
    kap = kappa_of(ref.beta[:m0, :m0])
    eH = rel(g["H"][:m0 + 1, :m0], ref.H[:m0 + 1, :m0])
    announce(f"f64 windows, third projection: orth={orth:.2e} resid={res:.2e} relH[:200]={eH:.2e} "
             f"(bound {10 * m0 * EPS64 * kap:.2e}, kappa {kap:.2e})")
    assert orth <= 1e-12
    assert res <= 100 * EPS64
    assert eH <= 10 * m0 * EPS64 * kap
    g["stream"].close()


def test_blocked_exact_rank_breakdown():
    """The block that crosses the rank is taken one snapshot at a time: the
    breakdown rule fires at snapshot 21 and the generating eigenvalues are exact."""
    w = datagen.get_workload("exact_rank_4096x64")
    X, lam, b = datagen.snapshots_numpy(w)
    g = _run_blocked(X, "f64")
    ref = oracle.foa_batch(X)
    assert g["q"] == ref.q == 20
    ev = np.linalg.eigvals(g["H"][:20, :20])
    err = match_eigs(ev, np.concatenate([lam, np.conj(lam)]))
    announce(f"exact rank: q={g['q']} status={g['status']} eig err={err:.2e}")
    assert err <= 1e-9
    g["stream"].close()


def test_blocked_mixed_with_single_pushes():
    """Single pushes, blocked pushes and parts of fewer than 4, in
    any order, continue one factorisation; FP32 snapshots."""
    import torch

    X = _noisy(4133, 50)
    g = _run_blocked(X, "f64", split=[("s", 3), ("b", 10), ("s", 5), ("b", 23), ("b", 9)],
                     snap_dtype=torch.float32)
    ref = oracle.foa_batch(X.astype(np.float32).astype(np.float64))
    _compare(g, ref, 10.0, EPS64, "mixed")
    g["stream"].close()


def test_blocked_nonfinite_snapshot():
    """A NaN inside a block: the block is rejected, the sequential kernels
    stop the stream before that snapshot."""
    from paper_1805_05821_amd import foa as F

    X = _noisy(2000, 20)
    X[123, 10] = np.nan
    g = _run_blocked(X, "f64")
    ref = oracle.foa_batch(X)
    assert ref.status == "nonfinite" and ref.q == 10
    assert g["q"] == 10 and g["status"] == F.FOA_E_NONFINITE
    assert np.abs(g["H"][:10, :9] - ref.H[:10, :9]).max() <= 1e-10 * np.abs(ref.H[:10, :9]).max()
    g["stream"].close()


def test_blocked_argument_errors():
    import torch

    from paper_1805_05821_amd import foa as F
    from paper_1805_05821_amd.stream import FOAStream

    s = FOAStream(1000, 8, prec="f32")
    X = torch.zeros((9, 1000), dtype=torch.float32, device="cuda")
    with pytest.raises(F.FOAError) as ei:
        s.push_blocked(X)
    assert ei.value.code == F.FOA_E_CAPACITY
    small = torch.empty(256, dtype=torch.uint8, device="cuda")
    with pytest.raises(F.FOAError) as ei:
        F.foa_push_blocked(s.ctx, X, 1000, 4, F.FOA_F32, small, small.numel())
    assert ei.value.code == F.FOA_E_NOMEM
    s.close()


@pytest.mark.parametrize("prec,n,N", [
    ("f64", 70, 30),      # the last panel's second half has no rows
    ("f64", 97, 60),      # one row in the last half panel
    ("f32", 70, 30),
    ("f64", 1100, 276),   # 4 wavefronts up to 256 columns, 8 beyond
    ("f64", 1500, 512),   # the widest tile, full
    ("f32", 1500, 512),
])
def test_block_tiles(prec, n, N):
    """Every tile width of the block passes and ragged last units, from single
    snapshots on (ld > n, FP32 snapshots): Gaussian snapshots (kappa_2 < 20)
    against the sequential oracle."""
    import torch

    from paper_1805_05821_amd.stream import FOAStream

    X = np.random.default_rng(n + N).standard_normal((n, N)).astype(np.float32).astype(np.float64)
    seq = oracle.foa_batch(X, tol=0.0)
    Xd = torch.full((N, n + 5), float("nan"), dtype=torch.float32, device="cuda")
    Xd[:, :n] = torch.from_numpy(np.ascontiguousarray(X.T)).to("cuda")
    s = FOAStream(n, N, prec=prec, breakdown_tol=0.0, ws_fill=0xFF)
    s.push_blocked(Xd[:, :n])
    H, B, q, m = s.state()
    g = dict(q=q, m=m, H=H, beta=B, V=s.basis(q).cpu().numpy().T)
    eps = EPS64 if prec == "f64" else EPS32
    kap, orth = _compare(g, seq, 10.0, eps, f"{prec} {n} x {N}")
    assert orth <= 10 * np.sqrt(q) * eps
    s.close()


@pytest.mark.parametrize("prec,dtype,ld", [("f64", "float64", 95_000_000), ("f32", "float32", 190_000_000),
                                           ("f32", "float64", 95_000_000)])
def test_blocked_rows_far_apart(prec, dtype, ld):
    """Snapshots so far apart that a block's buffer range passes 2^31 bytes, with
    values between them that must not be read as the rows past the end of a
    ragged stream: bitwise the results of the same snapshots side by side."""
    import torch

    n, p = 1000, 9
    dt = getattr(torch, dtype)
    X = np.random.default_rng(ld % 97).standard_normal((n, p))
    ref = _run_blocked(X, prec, snap_dtype=dt)
    from paper_1805_05821_amd.stream import FOAStream

    far = torch.full((p, ld), 1e3, dtype=dt, device="cuda")
    far[:, :n] = torch.from_numpy(np.ascontiguousarray(X.T)).to(device="cuda", dtype=dt)
    s = FOAStream(n, p, prec=prec, ws_fill=0xFF)
    s.push_blocked(far[:, :n])
    st, q = s.sync()
    H, B, q, m = s.state()
    assert q == ref["q"] == p
    assert np.array_equal(H, ref["H"]) and np.array_equal(B, ref["beta"])
    assert np.array_equal(s.basis(q).cpu().numpy().T, ref["V"])
    s.close()
    ref["stream"].close()
    del far
    torch.cuda.empty_cache()


@pytest.mark.parametrize("j0,pos", [(200, 2), (329, 0), (472, 3)])
def test_blocked_rejected_commit(j0, pos):
    """A dependent snapshot inside a block of a wide basis, blocks following in the
    run: the commit's breakdown test rejects the block while the commit's other
    workgroups form the H_bar products, nothing of it is kept and the sequential
    kernels stop the stream at that snapshot.  The same state every time, and the
    oracle's within the blocked bound."""
    n, N = 1300, 496
    X = np.random.default_rng(j0).standard_normal((n, N))
    d = j0 + pos
    X[:, d] = X[:, :d] @ np.random.default_rng(d).standard_normal(d) / np.sqrt(d)
    ref = oracle.foa_batch(X)
    assert ref.q == d
    m = d - 1
    kap = kappa_of(ref.beta[:m, :m])
    first = None
    for _ in range(3):
        g = _run_blocked(X, "f64")
        assert g["q"] == d and g["m"] == d
        eH = rel(g["H"][:d, :d], ref.H[:d, :d])
        announce(f"rejected at {d}: relH={eH:.2e}, kappa={kap:.2e}")
        assert eH <= 10.0 * EPS64 * kap * d
        if first is None:
            first = g
        assert np.array_equal(g["H"], first["H"]) and np.array_equal(g["beta"], first["beta"])
        assert np.array_equal(g["V"], first["V"])
        g["stream"].close()
