"""The work a user has this framework do, case by case: streams of snapshots
pushed through each form of the FOA step (three-sweep CGS2, blocked,
one-reduction, batched) in both basis precisions, the mode reconstruction and
a whole DMD analysis.

A pass starts from the handle and the snapshots that a program keeps: it
resets the stream, pushes every snapshot and reads the results back (H_bar,
beta and the basis; eigenvalues, amplitudes and modes for the last two paths).

Snapshots are travelling oscillations with amplitudes over half a decade and a
white background: x_j = Re(sum_m a_m phi_m lambda_m^j) + noise, the form of
the repository's workloads with a background that keeps kappa_2 moderate, so
that results are determined well beyond the storage precision.
"""

import math

import numpy as np
import torch

from paper_1805_05821_amd import foa as F
from paper_1805_05821_amd.stream import FOABatch, FOAStream

DEVICE = "cuda"
EPL = {"f32": 4, "f64": 8}  # bytes of an element


def listed():
    return [
        # the smallest calls: a short record of a small field (ragged rows), one
        # snapshot per call; launches and latency are all of it
        dict(name="push_1000x24_f32", path="push", n=1000, N=24, prec="f32", x="f32"),
        # the sizes of the exact-rank workload, one snapshot per call, FP64 basis
        dict(name="push_4096x64_f64", path="push", n=4096, N=64, prec="f64", x="f64"),
        # an ordinary stream with an odd row count, FP32 basis
        dict(name="push_100037x128_f32", path="push", n=100037, N=128, prec="f32", x="f32"),
        # noisy_2p20x200: an FP64 field of a million rows, FP64 basis
        dict(name="push_2p20x200_f64", path="push", n=1 << 20, N=200, prec="f64", x="f64"),
        # the throughput workload's 500 snapshots at an eighth of its rows (a pass
        # of the full size takes four seconds), FP32 basis
        dict(name="push_2p21x500_f32", path="push", n=1 << 21, N=500, prec="f32", x="f32"),
        # the same workload through the blocked form, at a quarter of its rows
        dict(name="blocked_2p22x500_f32", path="blocked", n=1 << 22, N=500, prec="f32", x="f32"),
        # blocked form, FP64 basis beyond 256 columns, ragged rows
        dict(name="blocked_300007x320_f64", path="blocked", n=300007, N=320, prec="f64", x="f64"),
        # one-reduction form of the throughput workload, an eighth of its rows
        dict(name="one_reduction_2p21x500_f32", path="one_reduction", n=1 << 21, N=500, prec="f32", x="f32"),
        # batched_256's shape (256 streams, 2^12..2^18 rows, 20..300 snapshots)
        dict(name="batch_256_f32", path="batch", S=256, n_lo=1 << 12, n_hi=1 << 18, N_lo=20, N_hi=300, prec="f32",
             x="f32", form="cgs2"),
        # a quarter as many streams in the one-reduction form
        dict(name="batch_64_one_reduction_f32", path="batch", S=64, n_lo=1 << 12, n_hi=1 << 18, N_lo=20, N_hi=300,
             prec="f32", x="f32", form="one_reduction"),
        # mode reconstruction of 160 packed columns (the large workload's), FP32
        # basis and modes; the stream and its eigenpairs are in hand
        dict(name="modes_2p22_r160_f32", path="modes", n=1 << 22, N=161, r=160, prec="f32", x="f32", phi="f32"),
        # a whole analysis with an FP64 basis: stream, truncate, modes in FP64
        dict(name="dmd_2p18x150_r60_f64", path="dmd", n=1 << 18, N=150, r=60, prec="f64", x="f64", phi="f64"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["push", "push", "push", "blocked", "blocked", "one_reduction", "one_reduction", "batch", "modes",
                       "dmd"])
    prec = rng.choice(["f32", "f64"])
    if path == "batch":
        n_lo = _log(rng, 300, 8000)
        return dict(path="batch", S=rng.randint(8, 64), n_lo=n_lo, n_hi=_log(rng, 2 * n_lo, 1 << 17),
                    N_lo=rng.randint(8, 40), N_hi=rng.randint(48, 200), prec=prec, x=rng.choice(["f32", prec]),
                    form=rng.choice(["cgs2", "one_reduction"]))
    if path == "modes":
        pairs = rng.randint(4, 80)
        return dict(path="modes", n=_log(rng, 5000, 1 << 21), N=2 * pairs + 1, r=2 * pairs, prec=prec,
                    x=rng.choice(["f32", prec]), phi=rng.choice([prec, "f64"]))
    if path == "dmd":
        pairs = rng.randint(3, 24)
        return dict(path="dmd", n=_log(rng, 2000, 1 << 18), N=rng.randint(3 * pairs + 8, 3 * pairs + 60), r=2 * pairs,
                    prec=prec, x=prec, phi=prec)
    if path == "one_reduction" and prec == "f64":
        N = _log(rng, 12, 250)
    else:
        N = _log(rng, 12, 500)
    rows = int(min(1 << 22, 2 ** 40 / N / N))  # no more than the largest listed stream's work
    n = _log(rng, max(700, 3 * N), rows)
    return dict(path=path, n=n, N=N, prec=prec, x=rng.choice(["f32", prec]))


# ---- inputs ------------------------------------------------------------------

def _pairs(N):
    return max(1, min(80, N // 3))


def _dtype(name):
    return torch.float64 if name == "f64" else torch.float32


def _snapshots(n, N, dtype, gen, pairs, noise):
    """(N, n) snapshots on the GPU, one per row."""
    M = pairs
    a = torch.logspace(0.0, -0.5, M, device=DEVICE, dtype=torch.float64)
    step = (math.pi - 0.2) / M
    om = 0.1 + step * (torch.arange(M, device=DEVICE, dtype=torch.float64) + 0.35
                       + 0.3 * torch.rand(M, generator=gen, device=DEVICE, dtype=torch.float64))
    sg = -0.002 * torch.rand(M, generator=gen, device=DEVICE, dtype=torch.float64)
    j = torch.arange(N, device=DEVICE, dtype=torch.float64)
    amp = a * torch.exp(j[:, None] * sg)
    time = torch.cat([amp * torch.cos(j[:, None] * om), -amp * torch.sin(j[:, None] * om)], dim=1).to(torch.float32)
    X = torch.empty((N, n), dtype=dtype, device=DEVICE)
    rms = float(a.square().sum().sqrt())
    chunk = max(1, (1 << 29) // max(N, 2 * M))
    for r0 in range(0, n, chunk):
        m = min(chunk, n - r0)
        phi = torch.randn((2 * M, m), generator=gen, device=DEVICE, dtype=torch.float32)
        e = torch.randn((N, m), generator=gen, device=DEVICE, dtype=torch.float32)
        X[:, r0:r0 + m] = torch.addmm(e, time, phi, beta=noise * rms)
    return X


def _noise(case):
    # background relative to the signal: the snapshots of an FP32 basis are
    # kept further from its rounding than those of an FP64 one
    if case["path"] in ("modes", "dmd"):
        return 0.02 if case["prec"] == "f32" else 0.005
    return 0.1 if case["prec"] == "f32" else 0.005


def _gen(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(1805_05821 + int(seed))
    return g


def _inputs(case, seed):
    """The snapshots of a case: one (N, n) matrix, or a list of them (batch)."""
    gen = _gen(seed)
    if case["path"] == "batch":
        # shapes belong to the case: the same for every seed
        r = np.random.default_rng(case["S"] * 1000003 + case["n_lo"] + case["N_hi"])
        ns = np.exp(r.uniform(math.log(case["n_lo"]), math.log(case["n_hi"]), case["S"])).astype(int)
        Ns = r.integers(case["N_lo"], case["N_hi"] + 1, case["S"])
        return [_snapshots(int(n), int(min(N, n // 3)), _dtype(case["x"]), gen, _pairs(int(min(N, n // 3))), _noise(case))
                for n, N in zip(ns, Ns)]
    pairs = case["r"] // 2 if "r" in case else _pairs(case["N"])
    return _snapshots(case["n"], case["N"], _dtype(case["x"]), gen, pairs, _noise(case))


def prepare(case, seed):
    X = _inputs(case, seed)
    if case["path"] == "batch":
        n = [x.shape[1] for x in X]
        N = [x.shape[0] for x in X]
        b = FOABatch(n, N, prec=case["prec"], device=DEVICE, form=case["form"])
        steps = max(N)
        ptrs = torch.tensor([[X[s][t].data_ptr() if t < N[s] else 0 for s in range(len(X))] for t in range(steps)],
                            dtype=torch.int64, device=DEVICE)
        views = [b.view(s) for s in range(len(X))]
        return dict(case=case, X=X, b=b, ptrs=ptrs, views=views, V=_flat(n, N, _dtype(case["prec"])))
    s = FOAStream(case["n"], case["N"], prec=case["prec"], device=DEVICE,
                  form="one_reduction" if case["path"] == "one_reduction" else "cgs2")
    st = dict(case=case, X=X, s=s)
    if "r" in case:
        st["phi"] = torch.empty((case["r"], case["n"]), dtype=_dtype(case["phi"]), device=DEVICE)
    if case["path"] == "modes":
        s.push_block(X)
        s.indicators()
        st["X"] = None
    return st


def _flat(n, N, dtype):
    return torch.empty(sum(a * b for a, b in zip(n, N)), dtype=dtype, device=DEVICE)


# ---- one pass ------------------------------------------------------------------

def _modes(st):
    s, case = st["s"], st["case"]
    lam, kind, amp, err = s.modes(m_max=case["r"], phi=st["phi"], phi_cols=case["r"],
                                  phi_dtype=F.FOA_F64 if case["phi"] == "f64" else F.FOA_F32)
    return [lam, kind, amp, err, st["phi"]]


def run(st):
    case = st["case"]
    path = case["path"]
    if path == "modes":
        return _modes(st)
    if path == "batch":
        b, x_dtype = st["b"], F.FOA_F64 if case["x"] == "f64" else F.FOA_F32
        b.reset()
        for t in range(st["ptrs"].shape[0]):
            b.push_ptrs(st["ptrs"][t], x_dtype)
        q, status = b.sync()
        H, B, off = [], [], 0
        v_dtype = F.FOA_F64 if case["prec"] == "f64" else F.FOA_F32
        for k, v in enumerate(st["views"]):
            h, bt, qk, _ = F.foa_get_state(v)
            H.append(h.ravel())
            B.append(bt.ravel())
            n = b.n[k]
            F.foa_copy_basis(v, st["V"][off:], n, v_dtype, qk)
            off += n * qk
        return [q, status, np.concatenate(H), np.concatenate(B), st["V"]]
    s, X = st["s"], st["X"]
    s.reset()
    if path == "blocked":
        s.push_blocked(X)
    elif path == "dmd":
        s.push_block(X)
        s.truncate(r_force=case["r"])
        return _modes(st)
    else:
        s.push_all(X)
    H, B, q, m = s.state()
    return [q, m, H, B, s.basis(q, _dtype(case["prec"]))]


# ---- what a pass cannot do without --------------------------------------------

def _stream_work(n, N, sv, sx, path):
    """Bytes and flops of the pushes of one stream: the sweeps over the basis
    columns held that the form's order of operations forces (three per
    snapshot for CGS2, two per four snapshots blocked, one per snapshot in the
    one-reduction form), each snapshot read once, each column written once and
    read once when the basis is handed out."""
    cols = N * (N - 1) / 2.0  # columns held, summed over the pushes
    io = n * N * (sx + sv)
    if path == "blocked":
        return n * cols * sv * 2 / 4 + io, n * cols * 8
    if path == "one_reduction":
        return n * cols * sv + io, n * cols * 8
    return n * cols * sv * 3 + io, n * cols * 10


def work(case):
    sv, sx = EPL[case["prec"]], EPL[case["x"]]
    if case["path"] == "batch":
        r = np.random.default_rng(case["S"] * 1000003 + case["n_lo"] + case["N_hi"])
        ns = np.exp(r.uniform(math.log(case["n_lo"]), math.log(case["n_hi"]), case["S"])).astype(int)
        Ns = r.integers(case["N_lo"], case["N_hi"] + 1, case["S"])
        parts = [_stream_work(int(n), int(min(N, n // 3)), sv, sx, case["form"]) for n, N in zip(ns, Ns)]
        out = sum(2 * int(n) * int(min(N, n // 3)) * sv for n, N in zip(ns, Ns))
        return dict(bytes=sum(p[0] for p in parts) + out, flops=sum(p[1] for p in parts))
    n, N = case["n"], case["N"]
    if case["path"] == "modes" or case["path"] == "dmd":
        sp, m, r = EPL[case["phi"]], N - 1, case["r"]
        by, fl = float(n) * (m * sv + r * sp), 2.0 * n * m * r
        if case["path"] == "dmd":
            b2, f2 = _stream_work(n, N, sv, sx, "push")
            by, fl = by + b2, fl + f2
        return dict(bytes=by, flops=fl)
    by, fl = _stream_work(n, N, sv, sx, case["path"])
    return dict(bytes=by + 2.0 * n * N * sv, flops=fl)


# ---- the same in plain 64-bit torch and numpy ----------------------------------

def _qr(X):
    """X = R^T V (snapshots and Arnoldi vectors as rows), R with a positive
    diagonal: Cholesky QR, three times, in float64."""
    V = X.to(torch.float64)
    N = V.shape[0]
    R = torch.eye(N, dtype=torch.float64, device=V.device)
    for _ in range(3):
        L = torch.linalg.cholesky(V @ V.T)
        V = torch.linalg.inv(L) @ V
        R = L.T @ R
    return V, R.cpu().numpy()


def _h_beta(R):
    """H_bar and beta as the state call lays them out (one zero row, and one zero column of beta)."""
    N = R.shape[0]
    H = np.zeros((N + 1, N - 1))
    H[:N] = np.triu(R[:, 1:] @ np.linalg.inv(R[:N - 1, :N - 1]), -1)
    B = np.zeros((N + 1, N + 1))
    B[:N, :N] = np.triu(R)
    return H, B


def exact(case, seed):
    X = _inputs(case, seed)
    if case["path"] == "batch":
        H, B, V = [], [], []
        for x in X:
            v, R = _qr(x)
            h, b = _h_beta(R)
            H.append(h.ravel())
            B.append(b.ravel())
            V.append(v.reshape(-1))
        N = np.array([x.shape[0] for x in X], dtype=np.int32)
        return [N, np.zeros_like(N), np.concatenate(H), np.concatenate(B), torch.cat(V)]
    V, R = _qr(X)
    N = R.shape[0]
    H, B = _h_beta(R)
    if "r" not in case:
        return [N, N - 1, H, B, V]
    # eigenvectors of unit norm with the entry of largest modulus real positive,
    # ordered by the coefficients of the first snapshot
    m, r = N - 1, case["r"]
    Hm, hlast = H[:m, :m], H[m, m - 1]
    U = np.linalg.svd(B[:m, :m])[0][:, :r] if r < m else np.eye(m)
    lam, Z = np.linalg.eig(U.T @ Hm @ U)
    big = Z[np.argmax(np.abs(Z), axis=0), np.arange(r)]
    Z = Z * (np.conj(big) / np.abs(big)) / np.linalg.norm(Z, axis=0)
    c = np.linalg.solve(Z, (B[0, 0] * U[0]).astype(complex))
    keep = [i for i in range(r) if lam[i].imag >= 0]
    keep.sort(key=lambda i: -abs(c[i]))
    Y = U @ Z
    HY = Hm @ Y
    top = HY - U @ (U.T @ HY)
    err = np.sqrt(np.sum(np.abs(top) ** 2, axis=0) + np.abs(hlast * Y[m - 1]) ** 2)
    kind = np.array([1 if lam[i].imag > 0 else 0 for i in keep], dtype=np.int8)
    phi = None  # after a truncation a mode's sign goes by the signs of the singular vectors, which are free
    if r == m:
        cols = []
        for i in keep:
            cols.append(Y[:, i].real)
            if lam[i].imag > 0:
                cols.append(Y[:, i].imag)
        phi = torch.from_numpy(np.array(cols)).to(V.device) @ V[:m]
    return [lam[keep], kind, np.abs(c[keep]), err[keep], phi]
