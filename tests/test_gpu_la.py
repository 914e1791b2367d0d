"""GPU checks of the batched dense building blocks (GEMM, Householder QR,
Q application, pivoted Cholesky, triangular solve) against NumPy/LAPACK."""
import ctypes as C

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

nd = pytest.importorskip("paper_2607_00928_amd")
from paper_2607_00928_amd import _lib  # noqa: E402

lib = _lib.lib
DEV = torch.device("cuda", 0)
CT = {0: (np.complex128, torch.complex128), 1: (np.complex64, torch.complex64)}
CT[2] = CT[1]   # complex64 with the products on the bf16 split
TOL = {0: 1e-12, 1: 2e-5, 2: 2e-5}
QB = 256   # reflectors per compact-WY block of the QR factors (T layout)


def crandn(rng, *shape):
    return (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)) / np.sqrt(2)


def to_dev(Mat, prec, cols=None):
    """column-major device copy (ld = rows)"""
    npt, tt = CT[prec]
    return torch.from_numpy(np.ascontiguousarray(Mat.T.astype(npt))).to(DEV)


def from_dev(t, m, n):
    return t.cpu().numpy().reshape(n, m).T


def i32(a):
    a = np.ascontiguousarray(a, dtype=np.int32)
    return a, a.ctypes.data_as(C.POINTER(C.c_int32))


def i64(a):
    a = np.ascontiguousarray(a, dtype=np.int64)
    return a, a.ctypes.data_as(C.POINTER(C.c_int64))


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("opa,opb", [(0, 0), (1, 0), (0, 1), (1, 1)])
def test_gemm_batched_ragged(prec, opa, opb):
    rng = np.random.default_rng(10 * prec + 2 * opa + opb)
    shapes = [(1, 1, 1), (70, 33, 19), (64, 64, 64), (130, 5, 200), (3, 150, 17), (65, 129, 0)]
    if prec == 2:   # a k = 1 product keeps its launch on the FP32 instructions
        shapes[0] = (1, 1, 2)
    mats, keep = [], []
    mnk, ld, ptr = [], [], []
    alpha = 0.7 - 0.3j
    for (m, n, k) in shapes:
        A = crandn(rng, *((m, k) if opa == 0 else (k, m)))
        B = crandn(rng, *((k, n) if opb == 0 else (n, k)))
        Cm = crandn(rng, m, n)
        ta, tb, tc = to_dev(A, prec), to_dev(B, prec), to_dev(Cm, prec)
        keep += [ta, tb, tc]
        mats.append((A, B, Cm, tc))
        mnk += [m, n, k]
        ld += [max(A.shape[0], 1), max(B.shape[0], 1), max(m, 1)]
        ptr += [ta.data_ptr(), tb.data_ptr(), tc.data_ptr()]
    a1, p1 = i32(mnk)
    a2, p2 = i32(ld)
    a3, p3 = i64(ptr)
    st = lib.nudft2_test_gemm(prec, opa, opb, len(shapes), p1, p2, p3, alpha.real, alpha.imag, 1.0)
    assert st == 0, lib.nudft2_last_error()
    for (m, n, k), (A, B, Cm, tc) in zip(shapes, mats):
        oA = A if opa == 0 else A.conj().T
        oB = B if opb == 0 else B.conj().T
        ref = alpha * (oA @ oB) + Cm
        got = from_dev(tc, m, n)
        scale = max(1.0, np.abs(ref).max())
        assert np.abs(got - ref).max() < TOL[prec] * scale * max(1, k) ** 0.5 * 10, (m, n, k)


@pytest.mark.parametrize("prec", [1, 2])
@pytest.mark.parametrize("opa,opb", [(0, 0), (1, 0), (0, 1), (1, 1)])
def test_gemm_fp32_entrywise_error(prec, opa, opb):
    """Each entry of a complex64 product against the FP64 product of the same
    (rounded) operands, relative to (|op(A)| |op(B)|)_ij: FP32 rounding of k
    products and sums stays within a few times 2^-24 sqrt(k) of it.  The bf16
    split (prec 2) must meet the same bound as the FP32 instructions: a
    dropped split product (a0 b1, a1 b0: 2^-8; a0 b2, a1 b1, a2 b0: 2^-16)
    or a lost plane would exceed it by orders of magnitude.  Odd k (the split
    kernel reads k in pairs), k = 2, tiles past the matrix edge, long k with
    the library's split choice, alpha complex, beta = 0.5."""
    rng = np.random.default_rng(300 + 4 * prec + 2 * opa + opb)
    shapes = [(70, 33, 19), (2, 3, 2), (129, 65, 33), (64, 64, 64), (200, 150, 999),
              (17, 300, 3001), (1, 130, 77)]
    alpha, beta = 0.8 - 0.5j, 0.5
    mats, keep, mnk, ld, ptr = [], [], [], [], []
    for (m, n, k) in shapes:
        A = crandn(rng, *((m, k) if opa == 0 else (k, m))).astype(np.complex64)
        B = crandn(rng, *((k, n) if opb == 0 else (n, k))).astype(np.complex64)
        Cm = crandn(rng, m, n).astype(np.complex64)
        ts = [to_dev(X, prec) for X in (A, B, Cm)]
        keep += ts
        mats.append((A, B, Cm, ts[2]))
        mnk += [m, n, k]
        ld += [A.shape[0], B.shape[0], m]
        ptr += [t.data_ptr() for t in ts]
    a1, p1 = i32(mnk)
    a2, p2 = i32(ld)
    a3, p3 = i64(ptr)
    st = lib.nudft2_test_gemm(prec, opa, opb, len(shapes), p1, p2, p3, alpha.real, alpha.imag, beta)
    assert st == 0, lib.nudft2_last_error()
    for (m, n, k), (A, B, Cm, tc) in zip(shapes, mats):
        oA = (A if opa == 0 else A.conj().T).astype(np.complex128)
        oB = (B if opb == 0 else B.conj().T).astype(np.complex128)
        ref = alpha * (oA @ oB) + beta * Cm.astype(np.complex128)
        scale = abs(alpha) * (np.abs(oA) @ np.abs(oB)) + beta * np.abs(Cm)
        err = (np.abs(from_dev(tc, m, n) - ref) / scale).max()
        assert err < 8 * 2.0 ** -24 * np.sqrt(k), (m, n, k, err)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("opa", [0, 1])
@pytest.mark.parametrize("beta", [0.0, 1.0])
def test_gemm_skinny(prec, opa, beta):
    """Products with at most 8 columns (the memory-bound path), including
    long k (split over workgroups) and a single row."""
    rng = np.random.default_rng(20 + 2 * prec + opa)
    shapes = [(1, 1, 1), (300, 1, 700), (5000, 3, 64), (17, 8, 3000), (64, 2, 40000), (1, 5, 9),
              (257, 7, 0)]
    mats, keep = [], []
    mnk, ld, ptr = [], [], []
    alpha = -0.4 + 1.1j
    for (m, n, k) in shapes:
        A = crandn(rng, *((m, k) if opa == 0 else (k, m)))
        B = crandn(rng, k, n)
        Cm = crandn(rng, m, n)
        ta, tb, tc = to_dev(A, prec), to_dev(B, prec), to_dev(Cm, prec)
        keep += [ta, tb, tc]
        mats.append((A, B, Cm, tc))
        mnk += [m, n, k]
        ld += [max(A.shape[0], 1), max(B.shape[0], 1), max(m, 1)]
        ptr += [ta.data_ptr(), tb.data_ptr(), tc.data_ptr()]
    a1, p1 = i32(mnk)
    a2, p2 = i32(ld)
    a3, p3 = i64(ptr)
    st = lib.nudft2_test_gemm(prec, opa, 0, len(shapes), p1, p2, p3, alpha.real, alpha.imag, beta)
    assert st == 0, lib.nudft2_last_error()
    for (m, n, k), (A, B, Cm, tc) in zip(shapes, mats):
        oA = A if opa == 0 else A.conj().T
        ref = alpha * (oA @ B) + beta * Cm
        got = from_dev(tc, m, n)
        scale = max(1.0, np.abs(ref).max())
        assert np.abs(got - ref).max() < TOL[prec] * scale * max(1, k) ** 0.5 * 10, (m, n, k)


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("opa", [0, 1])
@pytest.mark.parametrize("shapes", [
    # tiles of 16 rows, chunks of 16 k and rounds of 256 at and past their ends
    [(1, 9, 1), (16, 16, 16), (17, 16, 15), (33, 9, 65), (256, 16, 256), (100, 13, 1023), (5, 1, 300),
     (48, 16, 257), (40, 12, 0)],
    # k ranges summed through scratch (maxk >= 1024), a product with fewer of them
    [(256, 16, 9001), (31, 10, 1024), (16, 12, 300)],
    # 32 rows a workgroup
    [(65521, 9, 200)],
    # op C with few rows: blocks of 16 columns, also with k ranges
    [(32, 96, 700), (7, 17, 33), (1, 128, 300), (20, 33, 2), (16, 40, 0), (31, 5, 90)],
    [(32, 65, 2500), (9, 128, 1100)],
])
def test_gemm_up_to_16_columns(prec, opa, shapes):
    """Entrywise against the FP64 product (FP64: of the oracle's rounding),
    relative to |op(A)| |B|: a few roundings times sqrt(k); leading dimensions
    that leave columns aligned to single elements only."""
    rng = np.random.default_rng(500 + 4 * prec + opa)
    ct = np.complex64 if prec else np.complex128
    alpha, beta = 0.8 - 0.5j, 0.5
    mats, keep, mnk, ld, ptr = [], [], [], [], []
    for (m, n, k) in shapes:
        A = crandn(rng, *((m, k) if opa == 0 else (k, m))).astype(ct)
        B, Cm = crandn(rng, k, n).astype(ct), crandn(rng, m, n).astype(ct)
        pads = [np.concatenate([X, np.zeros((1, X.shape[1]), ct)]) for X in (A, B, Cm)]
        ts = [to_dev(X, prec) if X.size else torch.zeros(1, dtype=torch.complex128, device=DEV)
              for X in pads]
        keep += ts
        mats.append((A, B, Cm, ts[2]))
        mnk += [m, n, k]
        ld += [X.shape[0] for X in pads]
        ptr += [t.data_ptr() for t in ts]
    a1, p1 = i32(mnk)
    a2, p2 = i32(ld)
    a3, p3 = i64(ptr)
    st = lib.nudft2_test_gemm(prec, opa, 0, len(shapes), p1, p2, p3, alpha.real, alpha.imag, beta)
    assert st == 0, lib.nudft2_last_error()
    eps = 2.0 ** -24 if prec else 2.0 ** -53
    for (m, n, k), (A, B, Cm, tc) in zip(shapes, mats):
        oA = (A if opa == 0 else A.conj().T).astype(np.complex128)
        ref = alpha * (oA @ B.astype(np.complex128)) + beta * Cm.astype(np.complex128)
        scale = abs(alpha) * (np.abs(oA) @ np.abs(B)) + beta * np.abs(Cm)
        err = (np.abs(from_dev(tc, m + 1, n)[:m] - ref) / scale).max()
        assert err < 8 * eps * np.sqrt(max(k, 4)), (m, n, k, err)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("beta", [0.0, 0.5])
def test_gemm_skinny_ch_long_k_few_rows(prec, beta):
    """A^H B with at most 8 columns, a long k and few rows of C (the sweep's
    V^H c against a block of reflectors): a workgroup per row of C, no k
    split.  Ragged k (not a multiple of the 256-thread stride), one and eight
    columns, a row count that is not a multiple of anything."""
    rng = np.random.default_rng(400 + 2 * prec + int(beta > 0))
    shapes = [(256, 1, 11000), (200, 3, 9001), (5, 8, 4097), (77, 1, 2049)]
    alpha = 0.3 + 0.9j
    mats, keep, mnk, ld, ptr = [], [], [], [], []
    for (m, n, k) in shapes:
        A = crandn(rng, k, m)
        B = crandn(rng, k, n)
        Cm = crandn(rng, m, n)
        ts = [to_dev(X, prec) for X in (A, B, Cm)]
        keep += ts
        mats.append((A, B, Cm, ts[2]))
        mnk += [m, n, k]
        ld += [k, k, m]
        ptr += [t.data_ptr() for t in ts]
    a1, p1 = i32(mnk)
    a2, p2 = i32(ld)
    a3, p3 = i64(ptr)
    st = lib.nudft2_test_gemm(prec, 1, 0, len(shapes), p1, p2, p3, alpha.real, alpha.imag, beta)
    assert st == 0, lib.nudft2_last_error()
    for (m, n, k), (A, B, Cm, tc) in zip(shapes, mats):
        ref = alpha * (A.conj().T @ B) + beta * Cm
        got = from_dev(tc, m, n)
        scale = max(1.0, np.abs(ref).max())
        assert np.abs(got - ref).max() < TOL[prec] * scale * k ** 0.5 * 10, (m, n, k)


@pytest.mark.parametrize("prec", [0, 1, 2])
def test_geqrf_ormqr(prec):
    rng = np.random.default_rng(3 + prec)
    # around the 256-column blocks and their 128-column halves: a block with
    # one reflector in its right half, exactly one block, a last block of one
    # half, several blocks with partial halves, wide problems
    shapes = [(100, 37), (37, 100), (64, 64), (5, 3), (1030, 546), (33, 1), (300, 97),
              (3000, 70), (257, 300), (700, 129), (400, 256), (130, 700), (2000, 600),
              (600, 384), (1000, 513)]
    keep = []
    mn, ld, ptr, data = [], [], [], []
    for (m, n) in shapes:
        A = crandn(rng, m, n)
        k = min(m, n)
        nob = (k + QB - 1) // QB
        tsize = QB * QB * (nob - 1) + (k - QB * (nob - 1)) ** 2
        tA = to_dev(A, prec)
        # R starts as garbage: the factorization must write all of it
        tR = torch.full((n, k), 7.0 - 3.0j, dtype=CT[prec][1], device=DEV)   # k x n col-major
        tT = torch.full((tsize,), 5.0 + 1.0j, dtype=CT[prec][1], device=DEV)
        keep += [tA, tR, tT]
        data.append((A, tA, tR, tT))
        mn += [m, n]
        ld += [m, k]
        ptr += [tA.data_ptr(), tR.data_ptr(), tT.data_ptr()]
    a1, p1 = i32(mn)
    a2, p2 = i32(ld)
    a3, p3 = i64(ptr)
    st = lib.nudft2_test_geqrf(prec, len(shapes), p1, p2, p3)
    assert st == 0, lib.nudft2_last_error()
    # form Q (m x m) by applying Q to the identity, check Q R = A, Q unitary
    dims, ld2, ptr2, Qs = [], [], [], []
    for (m, n), (A, tA, tR, tT) in zip(shapes, data):
        tQ = to_dev(np.eye(m), prec)
        keep.append(tQ)
        Qs.append(tQ)
        dims += [m, min(m, n), m]
        ld2 += [m, m]
        ptr2 += [tA.data_ptr(), tT.data_ptr(), tQ.data_ptr()]
    b1, q1 = i32(dims)
    b2, q2 = i32(ld2)
    b3, q3 = i64(ptr2)
    st = lib.nudft2_test_ormqr(prec, 0, len(shapes), q1, q2, q3)
    assert st == 0, lib.nudft2_last_error()
    # explicit Q formation from the identity (trans = 2 skips the columns each
    # block leaves unchanged) must give the same Q
    ptr2i, Qi = [], []
    for (m, n), (A, tA, tR, tT) in zip(shapes, data):
        tQi = to_dev(np.eye(m), prec)
        keep.append(tQi)
        Qi.append(tQi)
        ptr2i += [tA.data_ptr(), tT.data_ptr(), tQi.data_ptr()]
    b4, q4 = i64(ptr2i)
    assert lib.nudft2_test_ormqr(prec, 2, len(shapes), q1, q2, q4) == 0, lib.nudft2_last_error()
    for (m, n), tQ, tQi in zip(shapes, Qs, Qi):
        d = np.abs(from_dev(tQi, m, m) - from_dev(tQ, m, m)).max()
        assert d < 10 * TOL[prec] * np.sqrt(m), (m, n, d)
    for (m, n), (A, tA, tR, tT), tQ in zip(shapes, data, Qs):
        k = min(m, n)
        Q = from_dev(tQ, m, m)
        R = from_dev(tR, k, n)
        assert np.abs(np.tril(R, -1)).max() == 0
        # A returns the explicit unit lower-trapezoidal reflectors
        V = from_dev(tA, m, n)[:, :k]
        assert np.abs(np.triu(V, 1)).max() == 0 and np.all(np.diag(V) == 1), (m, n)
        err = np.abs(Q[:, :k] @ R - A).max() / np.abs(A).max()
        orth = np.abs(Q.conj().T @ Q - np.eye(m)).max()
        print(f"qr {m}x{n} prec{prec}: recon {err:.1e} orth {orth:.1e}")
        assert err < 50 * TOL[prec] * np.sqrt(m)
        assert orth < 50 * TOL[prec] * np.sqrt(m)
        # |R| diagonal equals LAPACK's up to phases
        Rl = np.linalg.qr(A.astype(np.complex128), mode="r")
        assert np.allclose(np.abs(np.diag(R)), np.abs(np.diag(Rl)), rtol=1e-3 if prec else 1e-9)
    # Q^H (Q C) = C via the trans path
    dims3, ld3, ptr3, Cs = [], [], [], []
    for (m, n), (A, tA, tR, tT) in zip(shapes, data):
        Cm = crandn(rng, m, 7)
        tC = to_dev(Cm, prec)
        keep.append(tC)
        Cs.append((Cm, tC))
        dims3 += [m, min(m, n), 7]
        ld3 += [m, m]
        ptr3 += [tA.data_ptr(), tT.data_ptr(), tC.data_ptr()]
    c1, r1 = i32(dims3)
    c2, r2 = i32(ld3)
    c3, r3 = i64(ptr3)
    assert lib.nudft2_test_ormqr(prec, 0, len(shapes), r1, r2, r3) == 0
    assert lib.nudft2_test_ormqr(prec, 1, len(shapes), r1, r2, r3) == 0
    for (m, n), (Cm, tC) in zip(shapes, Cs):
        got = from_dev(tC, m, 7)
        assert np.abs(got - Cm).max() < 100 * TOL[prec] * np.sqrt(m)


def test_pchol_trace_rule():
    rng = np.random.default_rng(7)
    # up to 1100 rows: five cooperating workgroups per Gram, several panels
    sizes = [(40, 40), (300, 120), (473, 473), (17, 5), (1100, 70)]
    keep, data = [], []
    w, rmax, ptr = [], [], []
    tol2 = 1e-8
    for (n, rm) in sizes:
        # Hermitian PSD with geometrically decaying spectrum
        Qm, _ = np.linalg.qr(crandn(rng, n, n))
        lam = 10.0 ** (-12 * np.arange(n) / n)
        K = (Qm * lam) @ Qm.conj().T
        K = (K + K.conj().T) / 2
        tK = to_dev(K, 0)
        tL = torch.zeros((rm, n), dtype=torch.complex128, device=DEV)
        keep += [tK, tL]
        data.append((K, tK, tL, n, rm))
        w.append(n)
        rmax.append(rm)
        ptr += [tK.data_ptr(), tL.data_ptr()]
    a1, p1 = i32(w)
    a2, p2 = i32(rmax)
    a3, p3 = i64(ptr)
    ranks = np.zeros(len(sizes), np.int32)
    piv = np.zeros(sum(rmax), np.int32)
    st = lib.nudft2_test_pchol(len(sizes), p1, p2, p3, tol2,
                               ranks.ctypes.data_as(C.POINTER(C.c_int32)),
                               piv.ctypes.data_as(C.POINTER(C.c_int32)))
    assert st == 0, lib.nudft2_last_error()
    off = 0
    for (K, tK, tL, n, rm), r in zip(data, ranks):
        L = from_dev(tL, n, rm)[:, :r]
        p = piv[off:off + r]
        off += rm
        S = K - L @ L.conj().T
        tr = np.trace(K).real
        print(f"pchol n={n}: rank {r}, residual trace {np.trace(S).real / tr:.2e}")
        assert len(set(p.tolist())) == r
        if r < rm:
            assert np.trace(S).real <= tol2 * tr * (1 + 1e-6) + 1e-13 * tr
            assert np.trace(S).real >= -1e-10 * tr
        # L restricted to the pivot rows is lower triangular in pivot order
        Lp = L[p, :]
        assert np.abs(np.triu(Lp, 1)).max() < 1e-12 * np.abs(Lp).max()
        # the rank is not far from the trace-optimal rank of the spectrum
        lam = np.sort(np.linalg.eigvalsh(K))[::-1]
        tail = np.concatenate([np.cumsum(lam[::-1])[::-1], [0.0]])
        ropt = int(np.nonzero(tail <= tol2 * tr)[0][0])
        if r < rm:
            assert r <= 2 * ropt + 8


@pytest.mark.parametrize("sizes", [
    # one workgroup per Gram: waves, panels of 32 and rmax at and around their
    # ends, ranks of zero, one row per thread (<= 1024) and two
    [(1, 1, 1), (2, 2, 2), (31, 31, 31), (32, 32, 32), (33, 33, 33), (64, 64, 64), (65, 65, 40),
     (100, 32, 60), (100, 33, 60), (100, 64, 64), (0, 0, 0), (90, 0, 40), (50, 50, 0)],
    [(1024, 96, 70), (200, 200, 65), (7, 7, 7)],
    [(1025, 64, 64), (1023, 97, 96), (1536, 40, 33), (5, 5, 3)],
    # panels of 64 (Grams x order >= 65536)
    [(1030, 129, 128), (1030, 140, 65), (64, 64, 64)] + [(3, 2, 2)] * 61,
    # a column per launch over several workgroups
    [(1537, 140, 131), (64, 64, 64), (300, 300, 128)],
])
def test_pchol_greedy(sizes):
    # K of exact rank r with well separated pivots: the greedy order is the
    # oracle's, and L agrees to FP64 rounding (about w kappa eps, kappa <= 1e4)
    rng = np.random.default_rng(23)
    keep, data, ptr = [], [], []
    tol2 = 1e-11
    for (n, rm, rk) in sizes:
        F = crandn(rng, n, rk) * (2.0 ** (-10.0 * np.arange(n) / max(n, 1)))[rng.permutation(n), None] \
            if n and rk else np.zeros((n, rk))
        K = F @ F.conj().T
        tK = to_dev(K, 0) if n else torch.zeros(1, dtype=torch.complex128, device=DEV)
        tL = torch.zeros((max(rm, 1), max(n, 1)), dtype=torch.complex128, device=DEV)
        keep += [tK, tL]
        data.append((K, tL, n, rm, rk))
        ptr += [tK.data_ptr(), tL.data_ptr()]
    rmax = [s[1] for s in sizes]
    a1, p1 = i32([s[0] for s in sizes])
    a2, p2 = i32(rmax)
    a3, p3 = i64(ptr)
    ranks = np.zeros(len(sizes), np.int32)
    piv = np.zeros(sum(rmax), np.int32)
    st = lib.nudft2_test_pchol(len(sizes), p1, p2, p3, tol2,
                               ranks.ctypes.data_as(C.POINTER(C.c_int32)),
                               piv.ctypes.data_as(C.POINTER(C.c_int32)))
    assert st == 0, lib.nudft2_last_error()
    off = 0
    for (K, tL, n, rm, rk), r in zip(data, ranks):
        S, want = K.copy(), []
        Lw = np.zeros((n, min(rm, rk)), complex)
        for k in range(min(rm, rk)):
            p = int(np.argmax(np.where(np.isin(np.arange(n), want), -1.0, S.diagonal().real)))
            Lw[:, k] = S[:, p] / np.sqrt(S[p, p].real)
            S = S - np.outer(Lw[:, k], Lw[:, k].conj())
            want.append(p)
        assert r == min(rm, rk), (n, rm, rk, r)
        assert piv[off:off + r].tolist() == want, (n, rm, rk)
        off += rm
        if r:
            L = tL.cpu().numpy().T[:n, :r]
            assert np.abs(L - Lw).max() <= 1e-9 * np.abs(Lw).max(), (n, rm, rk)


@pytest.mark.parametrize("order,count", [(1344, 12), (1345, 11), (1345, 12)])
def test_pchol_greedy_in_long_lists(order, count):
    # both sides of the line between one workgroup and a launch per column, by
    # the order and the number of Grams above it
    test_pchol_greedy([(order, 40, 36)] * count + [(102, 40, 20)] * 3)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("nb", [1, 43, 400])
def test_qr_descriptor_lists_outgrow_the_pool(prec, nb):
    """The hooks' descriptor pool starts at 4 KiB: lists too long for kernel
    arguments move it to larger segments again and again during one batch (and
    FP64's error flag with it), behind launches that read the old ones."""
    rng = np.random.default_rng(31 + nb)
    m, n = 150, 136
    A = crandn(rng, nb, m, n)
    tA = torch.from_numpy(np.ascontiguousarray(A.transpose(0, 2, 1)).astype(CT[prec][0])).to(DEV)
    A = tA.cpu().numpy().transpose(0, 2, 1).astype(np.complex128)
    tR = torch.zeros((nb, n, n), dtype=CT[prec][1], device=DEV)
    tT = torch.zeros((nb, n * n), dtype=CT[prec][1], device=DEV)
    tQ = torch.eye(m, dtype=CT[prec][1], device=DEV).repeat(nb, 1, 1)
    a1, p1 = i32([m, n] * nb)
    a2, p2 = i32([m, n] * nb)
    a3, p3 = i64(sum([[t[b].data_ptr() for t in (tA, tR, tT)] for b in range(nb)], []))
    assert lib.nudft2_test_geqrf(prec, nb, p1, p2, p3) == 0, lib.nudft2_last_error()
    b1, q1 = i32([m, n, m] * nb)
    b2, q2 = i32([m, m] * nb)
    b3, q3 = i64(sum([[t[b].data_ptr() for t in (tA, tT, tQ)] for b in range(nb)], []))
    assert lib.nudft2_test_ormqr(prec, 0, nb, q1, q2, q3) == 0, lib.nudft2_last_error()
    Q = tQ.cpu().numpy().transpose(0, 2, 1).astype(np.complex128)
    R = tR.cpu().numpy().transpose(0, 2, 1).astype(np.complex128)
    err = np.abs(Q[:, :, :n] @ R - A).max(axis=(1, 2)) / np.abs(A).max(axis=(1, 2))
    assert err.max() < 50 * TOL[prec] * np.sqrt(m)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("ct", [0, 1])
def test_trsv(prec, ct):
    rng = np.random.default_rng(11 + ct)
    # one block (<= 128) with the lane-slot boundaries 64 / 65 / 128, and blocked orders
    sizes = [(1, 1), (50, 3), (300, 2), (7, 1), (700, 2), (257, 1), (64, 1), (65, 2), (128, 1),
             (129, 3)]
    keep, data, dims, ld, ptr = [], [], [], [], []
    for (k, nr) in sizes:
        # well-conditioned triangle (a unit-scale random triangle is
        # exponentially ill-conditioned in k)
        R = np.triu(crandn(rng, k, k), 1) / np.sqrt(k) + (2 + np.abs(crandn(rng, k))) * np.eye(k)
        B = crandn(rng, k, nr)
        tR, tB = to_dev(R, prec), to_dev(B, prec)
        keep += [tR, tB]
        data.append((R, B, tB, k, nr))
        dims += [k, nr]
        ld += [k, k]
        ptr += [tR.data_ptr(), tB.data_ptr()]
    a1, p1 = i32(dims)
    a2, p2 = i32(ld)
    a3, p3 = i64(ptr)
    assert lib.nudft2_test_trsv(prec, len(sizes), p1, p2, p3, ct) == 0
    for R, B, tB, k, nr in data:
        X = from_dev(tB, k, nr)
        ref = np.linalg.solve(R.conj().T if ct else R, B)
        assert np.abs(X - ref).max() < 100 * TOL[prec] * max(1, np.abs(ref).max())


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("ct", [0, 1])
@pytest.mark.parametrize("nb,k,nr", [(1, 128, 33), (3, 65, 5), (40, 30, 41), (150, 20, 65)])
def test_trsv_right_hand_sides(prec, ct, nb, k, nr):
    # 4 to 32 right-hand sides a workgroup, by the list's length; uneven lists.
    # A wave's solution is backward stable: an error of k roundings, times the
    # condition (below 8 for this triangle)
    rng = np.random.default_rng(50 + nb)
    ns = [max(1, nr - i % 7) for i in range(nb)]
    R = np.triu(crandn(rng, k, k), 1) / k + (2 + np.abs(crandn(rng, k))) * np.eye(k)
    Bs = [crandn(rng, k, n) for n in ns]
    tR = to_dev(R, prec)
    tBs = [to_dev(B, prec) for B in Bs]
    a1, p1 = i32(sum([[k, n] for n in ns], []))
    a2, p2 = i32([k, k] * nb)
    a3, p3 = i64(sum([[tR.data_ptr(), t.data_ptr()] for t in tBs], []))
    assert lib.nudft2_test_trsv(prec, nb, p1, p2, p3, ct) == 0, lib.nudft2_last_error()
    Rr = from_dev(tR, k, k).astype(np.complex128)
    eps = 2.0 ** -24 if prec else 2.0 ** -53
    for B, t, n in zip(Bs, tBs, ns):
        B = B.astype(CT[prec][0]).astype(np.complex128)
        ref = np.linalg.solve(Rr.conj().T if ct else Rr, B)
        assert np.abs(from_dev(t, k, n) - ref).max() < 8 * k * eps * np.abs(ref).max()


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("opa,opb", [(0, 0), (1, 0), (0, 1), (1, 1)])
def test_gemm_large_batch(prec, opa, opb):
    """A batch of 24 products of a few hundred rows and columns (many tiles,
    no k splitting): ragged m, n, k (not multiples of the tile or k stage), a
    tiny product and an empty one in the same batch, beta = 1."""
    rng = np.random.default_rng(40 + 10 * prec + 2 * opa + opb)
    shapes = [(600 - 7 * i, 520 + 5 * i, 200 + 13 * i) for i in range(24)]
    shapes += [(3, 2, 5), (0, 4, 4), (130, 129, 1 if prec != 2 else 3)]
    mats, keep = [], []
    mnk, ld, ptr = [], [], []
    alpha = 0.9 + 0.2j
    for (m, n, k) in shapes:
        A = crandn(rng, *((m, k) if opa == 0 else (k, m)))
        B = crandn(rng, *((k, n) if opb == 0 else (n, k)))
        Cm = crandn(rng, m, n)
        ta, tb, tc = to_dev(A, prec), to_dev(B, prec), to_dev(Cm, prec)
        keep += [ta, tb, tc]
        mats.append((A, B, Cm, tc))
        mnk += [m, n, k]
        ld += [max(A.shape[0], 1), max(B.shape[0], 1), max(m, 1)]
        ptr += [ta.data_ptr(), tb.data_ptr(), tc.data_ptr()]
    a1, p1 = i32(mnk)
    a2, p2 = i32(ld)
    a3, p3 = i64(ptr)
    st = lib.nudft2_test_gemm(prec, opa, opb, len(shapes), p1, p2, p3, alpha.real, alpha.imag, 1.0)
    assert st == 0, lib.nudft2_last_error()
    for (m, n, k), (A, B, Cm, tc) in zip(shapes, mats):
        if m == 0:
            continue
        oA = A if opa == 0 else A.conj().T
        oB = B if opb == 0 else B.conj().T
        ref = alpha * (oA @ oB) + Cm
        got = from_dev(tc, m, n)
        scale = max(1.0, np.abs(ref).max())
        assert np.abs(got - ref).max() < TOL[prec] * scale * max(1, k) ** 0.5 * 10, (m, n, k)


@pytest.mark.parametrize("opa,opb", [(0, 0), (1, 0), (0, 1), (1, 1)])
def test_gemm_forced_unsplit(opa, opb):
    """The tile kernel forced unsplit through the measurement hook: ragged m,
    n, k around the tile and k-stage sizes, a one-row and an empty product in
    the same batch, alpha complex, beta = 1."""
    rng = np.random.default_rng(60 + 2 * opa + opb)
    shapes = [(1100, 1030, 130), (129, 300, 17), (256, 128, 16), (1, 200, 33), (0, 5, 5),
              (385, 511, 1)]
    mats, keep = [], []
    mnk, ld, ptr = [], [], []
    alpha = 0.6 - 0.8j
    for (m, n, k) in shapes:
        A = crandn(rng, *((m, k) if opa == 0 else (k, m)))
        B = crandn(rng, *((k, n) if opb == 0 else (n, k)))
        Cm = crandn(rng, m, n)
        ta, tb, tc = to_dev(A, 1), to_dev(B, 1), to_dev(Cm, 1)
        keep += [ta, tb, tc]
        mats.append((A, B, Cm, tc))
        mnk += [m, n, k]
        ld += [max(A.shape[0], 1), max(B.shape[0], 1), max(m, 1)]
        ptr += [ta.data_ptr(), tb.data_ptr(), tc.data_ptr()]
    a1, p1 = i32(mnk)
    a2, p2 = i32(ld)
    a3, p3 = i64(ptr)
    ms = C.c_float(0)
    st = lib.nudft2_test_gemm_cfg(1, opa, opb, len(shapes), p1, p2, p3, alpha.real, alpha.imag,
                                  1.0, -1, C.byref(ms))
    assert st == 0, lib.nudft2_last_error()
    for (m, n, k), (A, B, Cm, tc) in zip(shapes, mats):
        if m == 0:
            continue
        oA = A if opa == 0 else A.conj().T
        oB = B if opb == 0 else B.conj().T
        ref = alpha * (oA @ oB) + Cm
        got = from_dev(tc, m, n)
        scale = max(1.0, np.abs(ref).max())
        assert np.abs(got - ref).max() < TOL[1] * scale * max(1, k) ** 0.5 * 10, (m, n, k)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("beta", [0.0, 1.0, -0.5])
def test_gemm_small_output_long_k(prec, beta):
    """A^H B with at most 32 x 32 outputs and a long k (the small-output
    path): Grams whose two operands are one matrix (same pointer), cross
    products, outputs that are not multiples of 16, k not a multiple of the
    per-workgroup slice, and an empty k in the same batch.  Bound: a
    forward error of 8 u sqrt(k) |a_i| |b_j| per entry."""
    rng = np.random.default_rng(80 + 3 * prec + int(2 * beta))
    npt, _ = CT[prec]
    u = np.finfo(npt).eps / 2
    # (m, n, k, same operand)
    shapes = [(16, 16, 100003, True), (15, 15, 50000, True), (20, 31, 9000, False),
              (32, 32, 8193, False), (5, 12, 20000, False), (30, 9, 12000, False),
              (16, 16, 0, False), (27, 27, 16500, True)]
    mats, keep = [], []
    mnk, ld, ptr = [], [], []
    alpha = 0.8 - 0.45j
    for (m, n, k, same) in shapes:
        A = crandn(rng, k, m)
        B = A if same else crandn(rng, k, n)
        Cm = crandn(rng, m, n)
        ta, tc = to_dev(A, prec), to_dev(Cm, prec)
        tb = ta if same else to_dev(B, prec)
        keep += [ta, tb, tc]
        mats.append((A, B, Cm, tc))
        mnk += [m, n, k]
        ld += [max(k, 1), max(k, 1), m]
        ptr += [ta.data_ptr(), tb.data_ptr(), tc.data_ptr()]
    a1, p1 = i32(mnk)
    a2, p2 = i32(ld)
    a3, p3 = i64(ptr)
    st = lib.nudft2_test_gemm(prec, 1, 0, len(shapes), p1, p2, p3, alpha.real, alpha.imag, beta)
    assert st == 0, lib.nudft2_last_error()
    for (m, n, k, same), (A, B, Cm, tc) in zip(shapes, mats):
        Ac, Bc = A.astype(npt).astype(np.complex128), B.astype(npt).astype(np.complex128)
        Cc = Cm.astype(npt).astype(np.complex128)
        ref = alpha * (Ac.conj().T @ Bc) + beta * Cc
        got = from_dev(tc, m, n)
        na = np.linalg.norm(Ac, axis=0)
        nb_ = np.linalg.norm(Bc, axis=0)
        bound = 8 * u * max(1, k) ** 0.5 * np.outer(na, nb_) + 8 * u * np.abs(beta * Cc) + 1e-300
        assert np.all(np.abs(got - ref) <= bound + 4 * u * np.abs(ref)), (m, n, k, same)


@pytest.mark.parametrize("prec,shapes", [
    (0, [(40000, 40), (20000, 70), (9000, 33), (600, 20)]),
    (1, [(40000, 40), (20000, 70), (9000, 33), (600, 20)]),
    (2, [(40000, 40), (20000, 70), (9000, 33), (600, 20)]),
    # taller than one row slab per CU holds (65536 FP64 / 131072 FP32 rows):
    # twice the rows per workgroup
    (0, [(90000, 36), (3000, 40)]),
    (1, [(140000, 36), (3000, 40)]),
])
def test_geqrf_tall_panels(prec, shapes):
    """Householder QR of tall panels that need many cooperating workgroups per
    panel (40000 rows: 79 FP32 / 157 FP64 workgroups exchanging column sums
    every column; up to 140000 rows with twice the rows per workgroup),
    batched with shorter ones.  Checks Q [R; 0] = A through the Q application,
    R upper triangular, and |diag R| against LAPACK."""
    rng = np.random.default_rng(90 + prec)
    keep, data = [], []
    mn, ld, ptr = [], [], []
    for (m, n) in shapes:
        A = crandn(rng, m, n)
        k = min(m, n)
        nob = (k + QB - 1) // QB
        tsize = QB * QB * (nob - 1) + (k - QB * (nob - 1)) ** 2
        tA = to_dev(A, prec)
        tR = torch.full((n, k), 7.0 - 3.0j, dtype=CT[prec][1], device=DEV)
        tT = torch.full((tsize,), 5.0 + 1.0j, dtype=CT[prec][1], device=DEV)
        keep += [tA, tR, tT]
        data.append((A, tA, tR, tT))
        mn += [m, n]
        ld += [m, k]
        ptr += [tA.data_ptr(), tR.data_ptr(), tT.data_ptr()]
    a1, p1 = i32(mn)
    a2, p2 = i32(ld)
    a3, p3 = i64(ptr)
    st = lib.nudft2_test_geqrf(prec, len(shapes), p1, p2, p3)
    assert st == 0, lib.nudft2_last_error()
    # C = [R; 0], then C <- Q C must reproduce A
    dims, ld2, ptr2, Cs = [], [], [], []
    for (m, n), (A, tA, tR, tT) in zip(shapes, data):
        k = min(m, n)
        R = from_dev(tR, k, n)
        assert np.abs(np.tril(R, -1)).max() == 0
        Cm = np.zeros((m, n), dtype=np.complex128)
        Cm[:k] = R
        tC = to_dev(Cm, prec)
        keep.append(tC)
        Cs.append(tC)
        dims += [m, k, n]
        ld2 += [m, m]
        ptr2 += [tA.data_ptr(), tT.data_ptr(), tC.data_ptr()]
        Rl = np.linalg.qr(A, mode="r")
        assert np.allclose(np.abs(np.diag(R)), np.abs(np.diag(Rl)), rtol=1e-3 if prec else 1e-9)
    b1, q1 = i32(dims)
    b2, q2 = i32(ld2)
    b3, q3 = i64(ptr2)
    assert lib.nudft2_test_ormqr(prec, 0, len(shapes), q1, q2, q3) == 0
    for (m, n), (A, tA, tR, tT), tC in zip(shapes, data, Cs):
        err = np.abs(from_dev(tC, m, n) - A).max() / np.abs(A).max()
        print(f"tall qr {m}x{n} prec{prec}: recon {err:.1e}")
        assert err < 50 * TOL[prec] * np.sqrt(m)


@pytest.mark.parametrize("opa,opb", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("beta", [0.0, 1.0])
def test_gemm_split_k_few_tiles(opa, opb, beta):
    """FP32 products with a long k and few output tiles (the k loop split
    over workgroups, atomic accumulation into a pre-scaled C): ragged m, n,
    k around the tile, k stage and split sizes, beta 0 and 1."""
    rng = np.random.default_rng(100 + 4 * opa + 2 * opb + int(beta))
    shapes = [(300, 200, 5000), (129, 77, 3001), (128, 64, 700), (255, 130, 1029)]
    mats, keep = [], []
    mnk, ld, ptr = [], [], []
    alpha = -0.3 + 0.95j
    for (m, n, k) in shapes:
        A = crandn(rng, *((m, k) if opa == 0 else (k, m)))
        B = crandn(rng, *((k, n) if opb == 0 else (n, k)))
        Cm = crandn(rng, m, n)
        ta, tb, tc = to_dev(A, 1), to_dev(B, 1), to_dev(Cm, 1)
        keep += [ta, tb, tc]
        mats.append((A, B, Cm, tc))
        mnk += [m, n, k]
        ld += [A.shape[0], B.shape[0], m]
        ptr += [ta.data_ptr(), tb.data_ptr(), tc.data_ptr()]
    a1, p1 = i32(mnk)
    a2, p2 = i32(ld)
    a3, p3 = i64(ptr)
    st = lib.nudft2_test_gemm(1, opa, opb, len(shapes), p1, p2, p3, alpha.real, alpha.imag, beta)
    assert st == 0, lib.nudft2_last_error()
    for (m, n, k), (A, B, Cm, tc) in zip(shapes, mats):
        oA = A if opa == 0 else A.conj().T
        oB = B if opb == 0 else B.conj().T
        ref = alpha * (oA @ oB) + beta * Cm
        got = from_dev(tc, m, n)
        scale = max(1.0, np.abs(ref).max())
        assert np.abs(got - ref).max() < TOL[1] * scale * k ** 0.5 * 10, (m, n, k)


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("opa,opb", [(0, 0), (1, 0)])
def test_gemm_long_descriptor_list(prec, opa, opb):
    """100 ragged products in one launch: a descriptor list longer than fits in
    the kernel arguments (read from device memory), with a skinny and a
    small-output batch of the same length (beta = 1, alpha complex)."""
    rng = np.random.default_rng(120 + 10 * prec + 2 * opa + opb)
    batches = [[(int(rng.integers(1, 200)), int(rng.integers(9, 150)), int(rng.integers(0, 300)))
                for _ in range(100)],
               [(int(rng.integers(1, 400)), int(rng.integers(1, 9)), int(rng.integers(1, 500)))
                for _ in range(100)]]
    if opa == 1:
        batches.append([(int(rng.integers(9, 33)), int(rng.integers(9, 33)),
                         int(rng.integers(8200, 9000))) for _ in range(100)])
    alpha = 0.25 + 0.7j
    for shapes in batches:
        mats, keep = [], []
        mnk, ld, ptr = [], [], []
        for (m, n, k) in shapes:
            A = crandn(rng, *((m, k) if opa == 0 else (k, m)))
            B = crandn(rng, *((k, n) if opb == 0 else (n, k)))
            Cm = crandn(rng, m, n)
            ta, tb, tc = to_dev(A, prec), to_dev(B, prec), to_dev(Cm, prec)
            keep += [ta, tb, tc]
            mats.append((A, B, Cm, tc))
            mnk += [m, n, k]
            ld += [max(A.shape[0], 1), max(B.shape[0], 1), m]
            ptr += [ta.data_ptr(), tb.data_ptr(), tc.data_ptr()]
        a1, p1 = i32(mnk)
        a2, p2 = i32(ld)
        a3, p3 = i64(ptr)
        st = lib.nudft2_test_gemm(prec, opa, opb, len(shapes), p1, p2, p3, alpha.real, alpha.imag,
                                  1.0)
        assert st == 0, lib.nudft2_last_error()
        for (m, n, k), (A, B, Cm, tc) in zip(shapes, mats):
            oA = A if opa == 0 else A.conj().T
            oB = B if opb == 0 else B.conj().T
            ref = alpha * (oA @ oB) + Cm
            got = from_dev(tc, m, n)
            scale = max(1.0, np.abs(ref).max())
            assert np.abs(got - ref).max() < TOL[prec] * scale * max(1, k) ** 0.5 * 10, (m, n, k)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("beta", [0.0, 1.0])
def test_gemm_small_m_wide_long_k(prec, beta):
    """A^H B with m <= 32, 32 < n <= 128 and a long k (a panel's reflectors
    against the columns they update): each wave of the kernel owns 32 output
    columns.  Ragged m, n (one wave partly or not at all used), k not a
    multiple of the per-workgroup range, an empty k in the batch."""
    rng = np.random.default_rng(140 + 3 * prec + int(2 * beta))
    npt, _ = CT[prec]
    u = np.finfo(npt).eps / 2
    shapes = [(32, 96, 9000), (20, 128, 5000), (32, 33, 4100), (5, 100, 6000), (32, 64, 4096),
              (17, 40, 0), (1, 127, 4500)]
    mats, keep = [], []
    mnk, ld, ptr = [], [], []
    alpha = -0.6 + 0.55j
    for (m, n, k) in shapes:
        A = crandn(rng, k, m)
        B = crandn(rng, k, n)
        Cm = crandn(rng, m, n)
        ta, tb, tc = to_dev(A, prec), to_dev(B, prec), to_dev(Cm, prec)
        keep += [ta, tb, tc]
        mats.append((A, B, Cm, tc))
        mnk += [m, n, k]
        ld += [max(k, 1), max(k, 1), m]
        ptr += [ta.data_ptr(), tb.data_ptr(), tc.data_ptr()]
    a1, p1 = i32(mnk)
    a2, p2 = i32(ld)
    a3, p3 = i64(ptr)
    st = lib.nudft2_test_gemm(prec, 1, 0, len(shapes), p1, p2, p3, alpha.real, alpha.imag, beta)
    assert st == 0, lib.nudft2_last_error()
    for (m, n, k), (A, B, Cm, tc) in zip(shapes, mats):
        Ac, Bc = A.astype(npt).astype(np.complex128), B.astype(npt).astype(np.complex128)
        Cc = Cm.astype(npt).astype(np.complex128)
        ref = alpha * (Ac.conj().T @ Bc) + beta * Cc
        got = from_dev(tc, m, n)
        na = np.linalg.norm(Ac, axis=0)
        nb_ = np.linalg.norm(Bc, axis=0)
        bound = 8 * u * max(1, k) ** 0.5 * np.outer(na, nb_) + 8 * u * np.abs(beta * Cc) + 1e-300
        assert np.all(np.abs(got - ref) <= bound + 4 * u * np.abs(ref)), (m, n, k)


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("opa,opb", [(0, 0), (1, 0), (0, 1)])
def test_gemm_few_row_tiles(prec, opa, opb):
    """Products with at most 256 rows and many column tiles (the shape of the
    V^H C products of the blocked QR): ragged m around the 64-row tiles, n not
    a multiple of 64, one launch with the k loop split and one without,
    beta = 1, alpha complex."""
    rng = np.random.default_rng(160 + 10 * prec + 2 * opa + opb)
    alpha = 0.45 - 0.85j
    for shapes in ([(256, 2000, 700), (200, 1500, 300), (129, 2100, 64), (64, 4096, 33)],
                   [(250, 3000, 150)] * 6):
        mats, keep = [], []
        mnk, ld, ptr = [], [], []
        for (m, n, k) in shapes:
            A = crandn(rng, *((m, k) if opa == 0 else (k, m)))
            B = crandn(rng, *((k, n) if opb == 0 else (n, k)))
            Cm = crandn(rng, m, n)
            ta, tb, tc = to_dev(A, prec), to_dev(B, prec), to_dev(Cm, prec)
            keep += [ta, tb, tc]
            mats.append((A, B, Cm, tc))
            mnk += [m, n, k]
            ld += [A.shape[0], B.shape[0], m]
            ptr += [ta.data_ptr(), tb.data_ptr(), tc.data_ptr()]
        a1, p1 = i32(mnk)
        a2, p2 = i32(ld)
        a3, p3 = i64(ptr)
        st = lib.nudft2_test_gemm(prec, opa, opb, len(shapes), p1, p2, p3, alpha.real, alpha.imag,
                                  1.0)
        assert st == 0, lib.nudft2_last_error()
        for (m, n, k), (A, B, Cm, tc) in zip(shapes, mats):
            oA = A if opa == 0 else A.conj().T
            oB = B if opb == 0 else B.conj().T
            ref = alpha * (oA @ oB) + Cm
            got = from_dev(tc, m, n)
            scale = max(1.0, np.abs(ref).max())
            assert np.abs(got - ref).max() < TOL[prec] * scale * k ** 0.5 * 10, (m, n, k)


@pytest.mark.parametrize("pd,ps", [(0, 0), (1, 1), (1, 0), (0, 1)])
def test_copy_conj_transpose(pd, ps):
    """Batched copies with precision change, plain and conjugate-transposed in
    one batch: ragged shapes that span several 32 x 32 tiles, one-row and
    one-column blocks, an empty one, padded leading dimensions on both sides.
    Bit-exact (a copy, conjugation and round-to-nearest conversion); the
    padding rows of every destination keep their sentinel."""
    rng = np.random.default_rng(70 + 2 * pd + ps)
    npd, _ = CT[pd]
    nps, _ = CT[ps]
    shapes = [(1000, 700, 1), (700, 1000, 0), (33, 31, 1), (1, 257, 1), (257, 1, 1), (0, 5, 1),
              (64, 64, 0), (95, 130, 1), (5, 3, 0), (2048, 40, 1)]
    keep, cases, dims, ld, ptr, ctl = [], [], [], [], [], []
    for (m, n, ct) in shapes:
        S = crandn(rng, m, n).astype(nps)
        lds = m + 3
        Sp = np.zeros((lds, max(n, 1)), dtype=nps)
        Sp[:m, :n] = S
        dm, dn = (n, m) if ct else (m, n)
        ldd = dm + 5
        Dp = np.full((ldd, max(dn, 1)), 7.0 - 3.0j, dtype=npd)
        tS = torch.from_numpy(np.ascontiguousarray(Sp.T)).to(DEV)
        tD = torch.from_numpy(np.ascontiguousarray(Dp.T)).to(DEV)
        keep += [tS, tD]
        ref = Dp.copy()
        ref[:dm, :dn] = (S.conj().T if ct else S).astype(npd)
        cases.append((tD, ref, ldd, max(dn, 1)))
        dims += [m, n]
        ld += [lds, ldd]
        ptr += [tS.data_ptr(), tD.data_ptr()]
        ctl.append(ct)
    a1, p1 = i32(dims)
    a2, p2 = i32(ld)
    a3, p3 = i64(ptr)
    a4, p4 = i32(ctl)
    assert lib.nudft2_test_copy(pd, ps, len(shapes), p1, p2, p3, p4) == 0
    for tD, ref, ldd, dn in cases:
        got = tD.cpu().numpy().reshape(dn, ldd).T
        assert np.array_equal(got, ref)


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("opa,opb", [(0, 0), (1, 0), (0, 1), (1, 1)])
def test_gemm_stream_k(prec, opa, opb):
    """Stream-K shares forced on a ragged batch: each descriptor's tiles x k
    stages dealt out in equal pieces that start and end inside tiles, added
    atomically to a pre-scaled C.  Shapes around the tile (64) and k stage
    (16), one with k = 1 stage, an empty k and an empty output in the same
    launch; beta = 0.5, alpha complex.  Also a single long product (the QR
    V^H C shape class at reduced size)."""
    rng = np.random.default_rng(140 + 8 * prec + 2 * opa + opb)
    batches = [[(300, 200, 5000), (129, 77, 3001), (64, 64, 16), (65, 63, 17), (200, 100, 0),
                (0, 40, 100), (1, 1, 999)],
               [(256, 1500, 3000)]]
    alpha, beta = 0.7 - 0.4j, 0.5
    for shapes in batches:
        mats, keep, mnk, ld, ptr = [], [], [], [], []
        for (m, n, k) in shapes:
            A = crandn(rng, *((m, k) if opa == 0 else (k, m)))
            B = crandn(rng, *((k, n) if opb == 0 else (n, k)))
            Cm = crandn(rng, m, n)
            ta, tb, tc = (to_dev(A, prec) if A.size else torch.zeros(1, dtype=CT[prec][1], device=DEV),
                          to_dev(B, prec) if B.size else torch.zeros(1, dtype=CT[prec][1], device=DEV),
                          to_dev(Cm, prec) if Cm.size else torch.zeros(1, dtype=CT[prec][1], device=DEV))
            keep += [ta, tb, tc]
            mats.append((A, B, Cm, tc))
            mnk += [m, n, k]
            ld += [max(1, A.shape[0]), max(1, B.shape[0]), max(1, m)]
            ptr += [ta.data_ptr(), tb.data_ptr(), tc.data_ptr()]
        a1, p1 = i32(mnk)
        a2, p2 = i32(ld)
        a3, p3 = i64(ptr)
        st = lib.nudft2_test_gemm_cfg(prec, opa, opb, len(shapes), p1, p2, p3, alpha.real,
                                      alpha.imag, beta, -3, None)
        assert st == 0, lib.nudft2_last_error()
        for (m, n, k), (A, B, Cm, tc) in zip(shapes, mats):
            if m == 0 or n == 0:
                continue
            oA = A if opa == 0 else A.conj().T
            oB = B if opb == 0 else B.conj().T
            ref = alpha * (oA @ oB) + beta * Cm
            got = from_dev(tc, m, n)
            scale = max(1.0, np.abs(ref).max())
            assert np.abs(got - ref).max() < TOL[prec] * scale * max(k, 1) ** 0.5 * 10, (m, n, k)


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("opa,opb", [(0, 0), (1, 0), (0, 1), (1, 1)])
def test_gemm_partial_tile_splits(prec, opa, opb):
    """k splits kept as partial tiles in scratch and summed in split order by a
    second kernel (forced, splits = -4): ragged outputs of one to a few tiles,
    k long and short (splits past k hold nothing), k = 0 and an empty output
    in the same launch, beta = 0.5 and 0, alpha complex.  Then the library's
    own choice on a batch of tall-panel Gram shapes (128 x 128, k = 9000),
    which takes this path."""
    rng = np.random.default_rng(160 + 8 * prec + 2 * opa + opb)
    alpha = -0.6 + 0.3j
    runs = [([(128, 128, 5000), (65, 127, 4099), (1, 64, 700), (64, 1, 33), (100, 90, 0),
              (0, 30, 200), (130, 70, 17)], -4, 0.5),
            ([(128, 128, 9000)] * 4 + [(128, 96, 8191)], 0, 0.0)]
    for shapes, sp, beta in runs:
        mats, keep, mnk, ld, ptr = [], [], [], [], []
        for (m, n, k) in shapes:
            A = crandn(rng, *((m, k) if opa == 0 else (k, m)))
            B = crandn(rng, *((k, n) if opb == 0 else (n, k)))
            Cm = crandn(rng, m, n)
            ts = [to_dev(X, prec) if X.size else torch.zeros(1, dtype=CT[prec][1], device=DEV)
                  for X in (A, B, Cm)]
            keep += ts
            mats.append((A, B, Cm, ts[2]))
            mnk += [m, n, k]
            ld += [max(1, A.shape[0]), max(1, B.shape[0]), max(1, m)]
            ptr += [t.data_ptr() for t in ts]
        a1, p1 = i32(mnk)
        a2, p2 = i32(ld)
        a3, p3 = i64(ptr)
        st = lib.nudft2_test_gemm_cfg(prec, opa, opb, len(shapes), p1, p2, p3, alpha.real,
                                      alpha.imag, beta, sp, None)
        assert st == 0, lib.nudft2_last_error()
        for (m, n, k), (A, B, Cm, tc) in zip(shapes, mats):
            if m == 0 or n == 0:
                continue
            oA = A if opa == 0 else A.conj().T
            oB = B if opb == 0 else B.conj().T
            ref = alpha * (oA @ oB) + beta * Cm
            got = from_dev(tc, m, n)
            scale = max(1.0, np.abs(ref).max())
            assert np.abs(got - ref).max() < TOL[prec] * scale * max(k, 1) ** 0.5 * 10, (m, n, k)


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("code", [-5, -6])
def test_gemm_forced_small_tiles(prec, code):
    """The small-output tile shapes the autotuner can pick for A^H B with
    m <= 32 (-5: 32 x 128 tiles, -6: 16- or 32-square tiles), forced on ragged
    batches with short and long k, k = 0 and an empty output in the same
    launch, beta = 0.5, alpha complex; shapes the tiles do not cover are
    rejected with E_INVAL and leave C untouched."""
    rng = np.random.default_rng(180 + 4 * prec - code)
    nmax = 128 if code == -5 else 32
    shapes = [(32, nmax, 5000), (17, nmax - 3, 333), (1, 9, 70), (32, 12, 1), (20, 20, 0),
              (0, 16, 100)]
    alpha, beta = 0.4 + 0.9j, 0.5
    mats, keep, mnk, ld, ptr = [], [], [], [], []
    for (m, n, k) in shapes:
        A = crandn(rng, k, m)
        B = crandn(rng, k, n)
        Cm = crandn(rng, m, n)
        ts = [to_dev(X, prec) if X.size else torch.zeros(1, dtype=CT[prec][1], device=DEV)
              for X in (A, B, Cm)]
        keep += ts
        mats.append((A, B, Cm, ts[2]))
        mnk += [m, n, k]
        ld += [max(1, k), max(1, k), max(1, m)]
        ptr += [t.data_ptr() for t in ts]
    a1, p1 = i32(mnk)
    a2, p2 = i32(ld)
    a3, p3 = i64(ptr)
    st = lib.nudft2_test_gemm_cfg(prec, 1, 0, len(shapes), p1, p2, p3, alpha.real, alpha.imag,
                                  beta, code, None)
    assert st == 0, lib.nudft2_last_error()
    for (m, n, k), (A, B, Cm, tc) in zip(shapes, mats):
        if m == 0 or n == 0:
            continue
        ref = alpha * (A.conj().T @ B) + beta * Cm
        got = from_dev(tc, m, n)
        scale = max(1.0, np.abs(ref).max())
        assert np.abs(got - ref).max() < TOL[prec] * scale * max(k, 1) ** 0.5 * 10, (m, n, k)
    # out of range: m > 32, n above the tile, op(A) = N
    for (m, n, k, opa) in [(33, 16, 100, 1), (16, nmax + 1, 100, 1), (16, 16, 100, 0)]:
        A = crandn(rng, *((k, m) if opa else (m, k)))
        B = crandn(rng, k, n)
        Cm = crandn(rng, m, n)
        ta, tb, tc = to_dev(A, prec), to_dev(B, prec), to_dev(Cm, prec)
        b1, q1 = i32([m, n, k])
        b2, q2 = i32([A.shape[0], k, m])
        b3, q3 = i64([ta.data_ptr(), tb.data_ptr(), tc.data_ptr()])
        st = lib.nudft2_test_gemm_cfg(prec, opa, 0, 1, q1, q2, q3, 1.0, 0.0, 0.0, code, None)
        assert st == 1 and b"forced small tile" in lib.nudft2_last_error()
        torch.cuda.synchronize()
        assert np.array_equal(from_dev(tc, m, n), Cm.astype(CT[prec][0]))


@pytest.mark.parametrize("prec", [0, 1])
def test_trtri_inverts_upper_triangles(prec):
    """Batched in-place inversion of upper-triangular matrices (the solves'
    stored D11^{-1} and root R^{-1}) against LAPACK's inverse, for orders
    around the 128-row diagonal blocks and the doubling joins."""
    rng = np.random.default_rng(77 + prec)
    ks = [1, 5, 128, 129, 300, 1000, 1537]
    keep, ref, kk, ld, ptr = [], [], [], [], []
    for k in ks:
        R = np.triu(crandn(rng, k, k)) / np.sqrt(k)
        R[np.diag_indices(k)] = 1.0 + 0.5 * rng.random(k) * np.exp(2j * np.pi * rng.random(k))
        t = to_dev(R, prec)
        keep.append(t)
        ref.append(np.linalg.inv(R))
        kk.append(k)
        ld.append(k)
        ptr.append(t.data_ptr())
    a1, p1 = i32(kk)
    a2, p2 = i32(ld)
    a3, p3 = i64(ptr)
    assert lib.nudft2_test_trtri(prec, len(ks), p1, p2, p3) == 0, lib.nudft2_last_error()
    for k, t, X in zip(ks, keep, ref):
        got = from_dev(t, k, k)
        err = np.linalg.norm(got - X) / np.linalg.norm(X)
        print(f"trtri k={k} prec{prec}: {err:.1e}")
        assert np.abs(np.tril(got, -1)).max() == 0
        assert err < (1e-13 if prec == 0 else 2e-5) * max(1.0, np.log2(k))


@pytest.mark.parametrize("graded", [False, True])
@pytest.mark.parametrize("prec", [0, 1])
def test_geqrf_dependent_columns(prec, graded):
    """QR of panels whose columns fall far below their norm against the
    earlier ones (where the FP32 panels split): numerical rank below the
    column count, repeated and zero columns, steeply graded columns, columns
    that differ by a small multiple of an earlier one, beside a well
    conditioned problem; m at the row pass's edges.  Q R = A column by column
    relative to the column's norm, Q unitary, both to rounding as in
    test_geqrf_ormqr."""
    rng = np.random.default_rng(700 + prec)
    eps = 1e-15 if prec == 0 else 6e-8
    mats = []
    for m, n, r in [(353, 160, 20), (64, 48, 5), (1100, 96, 40), (129, 129, 60), (40, 200, 33)]:
        A = crandn(rng, m, r) @ crandn(rng, r, n) / r ** 0.5
        mats.append(A + 4 * eps * crandn(rng, m, n))
    A = crandn(rng, 500, 130)
    A[:, 7] = A[:, 3]
    A[:, 40] = 0
    A[:, 41] = 2j * A[:, 2] + 3 * A[:, 39]
    A[:, 100:] = A[:, :30]
    mats.append(A)
    A = crandn(rng, 193, 64)
    mats.append(A * 10.0 ** (-np.arange(64) % 9))
    B = crandn(rng, 700, 70)
    for j in range(1, 70):
        B[:, j] = B[:, j - 1] + 10.0 ** -(j % 8) * B[:, j]
    mats.append(B)
    # a half lost per column: norms fall slowly, the panel's digits add up
    D = crandn(rng, 900, 130)
    for j in range(1, 130):
        D[:, j] = D[:, j - 1] + 0.6 * D[:, j]
    mats.append(D @ (np.eye(130) - 0.9 * np.eye(130, k=1)))
    i = np.arange(400)[:, None] / 400
    mats.append(1 / (i + np.arange(100) / 100 + 0.01 + 0.002j))   # Cauchy-like
    mats.append(crandn(rng, 300, 97))
    keep, data, mn, ld, ptr = [], [], [], [], []
    for A in mats:
        m, n = A.shape
        k = min(m, n)
        nob = (k + QB - 1) // QB
        tA = to_dev(A, prec)
        A = from_dev(tA, m, n).astype(np.complex128)   # as rounded
        tR = torch.full((n, k), 7.0 - 3.0j, dtype=CT[prec][1], device=DEV)
        tT = torch.full((QB * QB * (nob - 1) + (k - QB * (nob - 1)) ** 2,), 5.0 + 1.0j,
                        dtype=CT[prec][1], device=DEV)
        keep += [tA, tR, tT]
        data.append((A, tA, tR, tT))
        mn += [m, n]
        ld += [m, k]
        ptr += [t.data_ptr() for t in (tA, tR, tT)]
    a1, p1 = i32(mn)
    a2, p2 = i32(ld)
    a3, p3 = i64(ptr)
    geqrf = lib.nudft2_test_geqrf_graded if graded else lib.nudft2_test_geqrf
    assert geqrf(prec, len(mats), p1, p2, p3) == 0, lib.nudft2_last_error()
    dims, ld2, ptr2, Qs = [], [], [], []
    for A, tA, tR, tT in data:
        m, n = A.shape
        tQ = to_dev(np.eye(m), prec)
        Qs.append(tQ)
        dims += [m, min(m, n), m]
        ld2 += [m, m]
        ptr2 += [tA.data_ptr(), tT.data_ptr(), tQ.data_ptr()]
    b1, q1 = i32(dims)
    b2, q2 = i32(ld2)
    b3, q3 = i64(ptr2)
    assert lib.nudft2_test_ormqr(prec, 0, len(mats), q1, q2, q3) == 0, lib.nudft2_last_error()
    for i, ((A, tA, tR, tT), tQ) in enumerate(zip(data, Qs)):
        m, n = A.shape
        k = min(m, n)
        Q, R = from_dev(tQ, m, m).astype(np.complex128), from_dev(tR, k, n).astype(np.complex128)
        assert np.abs(np.tril(R, -1)).max() == 0
        cn = np.linalg.norm(A, axis=0)
        err = (np.linalg.norm(Q[:, :k] @ R - A, axis=0) / np.where(cn > 0, cn, 1)).max()
        orth = np.abs(Q.conj().T @ Q - np.eye(m)).max()
        print(f"dependent qr {i} {m}x{n} prec{prec}: recon {err:.1e} orth {orth:.1e}")
        assert err < 50 * TOL[prec] * np.sqrt(m)
        assert orth < 50 * TOL[prec] * np.sqrt(m)


def test_copy_lists_longer_than_a_launch():
    """70 000 conversions (and as many conjugate transposes) in one call, as a
    level of a batch of thousands of small problems has: more than one launch
    holds in grid.y.  Exact."""
    n = 70000
    S = torch.randn((n, 4), dtype=torch.complex64, device=DEV)
    D = torch.zeros((2 * n, 4), dtype=torch.complex128, device=DEV)
    src = S.data_ptr() + 32 * np.arange(n, dtype=np.int64)
    ptr = np.stack([np.tile(src, 2), D.data_ptr() + 64 * np.arange(2 * n, dtype=np.int64)], axis=1)
    a1, p1 = i32(np.full(4 * n, 2))
    a2, p2 = i32(np.full(4 * n, 2))
    a3, p3 = i64(ptr.ravel())
    a4, p4 = i32(np.repeat([0, 1], n))
    assert lib.nudft2_test_copy(0, 1, 2 * n, p1, p2, p3, p4) == 0, lib.nudft2_last_error()
    assert torch.equal(D[:n], S.to(torch.complex128))
    ct = S.reshape(n, 2, 2).transpose(1, 2).conj().reshape(n, 4)
    assert torch.equal(D[n:], ct.to(torch.complex128))


@pytest.mark.parametrize("shapes", [
    # one tall problem: as many row chunks as steps / 4, and the most
    [(4097, 33), (70, 40)], [(8193, 40), (5000, 64), (100, 128)], [(33001, 64)],
    # lists whose partial Grams fill the scratch, and one too long for it
    [(4200, 48)] * 32, [(4200, 40)] * 33,
])
@pytest.mark.parametrize("rank", [None, 9])
def test_geqrf_tall_panels(shapes, rank):
    """FP32 panels over thousands of rows, full rank and of rank 9 (their panels
    split): V's and T's reflectors times R give back A column by column, and
    are unitary.  A column is rounded to FP32 once per panel and half, and each
    of its at most n reflectors adds a rounding of the column's norm: 8 n 2^-24."""
    rng = np.random.default_rng(90)
    keep, mn, ld, ptr, cases = [], [], [], [], []
    for m, n in shapes:
        k = min(m, n)
        A = crandn(rng, m, n) if rank is None else crandn(rng, m, rank) @ crandn(rng, rank, n)
        tA = to_dev(A, 1)
        A = tA.to(torch.complex128).clone()
        tR = torch.full((n, k), 7.0, dtype=torch.complex64, device=DEV)
        tT = torch.zeros((k * k,), dtype=torch.complex64, device=DEV)
        keep += [tA, tR, tT]
        cases.append((A, tA, tR, tT, m, n, k))
        mn += [m, n]
        ld += [m, k]
        ptr += [t.data_ptr() for t in (tA, tR, tT)]
    a1, p1 = i32(mn)
    a2, p2 = i32(ld)
    a3, p3 = i64(ptr)
    assert lib.nudft2_test_geqrf(1, len(shapes), p1, p2, p3) == 0, lib.nudft2_last_error()
    for A, tA, tR, tT, m, n, k in cases:
        V = tA.to(torch.complex128)[:k].T.contiguous()          # m x k
        T = tT.to(torch.complex128).reshape(k, k).T.contiguous()
        R = tR.to(torch.complex128).T.contiguous()              # k x n
        E = torch.zeros((m, n), dtype=torch.complex128, device=DEV)
        E[:k] = R
        QR = E - V @ (T @ (V.conj().T.contiguous() @ E))
        nrm = torch.linalg.vector_norm(A, dim=1)
        err = (torch.linalg.vector_norm(QR.T - A, dim=1) / nrm).max().item()
        orth = V.conj().T.contiguous() @ V
        wy = T + T.conj().T - T.conj().T.contiguous() @ orth @ T   # zero where Q is unitary
        un = torch.linalg.matrix_norm(V @ wy, 2).item() if m < 10000 else wy.abs().max().item()
        print(f"tall {m}x{n}: {err:.1e} {un:.1e}")
        bound = 8 * 2.0 ** -24 * n
        assert err < bound and un < bound


@pytest.mark.parametrize("prec,opa,m,n,k,nb", [
    (2, 1, 256, 16, 256, 4), (2, 0, 256, 3, 256, 4), (0, 1, 100, 12, 700, 2),
    (2, 1, 32, 96, 512, 2), (0, 1, 20, 33, 600, 3),     # blocks of 16 columns
])
def test_gemm_choice_without_the_table(prec, opa, m, n, k, nb):
    """Code -2 is the library's choice but for the tuned table (the tuner's
    baseline): where the table has no entry it is code 0, bit for bit; code 1
    keeps the 64 x 64 tiles or the one-column kernels, to rounding."""
    rng = np.random.default_rng(60)
    cols = lambda X: to_dev(X, prec)
    ms = [[cols(crandn(rng, *s)) for s in (((m, k) if opa == 0 else (k, m)), (k, n))]
          for _ in range(nb)]
    a1, p1 = i32([m, n, k] * nb)
    a2, p2 = i32([m if opa == 0 else k, k, m] * nb)
    out = {}
    for code in (0, -2, 1):
        out[code] = torch.zeros((nb, n, m), dtype=CT[prec][1], device=DEV)
        a3, p3 = i64(sum([[A.data_ptr(), B.data_ptr(), out[code][i].data_ptr()]
                          for i, (A, B) in enumerate(ms)], []))
        assert lib.nudft2_test_gemm_cfg(prec, opa, 0, nb, p1, p2, p3, 1.0, 0.5, 0.0, code,
                                        None) == 0, lib.nudft2_last_error()
    assert torch.equal(out[0], out[-2])
    eps = 2.0 ** -24 if prec else 2.0 ** -53
    for i, (A, B) in enumerate(ms):
        scale = abs(1 + 0.5j) * ((A.abs() if opa else A.abs().T).to(torch.float64)
                                 @ B.abs().T.to(torch.float64))   # m x n of |op(A)| |B|
        err = ((out[0][i] - out[1][i]).T.abs() / scale).max().item()
        assert err < 16 * eps * np.sqrt(k)


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("opa,m,n,k,nb", [
    # each side of the lines between gemm_n16_kernel, the one-column kernels and
    # the tiles, with ragged sizes
    (1, 70, 5, 95, 3), (1, 70, 5, 97, 3), (1, 70, 8, 191, 3), (1, 70, 6, 192, 3),
    (1, 65, 9, 63, 30), (1, 65, 9, 31, 60), (1, 65, 16, 127, 200), (1, 65, 16, 129, 200),
    (0, 65, 2, 64, 7), (0, 65, 3, 63, 7), (0, 65, 4, 65, 80), (0, 65, 5, 191, 120),
    (0, 65, 16, 193, 120),
    (1, 31, 17, 63, 3), (1, 31, 48, 65, 9), (1, 31, 17, 100, 30), (1, 9, 128, 200, 20),
    (1, 31, 100, 1030, 3), (1, 31, 33, 1030, 40), (1, 31, 20, 1100, 150),
    # k ranges from half the CUs down, and none above
    (1, 250, 9, 511, 8), (1, 250, 9, 520, 8), (1, 250, 9, 1025, 9), (0, 250, 7, 1030, 8),
])
def test_gemm_route_lines(prec, opa, m, n, k, nb):
    """Entrywise as test_gemm_up_to_16_columns, on both sides of every line of
    the choice of kernel."""
    rng = np.random.default_rng(61)
    ct = CT[prec][0]
    A = crandn(rng, *((m, k) if opa == 0 else (k, m))).astype(ct)
    tA = to_dev(A, prec)
    Bs = [crandn(rng, k, n).astype(ct) for _ in range(min(nb, 3))]
    tBs = [to_dev(B, prec) for B in Bs]
    C0 = torch.randn((n, m), dtype=CT[prec][1], device=DEV)
    tC = C0.repeat(nb, 1, 1)
    a1, p1 = i32([m, n, k] * nb)
    a2, p2 = i32([A.shape[0], k, m] * nb)
    a3, p3 = i64(sum([[tA.data_ptr(), tBs[i % len(tBs)].data_ptr(), tC[i].data_ptr()]
                      for i in range(nb)], []))
    alpha, beta = 0.8 - 0.5j, 0.5
    st = lib.nudft2_test_gemm(prec, opa, 0, nb, p1, p2, p3, alpha.real, alpha.imag, beta)
    assert st == 0, lib.nudft2_last_error()
    oA = (A if opa == 0 else A.conj().T).astype(np.complex128)
    c0 = C0.cpu().numpy().T
    eps = 2.0 ** -24 if prec else 2.0 ** -53
    got = tC.cpu().numpy()
    for i in range(nb):
        B = Bs[i % len(Bs)]
        ref = alpha * (oA @ B.astype(np.complex128)) + beta * c0
        scale = abs(alpha) * (np.abs(oA) @ np.abs(B)) + beta * np.abs(c0)
        assert (np.abs(got[i].T - ref) / scale).max() < 8 * eps * np.sqrt(k), i


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("opa", [0, 1])
@pytest.mark.parametrize("beta", [0.0, 0.5, 1.0])
@pytest.mark.parametrize("n,code,shapes", [
    # one column, by the list's longest k: 16 lanes a row of C (op C) up to 512, a
    # wave a row up to 2048, a workgroup a row above; op N with a k split from 512
    (1, 0, [(1, 1), (300, 511), (257, 0), (33, 512), (5000, 64)]),
    (1, 0, [(300, 513), (64, 1023), (5, 9)]),
    (1, 0, [(300, 2047), (7, 1)]),
    (1, 0, [(77, 2049), (200, 9001), (5, 4097)]),
    (1, 0, [(64, 40000), (1, 9)]),
    # as many workgroups as fill the device: 256 rows each (op N)
    (1, 0, [(3, 5)] * 1030),
    (4, 0, [(3, 5)] * 1030),
    # two to four columns (FP32 op N: below the 16-column kernel's k of 64)
    (2, 0, [(300, 63), (17, 1), (1, 20)]),
    (4, 0, [(130, 60), (64, 33), (9, 0)]),
    # forced k splits keep the one-column kernels: 1, and 3 added atomically to a
    # scaled C
    (3, 1, [(300, 700), (70, 64), (1, 9)]),
    (8, 1, [(300, 500), (257, 7), (17, 0)]),
    (8, 1, [(17, 3000), (64, 513)]),
    (2, 3, [(64, 9000), (17, 3000)]),
    (8, 3, [(17, 3000), (300, 700), (5, 33)]),
    (8, 3, [(40, 480), (3, 100)]),
])
def test_gemm_one_column_kernels(prec, opa, beta, n, code, shapes):
    """The kernels of up to 8 columns, each reached by a list of its own (the
    route goes by the list's largest sizes): entrywise as
    test_gemm_up_to_16_columns."""
    rng = np.random.default_rng(80 + 2 * prec + opa)
    ct = CT[prec][0]
    alpha = -0.4 + 1.1j
    mats, keep, mnk, ld, ptr = [], [], [], [], []
    uniq = {}
    for i, (m, k) in enumerate(shapes):
        nc = n if i % 3 < 2 else 1
        if (m, k) not in uniq or len(shapes) < 100:
            A = crandn(rng, *((m, k) if opa == 0 else (k, m))).astype(ct)
            B, Cm = crandn(rng, k, nc).astype(ct), crandn(rng, m, nc).astype(ct)
            ta, tb = (to_dev(X, prec) if X.size else torch.zeros(1, dtype=torch.complex128,
                                                                 device=DEV) for X in (A, B))
            uniq[(m, k)] = (A, B, Cm, ta, tb, nc)
        A, B, Cm, ta, tb, nc = uniq[(m, k)]
        tc = to_dev(Cm, prec)
        keep += [ta, tb, tc]
        mats.append((A, B, Cm, tc, nc))
        mnk += [m, nc, k]
        ld += [max(A.shape[0], 1), max(k, 1), m]
        ptr += [ta.data_ptr(), tb.data_ptr(), tc.data_ptr()]
    a1, p1 = i32(mnk)
    a2, p2 = i32(ld)
    a3, p3 = i64(ptr)
    st = lib.nudft2_test_gemm_cfg(prec, opa, 0, len(shapes), p1, p2, p3, alpha.real, alpha.imag,
                                  beta, code, None)
    assert st == 0, lib.nudft2_last_error()
    eps = 2.0 ** -24 if prec else 2.0 ** -53
    for (m, k), (A, B, Cm, tc, nc) in zip(shapes, mats):
        oA = (A if opa == 0 else A.conj().T).astype(np.complex128)
        ref = alpha * (oA @ B.astype(np.complex128)) + beta * Cm.astype(np.complex128)
        scale = abs(alpha) * (np.abs(oA) @ np.abs(B)) + beta * np.abs(Cm)
        got = from_dev(tc, m, nc)
        if k == 0 and beta == 0:
            assert not got.any()
            continue
        assert (np.abs(got - ref) / scale).max() < 8 * eps * np.sqrt(max(k, 4)), (m, nc, k)


@pytest.mark.parametrize("shapes", [
    [(50, 32), (20, 31), (9, 1)], [(100, 33), (70, 64), (40, 5)], [(80, 65), (90, 20), (70, 32)],
])
def test_geqrf_few_panels_a_half(shapes):
    # one or two panels in the list's largest half, and three: T's merge
    test_geqrf_tall_panels(shapes, None)


@pytest.mark.parametrize("prec,graded", [(0, False), (1, False), (1, True)])
def test_geqrf_dependent_columns_to_rounding(prec, graded):
    """Where panels hold columns nearly dependent on earlier ones, Q R = A and Q
    unitary to a small multiple of the stored precision u, so that a panel split
    too late shows: a panel's own errors are some 2 u (its Gram and blocks are
    FP64, A, V, R and T are rounded once), those of k / 32 panels and of the
    products that join them add like independent ones: 16 u sqrt(k) in all.
    With splits at a thousandth of the digits (a square of the norm left at 4e-12
    of the terms' in place of 4e-9) the panel's arithmetic gives 1.4e-5 for the
    sums and 2.9e-5 for the Cauchy matrix, FP32's bound being 8e-6 and 9.5e-6."""
    rng = np.random.default_rng(710 + prec)
    u = 2.0 ** -24 if prec else 2.0 ** -53
    mats = []
    for m, n, r in [(353, 160, 20), (64, 48, 5), (129, 129, 60), (40, 200, 33), (5000, 64, 12)]:
        mats.append(crandn(rng, m, r) @ crandn(rng, r, n) / r ** 0.5 + 4 * u * crandn(rng, m, n))
    A = crandn(rng, 500, 130)
    A[:, 7] = A[:, 3]
    A[:, 40] = 0
    A[:, 41] = 2j * A[:, 2] + 3 * A[:, 39]
    A[:, 100:] = A[:, :30]
    mats.append(A)
    B = crandn(rng, 700, 70)      # sums: each column an earlier one and a little more
    for j in range(1, 70):
        B[:, j] = B[:, j - 1] + 10.0 ** -(j % 8) * B[:, j]
    mats.append(B)
    i = np.arange(400)[:, None] / 400
    mats.append(1 / (i + np.arange(100) / 100 + 0.01 + 0.002j))   # Cauchy
    keep, mn, ld, ptr = [], [], [], []
    for A in mats:
        m, n = A.shape
        k = min(m, n)
        tA = to_dev(A, prec)
        keep.append((tA.to(torch.complex128).clone(), tA,
                     torch.zeros((n, k), dtype=CT[prec][1], device=DEV),
                     torch.zeros(k * k, dtype=CT[prec][1], device=DEV)))
        mn += [m, n]
        ld += [m, k]
        ptr += [t.data_ptr() for t in keep[-1][1:]]
    a1, p1 = i32(mn)
    a2, p2 = i32(ld)
    a3, p3 = i64(ptr)
    geqrf = lib.nudft2_test_geqrf_graded if graded else lib.nudft2_test_geqrf
    assert geqrf(prec, len(mats), p1, p2, p3) == 0, lib.nudft2_last_error()
    for A, tV, tR, tT in keep:      # rows are columns
        n, m = A.shape
        k = min(m, n)
        V = tV.to(torch.complex128)[:k].T.contiguous()
        T = tT.to(torch.complex128).reshape(k, k).T.contiguous()
        E = torch.zeros((m, n), dtype=torch.complex128, device=DEV)
        E[:k] = tR.to(torch.complex128).T
        QR = E - V @ (T @ (V.conj().T.contiguous() @ E))
        nrm = torch.linalg.vector_norm(A, dim=1)
        err = torch.linalg.vector_norm(QR.T - A, dim=1) / torch.where(nrm > 0, nrm, 1.0)
        Q = torch.eye(m, k, dtype=torch.complex128, device=DEV)
        Q = Q - V @ (T @ V[:k].conj().T.contiguous())
        orth = (Q.conj().T.contiguous() @ Q
                - torch.eye(k, dtype=torch.complex128, device=DEV)).abs().max().item()
        print(f"dependent {m}x{n} prec{prec}: {err.max().item():.1e} {orth:.1e}")
        assert err.max().item() < 16 * u * k ** 0.5, (m, n)
        assert orth < 16 * u * k ** 0.5, (m, n)
