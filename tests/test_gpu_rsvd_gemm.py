"""GPU parity: lrqmm_rsvd and lrqmm_gemm stage by stage (oracle outputs as inputs).

Singular vectors are unique only up to sign, so factors are compared through
Sigma, through the rank-r product U diag(Sigma) Vt and through orthonormality.
Tolerances (float32 kernels against the float64 oracle):
  Sigma            rtol 2e-5
  U Sigma Vt       relative Frobenius 2e-4 (truncation inside a near-degenerate
                   bulk amplifies float32 rounding of the sketch products)
  C from factors   relative Frobenius 3e-6 (float32 accumulation of 2r terms + dequant)
  integer GEMM     bit exact
"""
import numpy as np
import pytest

from oracle import lrqmm_oracle as o
import lrqmm_workloads as wl
from gpu_util import say, to_dev, to_np, rel_fro

pytestmark = pytest.mark.gpu


def _residual_parts(X, axis, bits):
    amax = o.absmax(X, axis)
    _, s = o.scales(amax, bits)
    codes = o.quantize(X, amax, axis, bits)
    return amax, s, codes, o.residual(X, codes, s, axis)


RSVD_CASES = [
    # rows, cols, axis, bits, rank, p, q, kind
    (256, 256, o.ROWWISE, 8, 8, 0, 0, "uniform_pm1"),
    (256, 256, o.COLWISE, 8, 8, 0, 0, "uniform_pm1"),
    (300, 517, o.ROWWISE, 4, 12, 5, 1, "normal"),
    (517, 300, o.COLWISE, 4, 12, 5, 1, "normal"),
    (1000, 130, o.ROWWISE, 8, 16, 8, 2, "uniform01"),
    (130, 1000, o.COLWISE, 8, 16, 8, 2, "relu_normal"),
    (1024, 768, o.ROWWISE, 4, 32, 8, 1, "normal_outliers"),
    (768, 1024, o.COLWISE, 4, 64, 16, 2, "normal"),
    (96, 80, o.ROWWISE, 8, 80, 0, 0, "normal"),
    # 4100 rows make fewer Gram workgroups (33 of 128 rows) than 4096 columns (64 of 64): the scratch for the
    # Gram partials has to cover the larger of the two
    (4100, 4096, o.ROWWISE, 4, 24, 8, 1, "normal"),
    # a tall operand with a narrow sketch: more than 64 Gram workgroups, summed in several batches
    (20000, 64, o.ROWWISE, 4, 8, 0, 1, "relu_normal"),
    (64, 20000, o.COLWISE, 4, 8, 0, 1, "normal"),
    # the same with a sketch of 32 padded columns (71 partials of 1024 entries)
    (9000, 200, o.ROWWISE, 4, 20, 8, 1, "normal"),
    (200, 9000, o.COLWISE, 4, 20, 8, 1, "relu_normal"),
]


@pytest.mark.parametrize("rows,cols,axis,bits,rank,p,q,kind", RSVD_CASES)
def test_rsvd_against_oracle(rows, cols, axis, bits, rank, p, q, kind):
    import paper_2409_18772_amd as L
    say("rsvd", rows, cols, axis, bits, rank, p, q, kind)
    X = wl.random_matrix(kind, rows, cols, seed=rows * 3 + cols)
    amax, s, codes, R = _residual_parts(X, axis, bits)
    om = o.gaussian_sketch(99, axis, cols, rank + p)
    U0, S0, Vt0 = o.rsvd(R, rank, om, q)
    # with the oracle's sketch handed in
    U, S, Vt = L.lrqmm_rsvd(to_dev(X), to_dev(amax), axis, bits, rank, p, q, seed=99, omega=to_dev(om))
    U, S, Vt = to_np(U), to_np(S), to_np(Vt)
    assert np.allclose(S, S0, rtol=2e-5, atol=0)
    assert np.all(S[:-1] >= S[1:])
    Rr0 = (U0 * S0) @ Vt0
    Rr = (U.astype(np.float64) * S) @ Vt
    assert rel_fro(Rr0, Rr) < 2e-4
    assert np.max(np.abs(U.T.astype(np.float64) @ U - np.eye(rank))) < 2e-5
    assert np.max(np.abs(Vt.astype(np.float64) @ Vt.T - np.eye(rank))) < 2e-5
    # with the library's own generator (same counter-based stream as the oracle's)
    U2, S2, Vt2 = L.lrqmm_rsvd(to_dev(X), to_dev(amax), axis, bits, rank, p, q, seed=99)
    assert np.array_equal(to_np(S2), S) and np.array_equal(to_np(U2), U) and np.array_equal(to_np(Vt2), Vt)


# The products over whole reductions, at the edges of their tiles (16 results), steps (32 of the reduction), waves (8 steps) and ranges, on both sides of their
# limits; nothing is truncated, so the factors are determined to float32.
@pytest.mark.parametrize("rows,cols,axis,ell", [
    (63, 64, o.ROWWISE, 8), (64, 64, o.COLWISE, 16), (65, 95, o.ROWWISE, 9), (97, 271, o.COLWISE, 33), (255, 287, o.ROWWISE, 65),
    (80, 2687, o.ROWWISE, 20), (80, 2688, o.COLWISE, 20), (2719, 66, o.ROWWISE, 48), (130, 4099, o.COLWISE, 7), (4097, 120, o.ROWWISE, 24),
    (4113, 70, o.COLWISE, 40), (100, 8192, o.ROWWISE, 17), (8193, 70, o.ROWWISE, 12), (8200, 64, o.ROWWISE, 20), (70, 8193, o.COLWISE, 12)])
def test_rsvd_whole_reductions(rows, cols, axis, ell):
    test_rsvd_against_oracle(rows, cols, axis, 4, ell, 0, 1, "normal")


@pytest.mark.parametrize("M,N,K,rank,lda,ldb", [(100, 4100, 1200, 12, 1203, 4101), (3100, 70, 900, 20, 901, 77), (67, 90, 2700, 40, 2701, 90)])
def test_rsvd_whole_reductions_of_two_operands(M, N, K, rank, lda, ldb):
    """Operands that take tiles or ranges of different sizes, with odd row strides, in one launch: the bits of one operand alone."""
    import torch
    import paper_2409_18772_amd as L
    A, B = (torch.empty((r, ld), device="cuda").normal_()[:, :c] for r, ld, c in ((M, lda, K), (K, ldb, N)))
    D = torch.zeros((M, N), device="cuda")
    L.lrqmm_matmul_ex(A, B, D, 8, rank, 8, 1, seed=5)
    Ac, Bc = A.contiguous(), B.contiguous()
    codes, amax = L.lrqmm_quantize(Ac, L.AXIS_ROW, 8)
    codesT, amaxT = L.lrqmm_quantize(Bc, L.AXIS_COL, 8)
    fa = L.lrqmm_rsvd(Ac, amax, L.AXIS_ROW, 8, rank, 8, 1, seed=5)
    fb = L.lrqmm_rsvd(Bc, amaxT, L.AXIS_COL, 8, rank, 8, 1, seed=5)
    assert torch.equal(L.lrqmm_gemm(codes, amax, codesT, amaxT, 8, fa, fb), D)


# The small SVD by tridiagonalization (from 5 columns on), at the edges of its register widths (16, 24, 32, 40, 48, 64, 80
# columns), of its lane groups and of the padding of its rows; no truncation, so the factors are determined to float32.
@pytest.mark.parametrize("ell", [31, 32, 33, 40, 41, 47, 57, 58, 59, 64, 65, 72, 73, 79, 80])
def test_rsvd_small_svd_sizes(ell):
    test_rsvd_against_oracle(260, 300, o.ROWWISE, 4, ell, 0, 1, "normal")


@pytest.mark.parametrize("ell", [1, 2, 4, 5, 6, 7, 8, 9, 15, 16, 17, 23, 24, 25, 39, 48, 49, 63])
def test_rsvd_small_svd_narrow_sizes(ell):
    """Both sides of the limit to the Jacobi solver (5 columns) and of the other register widths."""
    test_rsvd_against_oracle(260, 300, o.ROWWISE, 4, ell, 0, 1, "normal")


@pytest.mark.parametrize("copies,ell", [(2, 6), (2, 16), (4, 24), (8, 24), (2, 48), (2, 64)])
def test_rsvd_repeated_singular_values_other_widths(copies, ell):
    test_rsvd_repeated_singular_values(copies, ell)


@pytest.mark.parametrize("flat,k,ell", [(1e-3, 3, 8), (1e-3, 3, 24), (1e-4, 3, 16), (3e-5, 3, 32), (1e-3, 5, 64)])
def test_rsvd_flat_tail_other_widths(flat, k, ell):
    test_rsvd_flat_tail_far_below_the_top(flat, k, ell)


@pytest.mark.parametrize("k", [0, 1, 7, 40])
def test_rsvd_rank_deficient_residual_with_a_wide_sketch(k):
    """A residual of rank k under a sketch of 40 columns: dead columns for k < 40 (zero rows in the small matrix, which the
    tridiagonal solver leaves to the Jacobi solver).  The last column carries every row's maximum, 127 steps, and has no
    residual; the other entries lie in [0, 1) steps, so their codes are 0 and they are the residual."""
    import paper_2409_18772_amd as L
    rng = np.random.default_rng(k)
    X = np.zeros((200, 160), dtype=np.float32)
    if k:
        low = rng.uniform(0, 1, (200, k)) @ rng.uniform(0, 1, (k, 159))
        X[:, :-1] = 0.9 * low / low.max()
    R = X.astype(np.float64)
    X[:, -1] = 127.0
    amax = o.absmax(X, o.ROWWISE)
    U, S, Vt = (to_np(t).astype(np.float64) for t in L.lrqmm_rsvd(to_dev(X), to_dev(amax), 0, 8, 40, 0, 1, seed=3))
    assert np.all(np.isfinite(U)) and np.all(np.isfinite(S)) and np.all(np.isfinite(Vt))
    # float32 products of length 200 on a matrix known exactly to rank k (R itself is rounded to float32)
    assert np.linalg.norm((U * S) @ Vt - R) <= 1e-5 * max(np.linalg.norm(R), 1e-30)


def _whole_rsvd_of(R, ell):
    """All ell factors of an operand whose residual is R (|R| < 1/2): rounding to nearest with a last column of 127 in every
    row makes the step 1, every other code 0 and the last column's residual 0.  Returns float64 U, S, Vt of R."""
    import paper_2409_18772_amd as L
    X = np.concatenate([R, np.full((R.shape[0], 1), 127.0)], axis=1).astype(np.float32)
    amax = o.absmax(X, o.ROWWISE)
    out = L.lrqmm_rsvd(to_dev(X), to_dev(amax), 0, 8, ell, 0, 1, seed=3, round_mode=o.NEAREST)
    U, S, Vt = (to_np(t).astype(np.float64) for t in out)
    assert np.all(Vt[:, -1] == 0)
    return U, S, Vt[:, :-1]


@pytest.mark.parametrize("copies,ell", [(2, 40), (2, 80), (4, 40), (8, 40), (4, 80)])
def test_rsvd_repeated_singular_values(copies, ell):
    """Every singular value of R several times (equal diagonal blocks; the float32 products separate the copies by about
    1e-9 of the largest): the eigenvectors that the tridiagonal solver finds one by one are then 1e-8 off orthogonal in a
    numpy model of it, inside 1e-11 .. 1e-4, and its results come from the correction step (seen with its flags printed).  No truncation, so R and each
    group of singular values are determined: tolerances as above (Sigma 2e-5; reconstruction to the rounding of the factors
    and of the float32 products)."""
    rng = np.random.default_rng(copies * 100 + ell)
    k = ell // copies
    u, _, v = np.linalg.svd(rng.uniform(0, 1, (60, 50)), full_matrices=False)
    s = np.linspace(3.0, 1.0, k)
    R = np.kron(np.eye(copies), (u[:, :k] * s) @ v[:k])
    f = 0.4 / np.abs(R).max()
    R = (R * f).astype(np.float32)
    U, S, Vt = _whole_rsvd_of(R, ell)
    assert np.allclose(S, np.repeat(f * s, copies), rtol=2e-5, atol=0)
    assert np.max(np.abs(U.T @ U - np.eye(ell))) < 2e-5
    assert np.max(np.abs(Vt @ Vt.T - np.eye(ell))) < 2e-5
    assert np.linalg.norm((U * S) @ Vt - R) <= 1e-5 * np.linalg.norm(R)


@pytest.mark.parametrize("flat,k,ell", [(1e-3, 3, 40), (1e-3, 7, 80), (1e-4, 3, 80), (5e-5, 3, 80), (3e-5, 3, 80)])
def test_rsvd_flat_tail_far_below_the_top(flat, k, ell):
    """k large singular values and a flat tail at `flat` of the largest: the tail's eigenvalues differ by a few roundings
    of the matrix norm.  At 1e-3 the tridiagonal solver finds vectors more than 1e-4 off orthogonal (seen with its flags
    printed), at 1e-4 and below its off-diagonal is about 1e-14 of the norm, the limit for going on: the result is dropped,
    after the check or before the eigenvectors, and the Jacobi solver takes over.  The tail itself is
    known to the float32 products' noise, about 1e-7 of the largest value per entry, so Sigma there is held to 2e-6 of it."""
    rng = np.random.default_rng(ell + k)
    m, n = 260, 300
    u, _ = np.linalg.qr(rng.standard_normal((m, ell)))
    v, _ = np.linalg.qr(rng.standard_normal((n, ell)))
    s = np.full(ell, flat)
    s[:k] = np.linspace(1.0, 0.5, k)
    R = (u * s) @ v.T
    f = 0.4 / np.abs(R).max()
    R = (R * f).astype(np.float32)
    U, S, Vt = _whole_rsvd_of(R, ell)
    say("flat tail", flat, "tail of S / S[0]:", S[k] / S[0], "...", S[-1] / S[0])
    assert np.all(S[:-1] >= S[1:])
    assert np.allclose(S[:k], f * s[:k], rtol=2e-5, atol=0)
    assert np.max(np.abs(S[k:] - f * s[k:])) <= 2e-6 * S[0]
    assert np.max(np.abs(U.T @ U - np.eye(ell))) < 2e-5
    assert np.linalg.norm((U * S) @ Vt - R) <= 1e-5 * np.linalg.norm(R)


@pytest.mark.parametrize("ell", [8, 20, 24, 31, 40, 48, 64, 80])
def test_rsvd_flat_tail_orthonormal_factors(ell):
    """Three large singular values and a flat tail at 1e-2 of the largest: the tail's eigenvalues (1e-4 of the norm) differ by
    the float32 products' noise, about 1e-11 of the norm.  Factors orthonormal to float32 (bound as below)."""
    rng = np.random.default_rng(ell)
    u, _ = np.linalg.qr(rng.standard_normal((260, ell)))
    v, _ = np.linalg.qr(rng.standard_normal((300, ell)))
    s = np.full(ell, 1e-2)
    s[:3] = (1.0, 0.8, 0.6)
    R = (u * s) @ v.T
    R = (R * (0.4 / np.abs(R).max())).astype(np.float32)
    U, S, Vt = _whole_rsvd_of(R, ell)
    say("flat tail", ell, np.max(np.abs(Vt @ Vt.T - np.eye(ell))))
    assert np.max(np.abs(U.T @ U - np.eye(ell))) < 2e-7
    assert np.max(np.abs(Vt @ Vt.T - np.eye(ell))) < 2e-7
    assert np.linalg.norm((U * S) @ Vt - R) <= 1e-5 * np.linalg.norm(R)


@pytest.mark.parametrize("shape", ["dense", "rows"])
@pytest.mark.parametrize("ell", [5, 8, 16, 17, 24, 31, 32, 40, 48, 64, 80])
def test_rsvd_steep_spectrum(ell, shape):
    """Singular values from 1 down to 1e-5 of the largest.  A row of Vt is B^T u / sigma rounded to float32, so with the
    eigenvalue right relative to itself an entry of V^T V is off by at most 2 u + u^2 (u = 2^-24: each row has norm 1, its
    rounding error norm u); 2e-7 leaves 0.8e-7 for the solver, 1e-15 of the largest eigenvalue against 1e-10 of it being
    1e-5.  rows: the rows of R differ in size as the singular values do, which leaves a graded small matrix."""
    rng = np.random.default_rng(ell)
    m, n = 260, 300
    s = 10.0 ** -np.linspace(0, 5, ell)
    v, _ = np.linalg.qr(rng.standard_normal((n, ell)))
    if shape == "dense":
        u, _ = np.linalg.qr(rng.standard_normal((m, ell)))
    else:
        u, h = np.zeros((m, ell)), m // ell
        for i in range(ell):
            u[i * h:(i + 1) * h, i] = rng.uniform(0.5, 1.0, h)
    R = (u * s) @ v.T
    R = (R * (0.4 / np.abs(R).max())).astype(np.float32)
    U, S, Vt = _whole_rsvd_of(R, ell)
    kept = S > 0            # (the last columns of a sketch may fall below the pivot limit: dropped, zero)
    say("steep", ell, shape, "kept", int(kept.sum()), "tail", S[kept][-1] / S[0])
    assert kept.sum() >= ell - 1 - ell // 16
    assert np.max(np.abs(U[:, kept].T @ U[:, kept] - np.eye(int(kept.sum())))) < 2e-7
    assert np.max(np.abs(Vt[kept] @ Vt[kept].T - np.eye(int(kept.sum())))) < 2e-7
    assert np.linalg.norm((U * S) @ Vt - R) <= 1e-5 * np.linalg.norm(R)


def test_rsvd_truncation_between_nearly_equal_singular_values():
    """A case in which the rank-r truncation is not determined at float32 resolution: the residual of the tall
    conv-shaped operand (100352 x 576, ReLU inputs) with l = 16, one power iteration, truncated to r = 8.  The
    power iteration packs the captured bulk singular values together (44.06 and 44.00 at positions 8 and 9:
    sigma_r / (sigma_r - sigma_r+1) = 778), so the singular vectors on the two sides of the cut mix under a
    perturbation of the projected matrix of a few 1e-6 -- what float32 accumulation over 10^5 rows leaves --
    by a few 1e-3, and U S V^T moves by about 2e-4 of its norm although every singular value stands to 1e-7.
    Both truncations are equally good rank-8 approximations.  So the comparison is on what is unique -- the
    singular values, the orthonormality of the factors, and the approximation error |R - U S V^T|_F, which
    must equal the oracle's to 1e-6 -- and the distance itself is only held to the perturbation estimate
    gap factor x 1e-5 relative to the part of U S V^T at the cut."""
    import paper_2409_18772_amd as L
    w = wl.CONFIGS["c5_resnet50_conv_int4_r8"]
    X, _ = wl.make_inputs(w)
    rank, p, q = 8, 8, 1
    amax, s, codes, R = _residual_parts(X, o.ROWWISE, w.bits)
    om = o.gaussian_sketch(w.sketch_seed, 0, X.shape[1], rank + p)
    Q = o.range_finder(R, om, q)
    spectrum = np.linalg.svd(Q.T @ R, compute_uv=False)
    gap = spectrum[rank - 1] / (spectrum[rank - 1] - spectrum[rank])
    U0, S0, Vt0 = o.rsvd(R, rank, om, q)
    U, S, Vt = L.lrqmm_rsvd(to_dev(X), to_dev(amax), 0, w.bits, rank, p, q, seed=w.sketch_seed)
    U, S, Vt = (to_np(t).astype(np.float64) for t in (U, S, Vt))
    Rr0, Rr = (U0 * S0) @ Vt0, (U * S) @ Vt
    e0, e1 = np.linalg.norm(R - Rr0), np.linalg.norm(R - Rr)
    d = rel_fro(Rr0, Rr)
    say("gap factor", gap, "sigma rel", np.max(np.abs(S - S0) / S0), "U S Vt distance", d, "approximation error",
        e1, "oracle", e0)
    assert gap > 100                                    # the case is what it is meant to be
    assert np.allclose(S, S0, rtol=2e-5, atol=0)
    assert np.max(np.abs(U.T @ U - np.eye(rank))) < 2e-5 and np.max(np.abs(Vt @ Vt.T - np.eye(rank))) < 2e-5
    assert abs(e1 - e0) <= 1e-6 * e0
    assert d <= gap * 1e-5 * S0[rank - 1] / np.linalg.norm(S0)


def test_rsvd_zero_residual_and_errors():
    import torch
    import paper_2409_18772_amd as L
    # entries are exact multiples of the step: residual is exactly zero
    codes = np.random.default_rng(0).integers(-7, 8, size=(64, 48)).astype(np.float32)
    codes[:, 0] = 7
    X = codes * np.float32(0.25)
    X = np.ascontiguousarray(X)
    amax = o.absmax(X, o.ROWWISE)
    assert np.all(o.residual(X, o.quantize(X, amax, 0, 4), o.scales(amax, 4)[1], 0) == 0)
    U, S, Vt = L.lrqmm_rsvd(to_dev(X), to_dev(amax), 0, 4, 4, 2, 1, seed=1)
    U, S, Vt = to_np(U), to_np(S), to_np(Vt)
    assert np.all(np.isfinite(U)) and np.all(np.isfinite(Vt))
    assert np.all(S == 0) and np.all((U * S) @ Vt == 0)
    x = to_dev(X)
    a = to_dev(amax)
    with pytest.raises(L.LrqmmError):
        L.lrqmm_rsvd(x, a, 0, 4, 0)                 # rank 0
    with pytest.raises(L.LrqmmError):
        L.lrqmm_rsvd(x, a, 0, 4, 40, 10)            # l > cols
    with pytest.raises(L.LrqmmError):
        L.lrqmm_rsvd(x, a, 0, 4, 4, workspace=L.Workspace(1024))   # workspace too small


GEMM_CASES = [
    # M, N, K, bits, rank
    (256, 256, 256, 8, 8),
    (128, 128, 64, 8, 0),
    (200, 136, 328, 4, 5),
    (129, 257, 1000, 8, 16),
    (1, 1, 16, 8, 1),
    (64, 640, 576, 4, 8),
    (500, 300, 77, 8, 3),       # K not a multiple of 16: byte-wise operand path
    (384, 512, 2048, 4, 32),
    (1000, 64, 576, 4, 8),      # at most 64 columns: 64 x 64 tiles
    (300, 40, 100, 8, 4),       # ... ragged, byte-wise operand path
    (257, 65, 128, 4, 0),       # one column more: back to the 128-wide tile
]


@pytest.mark.parametrize("M,N,K,bits,rank", GEMM_CASES)
def test_gemm_int_exact_and_compensation(M, N, K, bits, rank):
    import paper_2409_18772_amd as L
    say("gemm", M, N, K, bits, rank)
    A = wl.random_matrix("normal", M, K, seed=M + K)
    B = wl.random_matrix("normal", K, N, seed=N + K + 1)
    amA, sA, Aq, Ra = _residual_parts(A, o.ROWWISE, bits)
    amB, sB, Bq, Rb = _residual_parts(B, o.COLWISE, bits)
    fa = fb = None
    U = None
    if rank:
        U, S, Vt = o.rsvd(Ra, rank, o.gaussian_sketch(1, 0, K, rank), 1)
        W, G, Zt = o.rsvd(Rb, rank, o.gaussian_sketch(1, 1, N, rank), 1)
        f32 = lambda x: np.ascontiguousarray(x, dtype=np.float32)
        U, S, Vt, W, G, Zt = map(f32, (U, S, Vt, W, G, Zt))
        fa = tuple(map(to_dev, (U, S, Vt)))
        fb = tuple(map(to_dev, (W, G, Zt)))
    C, Cint = L.lrqmm_gemm(to_dev(Aq), to_dev(amA), to_dev(np.ascontiguousarray(Bq.T)), to_dev(amB), bits,
                           fa, fb, want_cint=True)
    ref_int = o.int_gemm(Aq, Bq)
    assert np.array_equal(to_np(Cint).astype(np.int64), ref_int)
    if rank:
        Cref = o.compensate(Aq, sA, Bq, sB, U, S, Vt, W, G, Zt)
    else:
        Cref = o.compensate(Aq, sA, Bq, sB, None, None, None, None, None, None)
    assert rel_fro(Cref, to_np(C)) < 3e-6
    # without the int32 side output the float result is identical
    C2 = L.lrqmm_gemm(to_dev(Aq), to_dev(amA), to_dev(np.ascontiguousarray(Bq.T)), to_dev(amB), bits, fa, fb)
    assert np.array_equal(to_np(C2), to_np(C))


# Reductions that end inside a 16-byte group, at its edges, below one group, one code behind a staged tile (64, 128) or a
# chunk of the code products (64, 256), on each GEMM kernel: 64 x 64 and, without whole tiles, 256 x 256; then the other
# tiles of the smaller kernel.
@pytest.mark.parametrize("M,N,K,rank", [(70, 90, k, min(k, 5)) for k in (1, 3, 15, 16, 17, 31, 63, 65, 127, 129, 271)]
                         + [(600, 33, 641, 7), (2817, 2820, 143, 0), (150, 70, 1301, 20),
                            # enough tiles for 128 x 128, 64 x 128 and (at most 64 columns) 64 x 64 ones
                            (2100, 2050, 65, 4), (1029, 2045, 70, 3), (32800, 40, 37, 2)])
def test_gemm_reduction_tails(M, N, K, rank):
    test_gemm_int_exact_and_compensation(M, N, K, 8, rank)


def test_gemm_extreme_codes_and_limits():
    import torch
    import paper_2409_18772_amd as L
    M, N, K = 96, 160, 4096
    Aq = np.full((M, K), -128, dtype=np.int8)
    Bq = np.full((K, N), -128, dtype=np.int8)
    Aq[::3] = 127
    am = np.full(M, 127.0, dtype=np.float32)
    bm = np.full(N, 127.0, dtype=np.float32)
    C, Cint = L.lrqmm_gemm(to_dev(Aq), to_dev(am), to_dev(np.ascontiguousarray(Bq.T)), to_dev(bm), 8,
                           want_cint=True)
    assert np.array_equal(to_np(Cint).astype(np.int64), o.int_gemm(Aq, Bq))
    lib = L.load_library()
    ws = L.Workspace(1 << 20)
    z = torch.zeros(16, device="cuda")
    # K too large for int32 accumulation at 8 bits
    assert lib.lrqmm_gemm(1, 1, 131072, 8, 0, z.data_ptr(), z.data_ptr(), z.data_ptr(), z.data_ptr(), None, None,
                          None, None, None, None, z.data_ptr(), None, ws.ptr, ws.nbytes, None) == -2
    # empty output
    assert lib.lrqmm_gemm(0, 5, 16, 8, 0, None, None, None, None, None, None, None, None, None, None, None, None,
                          None, 0, None) == 0
    # missing workspace
    assert lib.lrqmm_gemm(1, 1, 16, 8, 0, z.data_ptr(), z.data_ptr(), z.data_ptr(), z.data_ptr(), None, None, None,
                          None, None, None, z.data_ptr(), None, None, 0, None) == -3


# The large-tile kernel with panels of more than 64 columns (bfloat16 planes, 32 columns at a time): one column more than
# 64, a chunk that is not full, whole chunks, the widest; whole and ragged tiles, the last rows and columns of each.
@pytest.mark.parametrize("M,N,K,rank", [(2816, 3072, 256, 33), (2817, 2820, 300, 40), (2900, 2819, 143, 48), (3072, 2816, 384, 64),
                                        (2830, 2840, 200, 80)])
def test_gemm_wide_panels_on_large_tiles(M, N, K, rank):
    """Random factors, sampled rows against float64; alpha, beta and a strided destination; the int32 sums beside C.
    Bound: an entry is a float32 sum of 2r + 1 terms of total magnitude S, which errs by at most (2r + 2) 2^-24 S, plus
    three roundings of the dequantization; the panel entries are length-K sums of float32 rounding each: a factor 4."""
    import torch
    import paper_2409_18772_amd as L
    rng = np.random.default_rng(M + rank)
    say("wide panels", M, N, K, rank)
    Aq = rng.integers(-128, 128, (M, K), dtype=np.int8)
    Bq = rng.integers(-128, 128, (K, N), dtype=np.int8)
    amA, amB = rng.uniform(0.5, 2.0, M).astype(np.float32), rng.uniform(0.5, 2.0, N).astype(np.float32)
    f32 = lambda x: np.ascontiguousarray(x, dtype=np.float32)
    orth = lambda n: f32(np.linalg.qr(rng.standard_normal((n, rank)))[0])
    U, Vt, W, Zt = orth(M), f32(orth(K).T), orth(K), f32(orth(N).T)
    S, G = (f32(np.sort(rng.uniform(0.1, 3.0, rank))[::-1]) for _ in range(2))
    dev = [to_dev(t) for t in (Aq, amA, np.ascontiguousarray(Bq.T), amB)]
    fa, fb = tuple(map(to_dev, (U, S, Vt))), tuple(map(to_dev, (W, G, Zt)))
    C, Cint = L.lrqmm_gemm(*dev, 8, fa, fb, want_cint=True)
    rows = np.unique(np.concatenate([[0, 255, 256, M - 1, M - 2, M // 256 * 256 - 1], rng.integers(0, M, 12)]))
    rows = rows[(rows >= 0) & (rows < M)]
    assert np.array_equal(to_np(Cint)[rows].astype(np.int64), Aq[rows].astype(np.int64) @ Bq.astype(np.int64))
    sa, sb = (amA / np.float32(127)).astype(np.float64), (amB / np.float32(127)).astype(np.float64)
    At, Bt = Aq[rows] * sa[rows, None], Bq * sb[None, :]
    us, P, Q = U[rows].astype(np.float64) * S, Vt @ Bt + (Vt.astype(np.float64) @ W) @ (G[:, None] * Zt.astype(np.float64)), G[:, None] * Zt.astype(np.float64)
    Sw = At @ W.astype(np.float64)
    ref = At @ Bt + us @ P + Sw @ Q
    size = np.abs(At @ Bt) + np.abs(us) @ (np.abs(Vt) @ np.abs(Bt)) + np.abs(At) @ np.abs(W) @ np.abs(Q)
    err = np.abs(to_np(C)[rows] - ref)
    assert np.all(err <= 4 * (2 * rank + 3) * 2.0 ** -24 * size)
    assert rel_fro(ref, to_np(C)[rows]) < 3e-6
    D = torch.full((M, N + 5), 0.5, dtype=torch.float32, device="cuda")
    L.lrqmm_gemm_ex(dev[0], dev[1], dev[2], dev[3], 8, D[:, :N], 1.5, -0.5, fa, fb)
    assert torch.all(D[:, N:] == 0.5)
    want = 1.5 * to_np(C)[rows].astype(np.float64) - 0.25
    assert np.abs(to_np(D)[rows, :N] - want).max() <= 3 * 2.0 ** -24 * np.abs(want).max() + 2.0 ** -24


# Both sides of the limit between the large-tile kernel and 128 x 128 tiles (512 tiles of 128 x 128, two per compute unit), narrow
# and wide panels, whole tiles and ragged ones; many more rows than columns (few tiles wide) and the reverse.
@pytest.mark.parametrize("M,N,rank", [(4096, 2048, 20), (4096, 2048, 40), (4096, 2049, 20), (4096, 2049, 40), (2570, 2830, 33),
                                      (3072, 3072, 33), (3072, 3072, 64), (4096, 2304, 12), (33024, 256, 16), (300, 17500, 33)])
def test_gemm_on_both_sides_of_the_large_tile_limit(M, N, rank):
    test_gemm_wide_panels_on_large_tiles(M, N, 144, rank)


# The smaller tiles: panels of 8 columns to 160 around the chunks of 32 that the epilogue takes at a time, on each tile shape
# (64 x 64, 64 x 128, 128 x 128), ragged at every edge, reductions of half a staged tile, one, and one byte more.
@pytest.mark.parametrize("M,N,K,rank", [(130, 70, 90, 1), (65, 129, 128, 4), (130, 70, 129, 12), (130, 70, 90, 16), (64, 64, 64, 17),
                                        (129, 191, 257, 32), (130, 97, 143, 33), (100, 190, 100, 80), (1030, 2050, 130, 20),
                                        (1030, 2050, 64, 36), (2050, 2049, 129, 16), (2050, 2049, 100, 49), (9000, 33, 40, 8)])
def test_gemm_panel_widths_on_small_tiles(M, N, K, rank):
    test_gemm_wide_panels_on_large_tiles(M, N, K, rank)


# Panels: rows of one workgroup short and over (32, 64 rows), k blocks that eight waves do not share evenly or that leave waves idle,
# every width of the factors; 64 rows a workgroup (16384 rows and more, both sides of the limit; 65 columns and more keep 32); tall operands with short rows in
# the persistent kernel, on both sides of its limits in rows, columns of the factor and K; each operand as the tall one; the tall
# kernel (from 32768, 49152, 57344, 65536 and 98304 rows on, by the width and the other operand's rows) and its limits: one chunk of planes, a
# last one of one k block and a whole one, rows and columns that end early, K below one load, a wave without rows.  Right panels whose
# groups of rows of a column end early, at every width of a group.
@pytest.mark.parametrize("M,N,K,bits,rank", [(33, 31, 65, 8, 1), (65, 97, 513, 8, 16), (64, 40, 577, 4, 17), (130, 95, 1100, 8, 33), (100, 129, 700, 4, 50),
                                             (96, 161, 2000, 8, 80), (16289, 64, 700, 8, 12), (16353, 30, 700, 8, 12), (16390, 70, 130, 4, 40),
                                             (17000, 90, 513, 4, 80), (16385, 70, 130, 8, 64), (16385, 70, 130, 8, 65), (16383, 60, 576, 4, 8), (16385, 61, 575, 4, 8), (20000, 33, 640, 8, 16),
                                             (20001, 20, 641, 8, 3), (50, 16401, 129, 4, 5), (70, 17001, 90, 8, 64),
                                             (32768, 40, 769, 8, 3), (32801, 24, 641, 4, 16), (33025, 20, 15, 8, 10), (33000, 50, 380, 8, 20), (49153, 41, 385, 8, 32),
                                             (49500, 60, 193, 4, 33), (49200, 60, 385, 8, 40), (65537, 50, 193, 8, 48), (65600, 48, 577, 4, 40), (66001, 30, 1601, 8, 9),
                                             (30, 32769, 1089, 8, 13), (40, 32999, 400, 4, 31), (60, 49155, 449, 8, 45),
                                             (49153, 41, 769, 8, 3), (49201, 24, 641, 4, 16), (49155, 20, 15, 8, 10), (49160, 129, 128, 8, 20), (40000, 129, 130, 8, 20),
                                             (98310, 60, 193, 4, 33), (98305, 50, 385, 8, 48), (57345, 128, 192, 8, 40), (57350, 129, 192, 8, 40),
                                             (37, 16403, 70, 8, 24), (55, 16405, 129, 4, 50), (73, 16407, 80, 8, 72), (31, 1023, 130, 8, 31),
                                             (66, 1025, 70, 4, 47), (65, 1027, 65, 8, 63), (81, 1026, 90, 8, 79), (40, 32999, 1217, 8, 31), (60, 49155, 1217, 8, 45)])
def test_gemm_panels(M, N, K, bits, rank):
    """Sampled rows against float64.  A term of the products is exact, the planes carry the factors to 2^-27 and a sum of K terms in
    float32 is off by less than K 2^-24 of the terms' absolute sum, of the order of sqrt(K) 2^-24 in practice: 3e-6, as above."""
    import paper_2409_18772_amd as L
    rng = np.random.default_rng(M + N + K)
    say("panels", M, N, K, bits, rank)
    q = 2 ** (bits - 1)
    Aq = rng.integers(-q, q, size=(M, K), dtype=np.int8)
    Bt = rng.integers(-q, q, size=(N, K), dtype=np.int8)
    amA, amB = (rng.uniform(0.5, 2.0, n).astype(np.float32) for n in (M, N))
    f32 = lambda *shape: rng.standard_normal(shape).astype(np.float32)
    U, S, Vt, W, G, Zt = f32(M, rank), np.abs(f32(rank)), f32(rank, K), f32(K, rank), np.abs(f32(rank)), f32(rank, N)
    C = to_np(L.lrqmm_gemm(to_dev(Aq), to_dev(amA), to_dev(Bt), to_dev(amB), bits, tuple(map(to_dev, (U, S, Vt))),
                           tuple(map(to_dev, (W, G, Zt)))))
    rows = np.unique(np.r_[0:3, 30:34, 62:66, M - 35:M - 30, M - 3:M, rng.integers(0, M, 40)])
    rows = rows[(rows >= 0) & (rows < M)]
    s = lambda am: (am / np.float32(q - 1)).astype(np.float64)
    d = np.float64
    At, Bd = Aq[rows] * s(amA)[rows, None], Bt.T * s(amB)[None, :]
    US, GZ = U[rows].astype(d) * S, G[:, None].astype(d) * Zt
    want = At @ Bd + US @ (Vt.astype(d) @ Bd) + (At @ W.astype(d) + US @ (Vt.astype(d) @ W.astype(d))) @ GZ
    assert rel_fro(want, C[rows]) < 3e-6
    # ... and no row or column far from it
    assert np.abs(C[rows] - want).max() < 1e-4 * np.sqrt((want ** 2).mean())
