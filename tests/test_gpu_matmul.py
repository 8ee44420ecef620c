"""GPU parity: the whole hot path (lrqmm_matmul) against the oracle's Algorithm 2.

Tolerance: relative Frobenius error of C against the float64 oracle
    tol = max(1e-5, 2 * 2^-24 * kappa),   kappa = (|C0|_F + |C - C0|_F) / |C|_F.
The GPU path computes the sketch products and the epilogue in float32 (Gram /
Cholesky / Jacobi in float64); emulating the factorization arithmetic on the CPU
gives 6e-9 (int8, Gaussian) to 5e-7 (int4 with outliers), so 1e-5 covers it with
room for accumulation-order differences.  The epilogue adds the compensation to
the dequantized product C0 in float32, so each output carries about one float32
rounding of |C0| and one of |C - C0|: when the two nearly cancel (floor
quantization of zero-mean data at 4 bits: |C0| is 40-200 times |C|) that
rounding, 2^-24 * kappa relative to C, is the floor of what float32 can deliver;
the factor 2 is margin for the 2r-term accumulation.
"""
import numpy as np
import pytest

from oracle import lrqmm_oracle as o
import lrqmm_workloads as wl
from gpu_util import say, to_dev, to_np, rel_fro, check_elementwise

pytestmark = pytest.mark.gpu

TOL = 1e-5


def tol_for(ref):
    C, C0 = ref["C"], ref["C0"]
    kappa = (np.linalg.norm(C0) + np.linalg.norm(C - C0)) / np.linalg.norm(C)
    return max(TOL, 2 * 2.0 ** -24 * kappa)


def _run_gpu(w, A, B):
    import paper_2409_18772_amd as L
    return to_np(L.lrqmm_matmul(to_dev(A), to_dev(B), w.bits, w.rank, w.oversample, w.power_iters,
                                seed=w.sketch_seed))


def test_config_one_full():
    w = wl.CONFIGS["c1_256_int8_r8"]
    A, B = wl.make_inputs(w)
    say("matmul", w.name)
    C = _run_gpu(w, A, B)
    ref = o.lrqmm(A, B, w.bits, w.rank, w.oversample, w.power_iters, seed=w.sketch_seed)
    assert rel_fro(ref["C"], C) < TOL
    check_elementwise(C, ref, w.rank, what=w.name)
    exact = o.exact_product(A, B)
    assert o.rel_err(exact, C) <= o.rel_err(exact, ref["C0"])
    # bit-identical on a second run (no atomics on floats, fixed reduction orders)
    assert np.array_equal(C, _run_gpu(w, A, B))


SMALL = [
    # name, M, N, K   (ragged: not multiples of any tile size)
    ("c2_4096_int8_r16", 200, 136, 328),
    ("c3_4096_int4_r32_outliers", 333, 517, 260),
    ("c4_16384_int4_r64", 640, 512, 768),
    ("c5_resnet50_conv_int4_r8", 3000, 64, 576),
    ("c1_256_int8_r8", 77, 50, 93),
]


@pytest.mark.parametrize("name,M,N,K", SMALL)
def test_scaled_configs_full_output(name, M, N, K):
    w = wl.scaled_config(name, M, N, K)
    A, B = wl.make_inputs(w)
    say("matmul", w.name)
    C = _run_gpu(w, A, B)
    ref = o.lrqmm(A, B, w.bits, w.rank, w.oversample, w.power_iters, seed=w.sketch_seed)
    d = rel_fro(ref["C"], C)
    say(w.name, "gpu vs oracle", d, "tol", tol_for(ref))
    assert d < tol_for(ref)
    check_elementwise(C, ref, w.rank, what=w.name)


SHORT_ROWS = [
    # M, N, K, rank, oversample, power_iters: K a multiple of 16 up to 576, ragged M
    (130, 70, 96, 4, 4, 1),
    (1000, 64, 576, 8, 0, 0),
    (257, 40, 640, 12, 4, 2),
    (64, 33, 400, 12, 8, 0),
    (500, 80, 272, 16, 8, 1),
    (90, 48, 16, 4, 0, 0),
    (2100, 24, 208, 5, 0, 1),
    (33, 40, 336, 16, 0, 0),
    (700, 64, 544, 8, 8, 1),
    (20, 24, 64, 4, 0, 0),
]


# Taller ones, below the rows from which A is read once (see test_limits_of_a_single_read): the joint passes over whole and ragged
# last tiles, the shortest and longest rows, unequal shares of the reduction, longer rows and a wider sketch.
TALL_SHORT_ROWS = [
    (8192, 64, 576, 8, 0, 0),
    (8193, 70, 96, 4, 4, 1),
    (8207, 33, 16, 4, 0, 0),
    (9000, 24, 208, 5, 0, 1),
    (10000, 40, 336, 16, 0, 0),
    (8300, 20, 544, 8, 8, 2),
    (8200, 40, 640, 12, 4, 1),
    (8300, 600, 610, 12, 4, 1),
    (8200, 33, 400, 12, 8, 0),
]


@pytest.mark.parametrize("mode", [o.FLOOR, o.NEAREST])
@pytest.mark.parametrize("M,N,K,r,p,q", SHORT_ROWS + TALL_SHORT_ROWS)
def test_short_rows_of_a_single_read(M, N, K, r, p, q, mode):
    """A with short rows and a sketch of at most 16 columns, below and above the number of rows from which row maxima,
    codes and the sketch product come from one read of A.  Checked against
    the oracle, and against the same call on a copy of A whose row stride (K + 1) rules that kernel out, so that
    the maxima and the quantizing pass run: the two differ only in the order in which the sketch
    product is summed."""
    import torch
    import paper_2409_18772_amd as L
    A = wl.random_matrix("relu_normal", M, K, seed=51)
    B = wl.random_matrix("normal", K, N, seed=52)
    say("short rows", M, N, K, "rank", r, "p", p, "q", q, "mode", mode)
    dA, dB = to_dev(A), to_dev(B)
    C = to_np(L.lrqmm_matmul(dA, dB, 4, r, p, q, seed=9, round_mode=mode))
    ref = o.lrqmm(A, B, 4, r, p, q, seed=9, round_mode=mode)
    d = rel_fro(ref["C"], C)
    say("gpu vs oracle", d, "tol", tol_for(ref))
    assert d < tol_for(ref)
    check_elementwise(C, ref, r, what=f"short rows {M}x{N}x{K}")
    wide = torch.zeros((M, K + 1), dtype=torch.float32, device="cuda")
    wide[:, :K] = dA
    D = torch.empty((M, N), dtype=torch.float32, device="cuda")
    L.lrqmm_matmul_ex(wide[:, :K], dB, D, 4, r, p, q, seed=9, round_mode=mode)
    assert rel_fro(C, to_np(D)) < tol_for(ref)
    # a row stride the one-read kernel accepts (K + 4): the same kernels on a window, the same bits
    wide4 = torch.zeros((M, K + 4), dtype=torch.float32, device="cuda")
    wide4[:, :K] = dA
    D4 = torch.empty((M, N), dtype=torch.float32, device="cuda")
    L.lrqmm_matmul_ex(wide4[:, :K], dB, D4, 4, r, p, q, seed=9, round_mode=mode)
    assert np.array_equal(C, to_np(D4))


@pytest.mark.parametrize("M,K,r,p,q", [(93438, 16, 2, 0, 0), (93437, 64, 16, 0, 0), (78760, 80, 5, 0, 0), (56720, 128, 8, 0, 0), (44500, 192, 8, 0, 0),
                                       (42600, 208, 3, 0, 0), (37281, 272, 8, 0, 0), (32240, 384, 16, 0, 0), (31751, 400, 8, 0, 0),
                                       (29185, 512, 2, 0, 0), (28917, 528, 8, 0, 0), (28161, 576, 16, 0, 0), (28159, 576, 16, 0, 0),
                                       (28200, 576, 4, 4, 0), (28165, 576, 12, 0, 1), (44487, 192, 4, 4, 1)])
def test_both_products_of_a_single_read(M, K, r, p, q):
    """Tall operands with short rows on both sides of the limits of a single read (see test_limits_of_a_single_read), rows past the last
    tile, columns past the last block of 64, with and without truncation or a power iteration."""
    test_short_rows_of_a_single_read(M, 48, K, r, p, q, o.FLOOR)


@pytest.mark.parametrize("M,K,r,p,q", [(96875, 16, 2, 0, 0), (96875, 64, 10, 0, 0), (96875, 64, 11, 0, 0), (56945, 144, 8, 0, 0), (40973, 288, 8, 0, 1),
                                       (33855, 384, 8, 8, 0), (32769, 400, 16, 0, 0), (32769, 432, 8, 0, 0), (32769, 576, 8, 0, 0),
                                       (32769, 576, 4, 4, 1)])
def test_limits_of_a_single_read(M, K, r, p, q):
    """The rows from which A is read once (quantization with one or both products): there C differs in bits from that of a copy whose
    row stride rules those kernels out; with one row less it does not."""
    import torch
    import paper_2409_18772_amd as L
    gen = torch.Generator(device="cuda").manual_seed(63)
    wide = torch.empty((M, K + 1), device="cuda").normal_(generator=gen).clamp_(min=0.0)
    B = torch.empty((K, 40), device="cuda").normal_(generator=gen)
    for rows in (M - 1, M):
        say("limit", rows, K, r, p, q)
        C = L.lrqmm_matmul(wide[:rows, :K].contiguous(), B, 4, r, p, q, seed=9)
        D = torch.empty_like(C)
        L.lrqmm_matmul_ex(wide[:rows, :K], B, D, 4, r, p, q, seed=9)
        assert torch.equal(C, D) == (rows < M)
        assert rel_fro(to_np(C), to_np(D)) < TOL


# Every block of 64 columns of the kernel that forms both products (q = 0, nothing truncated, at most a sixth as many sketch columns as A
# has), then widths of the one that forms R Omega alone, by steps of 32 columns; whole and ragged last tiles.
ONE_READ = [(96877, 16, 2, 0, 0), (96890, 64, 8, 0, 0), (82500, 80, 13, 0, 0), (60947, 128, 8, 0, 0), (48960, 192, 16, 0, 0), (47119, 208, 4, 0, 0),
            (41920, 272, 8, 0, 0), (33861, 384, 16, 0, 0), (32773, 400, 8, 0, 0), (32784, 512, 12, 0, 0), (32775, 528, 8, 0, 0), (32777, 576, 16, 0, 0),
            (96881, 16, 4, 0, 1), (96880, 32, 16, 0, 0), (96883, 64, 16, 0, 0), (72920, 96, 4, 4, 1), (53761, 160, 8, 8, 0), (47120, 208, 5, 0, 2),
            (38700, 336, 16, 0, 1), (32771, 480, 8, 4, 0), (32779, 544, 8, 8, 1), (32784, 576, 12, 0, 1)]


@pytest.mark.parametrize("mode,bits", [(o.FLOOR, 8), (o.NEAREST, 4), (o.NEAREST, 8)])
@pytest.mark.parametrize("M,K,r,p,q", ONE_READ)
def test_kernels_of_a_single_read(M, K, r, p, q, mode, bits):
    """Both rounding modes and code widths in the kernels that read a tall A once, against the oracle; that they ran shows in the
    bits, which differ from those of a copy whose row stride rules them out."""
    import torch
    import paper_2409_18772_amd as L
    N = 16
    A = wl.random_matrix("relu_normal", M, K, seed=64)
    B = wl.random_matrix("normal", K, N, seed=65)
    say("one read", M, K, "rank", r, "p", p, "q", q, "mode", mode, "bits", bits)
    dA, dB = to_dev(A), to_dev(B)
    C = to_np(L.lrqmm_matmul(dA, dB, bits, r, p, q, seed=9, round_mode=mode))
    ref = o.lrqmm(A, B, bits, r, p, q, seed=9, round_mode=mode)
    d = rel_fro(ref["C"], C)
    say("gpu vs oracle", d, "tol", tol_for(ref))
    assert d < tol_for(ref)
    # A truncation (p > 0) between nearly equal singular values is not unique in float32: for the residuals of 72920 x 96, 4 bits, nearest,
    # s_4 / (s_4 - s_5) = 234, so that roundings of 2^-24 turn the vectors at the cut by 234 times as much, and single elements of C by
    # up to that many 2^-24 S, where the budget allows 44; the norm stays within its tolerance.
    if p == 0:
        check_elementwise(C, ref, r, what=f"one read {M}x{N}x{K}")
    wide = torch.zeros((M, K + 1), dtype=torch.float32, device="cuda")
    wide[:, :K] = dA
    D = torch.empty((M, N), dtype=torch.float32, device="cuda")
    L.lrqmm_matmul_ex(wide[:, :K], dB, D, bits, r, p, q, seed=9, round_mode=mode)
    assert not np.array_equal(C, to_np(D))


def _tall_operand(kind, M, K, seed=61):
    rng = np.random.default_rng(seed)
    noise = rng.standard_normal((M, K))
    name, _, size = kind.partition(" ")
    if name == "scaled":                    # every entry
        A = np.maximum(noise, 0.0) * float(size)
    elif name == "factor":                  # rank 1 times 1 + noise
        A = np.outer(rng.random(M) + 0.5, rng.random(K) + 0.5) * (1.0 + float(size) * noise)
    elif name == "plus":                    # rank 1 plus noise
        A = np.outer(rng.random(M) + 0.5, rng.random(K) + 0.5) + float(size) * noise
    elif name == "graded":                  # columns over `size` powers of ten
        A = noise * np.logspace(0.0, -float(size), K)
    elif name == "columns":                 # a scale of its own for every column
        A = np.maximum(noise, 0.0) * np.exp(float(size) * rng.standard_normal(K))
    elif name == "means":                   # a mean of its own for every column
        A = np.maximum(noise + float(size) * rng.standard_normal(K), 0.0)
    elif name == "rank":                    # fewer dimensions than the sketch has columns, and entries that are codes themselves
        A = np.rint(7.0 * rng.random((M, int(size))))[:, np.arange(K) % int(size)]
    return A.astype(np.float32)


@pytest.mark.parametrize("mode", [o.FLOOR, o.NEAREST])
@pytest.mark.parametrize("kind", ["scaled 1e19", "scaled 1e12", "scaled 1e9", "scaled 1e-7", "scaled 1e-10", "scaled 1e-16", "scaled 1e-22", "scaled 1e-25",
                                  "factor 1e-1", "factor 3e-2", "factor 1e-2", "factor 1e-4", "factor 1e-5", "plus 1e-1", "plus 1e-2",
                                  "plus 1e-3", "graded 6", "columns 1", "columns 3", "means 1", "means 3", "rank 3", "rank 1"])
def test_tall_operands_with_structure(kind, mode):
    """Tall operands read once, q = 0, whose sample matrix is far from orthogonal or far from unit scale: C is as close to float64 as on a copy whose
    row stride (K + 1) rules the one-read kernel out, where R^T Q is a product of its own.  Each of the two rounds C's two terms to
    float32 once more than float64 does, 2^-24 kappa."""
    import torch
    import paper_2409_18772_amd as L
    M, N, K, r = 32800, 24, 576, 8
    A = _tall_operand(kind, M, K)
    B = wl.random_matrix("normal", K, N, seed=62)
    say("structured", kind, "mode", mode)
    dA, dB = to_dev(A), to_dev(B)
    ref = o.lrqmm(A, B, 4, r, 0, 0, seed=9, round_mode=mode)
    wide = torch.zeros((M, K + 1), dtype=torch.float32, device="cuda")
    wide[:, :K] = dA
    D = torch.empty((M, N), dtype=torch.float32, device="cuda")
    L.lrqmm_matmul_ex(wide[:, :K], dB, D, 4, r, 0, 0, seed=9, round_mode=mode)
    d_general = rel_fro(ref["C"], to_np(D))
    d = rel_fro(ref["C"], to_np(L.lrqmm_matmul(dA, dB, 4, r, 0, 0, seed=9, round_mode=mode)))
    kappa = (np.linalg.norm(ref["C0"]) + np.linalg.norm(ref["C"] - ref["C0"])) / np.linalg.norm(ref["C"])
    say("from float64: one read", d, "two", d_general, "kappa", kappa)
    assert d <= 1.5 * d_general + 2.0 ** -24 * kappa


def test_rank_zero_is_direct_quant_and_modes():
    import paper_2409_18772_amd as L
    A = wl.random_matrix("normal", 150, 200, seed=1)
    B = wl.random_matrix("normal", 200, 170, seed=2)
    for mode in (o.FLOOR, o.NEAREST):
        C = to_np(L.lrqmm_matmul(to_dev(A), to_dev(B), 8, 0, round_mode=mode))
        ref = o.lrqmm(A, B, 8, 0, round_mode=mode)
        assert rel_fro(ref["C"], C) < 1e-6
        check_elementwise(C, ref, 0, what=f"rank 0, round mode {mode}")
    C = to_np(L.lrqmm_matmul(to_dev(A), to_dev(B), 4, 6, 2, 1, seed=3, round_mode=o.NEAREST))
    ref = o.lrqmm(A, B, 4, 6, 2, 1, seed=3, round_mode=o.NEAREST)
    assert rel_fro(ref["C"], C) < TOL


def test_degenerate_inputs():
    import torch
    import paper_2409_18772_amd as L
    A = np.zeros((64, 96), dtype=np.float32)
    B = wl.random_matrix("normal", 96, 80, seed=2)
    C = to_np(L.lrqmm_matmul(to_dev(A), to_dev(B), 8, 4, 2, 1))
    assert np.all(C == 0)
    A = wl.random_matrix("normal", 64, 96, seed=1)
    A[5] = 0
    B[:, 7] = 0
    C = to_np(L.lrqmm_matmul(to_dev(A), to_dev(B), 8, 4, 2, 1, seed=5))
    ref = o.lrqmm(A, B, 8, 4, 2, 1, seed=5)
    assert rel_fro(ref["C"], C) < TOL
    assert np.all(C[5] == 0) and np.all(C[:, 7] == 0)
    with pytest.raises(L.LrqmmError):
        L.lrqmm_matmul(to_dev(A), to_dev(B), 8, 60, 30)          # l > K
    with pytest.raises(L.LrqmmError):
        L.lrqmm_matmul(to_dev(A), to_dev(B), 8, 81, 0)
    e = torch.empty((0, 96), dtype=torch.float32, device="cuda")
    assert L.lrqmm_matmul(e, to_dev(B), 8, 0).shape == (0, 80)


RAGGED = [
    # M, N, K, rank, oversample, power_iters, pad: nothing a multiple of a tile, chunk or store width; sketches of 2 to 5
    # tiles of 16 columns; the last two on the eight-wave workgroups of wide sketches
    (131, 97, 203, 20, 8, 1, 3),
    (70, 301, 65, 24, 8, 1, 0),
    (257, 66, 129, 33, 8, 1, 1),
    (129, 191, 127, 50, 10, 0, 5),
    (63, 70, 1031, 17, 0, 2, 2),
    (4099, 96, 1027, 60, 16, 0, 1),
    (96, 1027, 4099, 50, 6, 1, 0),
]


@pytest.mark.parametrize("mode", [o.FLOOR, o.NEAREST])
@pytest.mark.parametrize("M,N,K,r,p,q,pad", RAGGED)
def test_ragged_operands(M, N, K, r, p, q, pad, mode):
    """Quantization fused into the first residual pass and the passes themselves on shapes and row strides that suit no
    tile: against the oracle, and bit for bit against the separate calls (same arithmetic in the same order)."""
    import torch
    import paper_2409_18772_amd as L
    A, B = wl.random_matrix("uniform01", M, K, seed=61), wl.random_matrix("uniform01", K, N, seed=62)
    wa = torch.zeros((M, K + pad), dtype=torch.float32, device="cuda")
    wb = torch.zeros((K, N + pad), dtype=torch.float32, device="cuda")
    wa[:, :K], wb[:, :N] = to_dev(A), to_dev(B)
    dA, dB = wa[:, :K], wb[:, :N]
    say("ragged", M, N, K, "rank", r, "p", p, "q", q, "pad", pad, "mode", mode)
    D = torch.empty((M, N), dtype=torch.float32, device="cuda")
    C = to_np(L.lrqmm_matmul_ex(dA, dB, D, 8, r, p, q, seed=9, round_mode=mode))
    ref = o.lrqmm(A, B, 8, r, p, q, seed=9, round_mode=mode)
    d = rel_fro(ref["C"], C)
    say("gpu vs oracle", d, "tol", tol_for(ref))
    assert d < tol_for(ref)
    Aq, amA = L.lrqmm_quantize_ex(dA, L.AXIS_ROW, 8, mode)
    BqT, amB = L.lrqmm_quantize_ex(dB, L.AXIS_COL, 8, mode)
    assert np.array_equal(to_np(Aq), ref["Aq"]) and np.array_equal(to_np(BqT), ref["Bq"].T)
    fa = L.lrqmm_rsvd_ex(dA, amA, L.AXIS_ROW, 8, r, p, q, seed=9, round_mode=mode)
    fb = L.lrqmm_rsvd_ex(dB, amB, L.AXIS_COL, 8, r, p, q, seed=9, round_mode=mode)
    assert np.array_equal(to_np(L.lrqmm_gemm(Aq, amA, BqT, amB, 8, fa, fb)), C)


def _separate_calls(L, dA, dB, bits, r, p, q, seed):
    """The whole call as its parts: each operand quantized and factored by itself, then the product."""
    Aq, amA = L.lrqmm_quantize(dA, L.AXIS_ROW, bits)
    BqT, amB = L.lrqmm_quantize(dB, L.AXIS_COL, bits)
    fa = L.lrqmm_rsvd(dA, amA, L.AXIS_ROW, bits, r, p, q, seed=seed)
    fb = L.lrqmm_rsvd(dB, amB, L.AXIS_COL, bits, r, p, q, seed=seed)
    return L.lrqmm_gemm(Aq, amA, BqT, amB, bits, fa, fb)


@pytest.mark.parametrize("M,N,K,r,p", [(2700, 2600, 2500, 16, 8), (3300, 3300, 3300, 32, 8), (4096, 2001, 3900, 20, 8), (2000, 4096, 3955, 24, 8),
                                       (2000, 4096, 3956, 24, 8), (1999, 4096, 3900, 24, 8), (4097, 2100, 2000, 24, 8)])
def test_factorizations_together_and_in_two_chains(M, N, K, r, p):
    """Both sides of the limits between two chains and factorizations that advance together (sides from 2000 to 4096, 16.2 million elements an
    operand), with the product fused and early: the bits of the separate calls."""
    import torch
    import paper_2409_18772_amd as L
    gen = torch.Generator(device="cuda").manual_seed(7)
    dA, dB = (torch.empty(s, device="cuda").normal_(generator=gen) for s in ((M, K), (K, N)))
    say("together or two chains", M, N, K, r, p)
    C = to_np(L.lrqmm_matmul(dA, dB, 8, r, p, 1, seed=9))
    assert np.array_equal(to_np(_separate_calls(L, dA, dB, 8, r, p, 1, 9)), C)


@pytest.mark.parametrize("M,N,K,r,p", [(768, 4096, 4096, 16, 8), (769, 4096, 4096, 16, 8), (100, 4096, 4096, 32, 8), (65, 3300, 4096, 24, 0),
                                       (700, 3999, 3301, 64, 16), (768, 4097, 4000, 24, 8)])
def test_few_rows_beside_a_large_operand(M, N, K, r, p):
    """Both sides of the limit from which an A of few rows has a chain of its own, with the large operand's passes in either form."""
    test_factorizations_together_and_in_two_chains(M, N, K, r, p)


@pytest.mark.parametrize("M,N,K,r,p", [(2200, 600, 300, 20, 8), (300, 600, 2200, 17, 0), (2100, 300, 2500, 24, 8),
                                       (300, 2300, 700, 20, 0)])
def test_factors_do_not_depend_on_the_other_operand(M, N, K, r, p):
    """Sketches of 32 padded columns where one operand's tall factor has more than 2048 rows (the Gram kernel takes it in
    64-row tiles) and the other's has fewer (16-row tiles, the splits of a pass added in two runs), in one launch: the sums
    of each keep their own order, so the whole call gives the bits of the separate calls."""
    import paper_2409_18772_amd as L
    dA, dB = to_dev(wl.random_matrix("normal", M, K, seed=81)), to_dev(wl.random_matrix("uniform01", K, N, seed=82))
    say("one long factor", M, N, K, r, p)
    C = to_np(L.lrqmm_matmul(dA, dB, 8, r, p, 1, seed=9))
    assert np.array_equal(to_np(_separate_calls(L, dA, dB, 8, r, p, 1, 9)), C)


@pytest.mark.parametrize("M,N,K,r,p", [(640, 300, 512, 16, 8), (640, 300, 512, 32, 8), (640, 300, 512, 60, 12),
                                       (300, 640, 500, 16, 8), (300, 640, 500, 32, 8), (300, 640, 512, 32, 8),
                                       (300, 640, 512, 60, 12), (4096, 300, 1024, 60, 12)])
def test_guard_free_pass_kernels_equal_the_guarded_ones_bitwise(M, N, K, r, p):
    """A launch of a residual pass is guard-free when every operand in it has whole chunks and strips.  Beside a partner
    without them an operand of whole tiles takes the guarded form, by itself the guard-free one (A in the first three
    shapes, B's R.W in the next two, B's Rt.W in two more; in the last also four waves per workgroup in the pair, eight
    alone): same arithmetic in the same order, so the whole call gives the bits of the separate calls."""
    import paper_2409_18772_amd as L
    dA, dB = to_dev(wl.random_matrix("normal", M, K, seed=83)), to_dev(wl.random_matrix("uniform01", K, N, seed=84))
    say("guarded vs guard-free", M, N, K, r, p)
    C = to_np(L.lrqmm_matmul(dA, dB, 4, r, p, 1, seed=9))
    assert np.array_equal(to_np(_separate_calls(L, dA, dB, 4, r, p, 1, 9)), C)


# Codes travel packed inside the call, up to five bits in six.  Edges of the 32-row and 64-code blocks (one short, whole, one over), odd
# numbers of k blocks and fewer than the stages of the product, 128 x 128 / 64 x 128 / 64 x 64 / 256 x 256 tiles, tiles cut along K
# beside the SVDs, and both sides of the longest reduction of 5-bit codes in six bits (sums next to the limit: below).
PACKED = [(128, 96, 128, 4, 24, 8), (127, 97, 191, 4, 20, 8), (129, 160, 193, 2, 17, 0), (320, 321, 385, 5, 24, 8),
          (1025, 1000, 449, 3, 40, 8), (2080, 2049, 320, 4, 17, 0), (3100, 2900, 200, 4, 36, 0), (4096, 4096, 1024, 4, 32, 8),
          (64, 96, 65536, 5, 17, 0), (96, 64, 65540, 5, 17, 0)]
# Codes of six bits and more travel as bytes in the same blocks.
PACKED += [(127, 97, 191, 8, 20, 8), (129, 160, 193, 6, 17, 0), (33, 34, 35, 8, 17, 0), (320, 321, 385, 7, 24, 8), (1025, 1000, 449, 8, 40, 8),
           (1537, 1021, 1100, 8, 24, 8), (2080, 2049, 320, 8, 17, 0), (3100, 2900, 200, 8, 36, 0), (4096, 4096, 1024, 8, 32, 8),
           (64, 96, 131071, 8, 17, 0)]
# Tall operands, whose panels have a kernel of their own: one to three tiles of factor columns, one chunk of planes and more, both formats.
PACKED += [(49201, 40, 833, 8, 12, 8), (98310, 50, 200, 8, 40, 8), (32801, 40, 833, 8, 12, 8), (33000, 45, 321, 4, 20, 8), (65600, 60, 200, 8, 40, 8), (65537, 49, 130, 3, 33, 8),
           (40, 32802, 833, 4, 12, 8), (70, 49153, 321, 8, 41, 8)]


@pytest.mark.parametrize("M,N,K,bits,r,p", PACKED)
def test_packed_codes_give_the_bits_of_the_separate_calls(M, N, K, bits, r, p):
    """The separate calls quantize to bytes and multiply on the int8 matrix cores: integer sums are the same, and so are all
    roundings behind them."""
    import paper_2409_18772_amd as L
    dA, dB = to_dev(wl.random_matrix("normal", M, K, seed=91)), to_dev(wl.random_matrix("uniform_pm1", K, N, seed=92))
    say("packed codes", M, N, K, "bits", bits, r, p)
    C = to_np(L.lrqmm_matmul(dA, dB, bits, r, p, 1, seed=9))
    assert np.array_equal(to_np(_separate_calls(L, dA, dB, bits, r, p, 1, 9)), C)


def _amax_that_rounds_up(qmax):
    """A float32 maximum a with fl(a * fl(qmax / a)) > qmax: -a then has the code -(qmax + 1)."""
    a = np.linspace(1.0, 2.0, 4096, dtype=np.float32)
    return a[a * (np.float32(qmax) / a) > np.float32(qmax)][0]


# bits and the longest reduction that travels in six bits, K 4^(bits - 1) = 2^24.
@pytest.mark.parametrize("M,N,bits,K", [(64, 96, 5, 65536), (70, 33, 4, 262144), (33, 40, 3, 1048576), (256, 300, 5, 65536)])
@pytest.mark.parametrize("turn", [False, True])
def test_six_bit_sums_next_to_their_limit(M, N, bits, K, turn):
    """Codes -(qmax + 1), one in sixteen a smaller one at irregular places: sums up to 2^24 in units of one product, odd ones among
    them, where float32 ends to hold every integer.  turn: the second half of the reduction has the other sign, so that the
    partial sums pass half of it.  Against the int8 product of the separate calls, bit for bit, and its sums against int64 on the
    CPU in one row."""
    import torch
    import paper_2409_18772_amd as L
    qmax = 2 ** (bits - 1) - 1
    a = float(_amax_that_rounds_up(qmax))

    def operand(rows, cols, seed, kdim):
        gen = torch.Generator(device="cuda").manual_seed(seed)
        u = torch.rand((rows, cols), generator=gen, device="cuda")
        x = torch.where(u < 1 / 16, torch.full_like(u, -0.97 * a), torch.full_like(u, -a))
        if turn and kdim is not None:
            x.narrow(kdim, K // 2, K - K // 2).neg_()
        return x
    dA, dB = operand(M, K, 1, 1), operand(K, N, 2, None)
    say("six-bit sums", M, N, K, bits, "turn", turn)
    Aq, amA = L.lrqmm_quantize(dA, L.AXIS_ROW, bits)
    BqT, amB = L.lrqmm_quantize(dB, L.AXIS_COL, bits)
    ws = L.Workspace.for_problem(M, N, K, 17, 0)
    fa = L.lrqmm_rsvd(dA, amA, L.AXIS_ROW, bits, 17, 0, 0, seed=9, workspace=ws)
    fb = L.lrqmm_rsvd(dB, amB, L.AXIS_COL, bits, 17, 0, 0, seed=9, workspace=ws)
    want, Cint = L.lrqmm_gemm(Aq, amA, BqT, amB, bits, fa, fb, want_cint=True, workspace=ws)
    assert int(Aq.min()) == -qmax - 1 and int(BqT.min()) == -qmax - 1
    half = K // 2 if turn else K
    largest = (Aq[:, :half].float() @ BqT[:, :half].float().T).abs().max()
    assert float(largest) > (2 ** 22 if turn else 2 ** 23) and bool((Cint % 2 != 0).any())
    row = np.asarray(to_np(Aq)[0], np.int64) @ np.asarray(to_np(BqT), np.int64).T
    assert np.array_equal(row, to_np(Cint)[0])
    assert torch.equal(L.lrqmm_matmul(dA, dB, bits, 17, 0, 0, seed=9, workspace=ws), want)


# The same without a factorization: rows in the registers of a wave or (beyond 4096 codes) of a workgroup, in one to four loads, rows
# that end inside a load, 16-row groups that end early.
@pytest.mark.parametrize("M,N,K,bits", [(256, 256, 64, 4), (131, 97, 193, 4), (65, 100, 1030, 5), (300, 130, 4096, 2), (70, 64, 4099, 4),
                                        (97, 300, 9001, 4), (2100, 2300, 700, 4), (256, 256, 64, 8), (131, 97, 193, 8),
                                        (5, 4, 4, 8), (65, 100, 1030, 6), (70, 64, 4099, 8), (97, 300, 9001, 8), (2100, 2300, 700, 8)] +
                         # more than 512 tiles of 128 x 128: the 256 x 256 tiles that store the product themselves, ragged and whole
                         [(3100, 2901, 200, 4), (4096, 4096, 320, 4), (3100, 2901, 200, 8), (4096, 4096, 320, 8)] +
                         # tall operands on both sides of the limits up to which their rows stay bytes
                         [(16383, 33, 65, 8), (16385, 33, 65, 8), (16390, 768, 40, 8), (16390, 769, 40, 8), (16391, 20, 512, 8),
                          (16391, 20, 513, 8), (16390, 512, 40, 4), (16390, 513, 40, 4), (16391, 20, 384, 4), (16391, 20, 385, 4),
                          (16391, 20, 516, 8), (16391, 20, 388, 4), (16390, 12, 15, 8), (65536, 17, 383, 8), (65537, 64, 129, 4), (65537, 65, 129, 4),
                          (3071, 30, 4100, 8), (3073, 64, 4100, 8), (3073, 385, 4100, 4), (3073, 256, 8196, 8), (3073, 257, 8196, 8), (3073, 65, 8196, 4), (16385, 33, 4097, 8)])
def test_packed_codes_without_a_factorization(M, N, K, bits):
    import paper_2409_18772_amd as L
    dA, dB = to_dev(wl.random_matrix("normal", M, K, seed=93)), to_dev(wl.random_matrix("uniform_pm1", K, N, seed=94))
    say("packed codes, rank 0", M, N, K, "bits", bits)
    C = to_np(L.lrqmm_matmul(dA, dB, bits, 0))
    Aq, amA = L.lrqmm_quantize(dA, L.AXIS_ROW, bits)
    BqT, amB = L.lrqmm_quantize(dB, L.AXIS_COL, bits)
    assert np.array_equal(to_np(L.lrqmm_gemm(Aq, amA, BqT, amB, bits)), C)


# Extents below one 16-byte load (four values), one operand at a time and together: N < 4 against long rows of A, K < 4
# against wide rows of B, both, M < 4; the last shape has enough elements for the two-stream schedule.
TINY_EXTENTS = [(100, 1, 300, 1), (70, 3, 517, 3), (100, 2, 1000, 1), (90, 200, 3, 2), (100, 100, 3, 1), (300, 2, 1, 1),
                (5, 3, 2, 2), (2, 300, 300, 2), (3, 5, 4, 3), (4500, 3, 3000, 2)]


@pytest.mark.parametrize("tensor", [False, True])
@pytest.mark.parametrize("M,N,K,r", TINY_EXTENTS)
def test_extents_below_one_load(M, N, K, r, tensor):
    """Group maxima, codes and both factorizations where an extent is smaller than a load: against the oracle, and against
    the separate calls, whose quantizers are kernels of their own (a wrong maximum anywhere in an operand moves C by the
    size of its terms; at ranks this small the two differ by float32 roundings of the sketch products)."""
    import torch
    import paper_2409_18772_amd as L
    A, B = wl.random_matrix("normal", M, K, seed=71), wl.random_matrix("normal", K, N, seed=72)
    dA, dB = to_dev(A), to_dev(B)
    sm = L.SCALE_TENSOR if tensor else L.SCALE_VECTOR
    say("tiny extents", M, N, K, "rank", r, "tensor", tensor)
    D = torch.empty((M, N), dtype=torch.float32, device="cuda")
    C = to_np(L.lrqmm_matmul_ex(dA, dB, D, 8, r, 0, 1, seed=9, scale_mode=sm))
    ref = o.lrqmm(A, B, 8, r, 0, 1, seed=9, per_tensor=tensor)
    d = rel_fro(ref["C"], C)
    say("gpu vs oracle", d, "tol", tol_for(ref))
    assert d < tol_for(ref)
    check_elementwise(C, ref, r, what=f"tiny extents {M}x{N}x{K}")
    Aq, amA = L.lrqmm_quantize_ex(dA, L.AXIS_ROW, 8, o.FLOOR, sm)
    BqT, amB = L.lrqmm_quantize_ex(dB, L.AXIS_COL, 8, o.FLOOR, sm)
    assert np.array_equal(to_np(Aq), ref["Aq"]) and np.array_equal(to_np(BqT), ref["Bq"].T)
    fa = L.lrqmm_rsvd_ex(dA, amA, L.AXIS_ROW, 8, r, 0, 1, seed=9)
    fb = L.lrqmm_rsvd_ex(dB, amB, L.AXIS_COL, 8, r, 0, 1, seed=9)
    assert rel_fro(to_np(L.lrqmm_gemm(Aq, amA, BqT, amB, 8, fa, fb)), C) < 2 * tol_for(ref)


# M, N, K, rank, power_iters: no oversampling and up to 16 columns.  Column counts around the 16 of a workgroup of the
# final kernel, splits of the last pass from 1 to 64, the narrowest and widest such sketch, both schedules.
UNTRUNCATED = [(40, 33, 16, 1, 0), (130, 97, 79, 16, 1), (65, 64, 31, 15, 2), (700, 17, 1030, 7, 1), (9000, 18, 33, 16, 0),
               (8200, 129, 575, 9, 0), (9000, 40, 1500, 3, 0)]


@pytest.mark.parametrize("dist", ["uniform01", "normal", "low_rank"])
@pytest.mark.parametrize("M,N,K,r,q", UNTRUNCATED)
def test_untruncated_narrow_sketch(M, N, K, r, q, dist):
    """rank == sketch width <= 16: the call forms Q (Q^T R) without the small SVD; the oracle and the separate calls form
    U diag(Sigma) Vt of the same matrix.  low_rank: a residual of rank 1 (A constant: its codes leave one value per row and
    the maxima's entries zero), so that most columns of Q are dropped.  Frobenius only: the element-wise budget counts the
    2r + 1 terms of an entry, and at ranks this small the rounding of the length-K panel sums is the larger part (with or
    without the SVD)."""
    import paper_2409_18772_amd as L
    if dist == "low_rank":
        A = np.full((M, K), 0.3, dtype=np.float32) * (1 + np.arange(M, dtype=np.float32)[:, None] % 3)
        A[:, 0] = 1.0
        B = np.full((K, N), 0.7, dtype=np.float32)
        B[0] = 1.0
    else:
        A, B = wl.random_matrix(dist, M, K, seed=91), wl.random_matrix(dist, K, N, seed=92)
    dA, dB = to_dev(A), to_dev(B)
    say("untruncated", M, N, K, "rank", r, "q", q, dist)
    C = to_np(L.lrqmm_matmul(dA, dB, 8, r, 0, q, seed=9))
    ref = o.lrqmm(A, B, 8, r, 0, q, seed=9)
    d = rel_fro(ref["C"], C)
    say("gpu vs oracle", d, "tol", tol_for(ref))
    assert d < tol_for(ref)
    assert rel_fro(to_np(_separate_calls(L, dA, dB, 8, r, 0, q, 9)), C) < 2 * tol_for(ref)


@pytest.mark.parametrize("big,small", [((359, 2053, 1604), (288, 2053, 1604)), ((228, 691, 3550), (224, 691, 3550)),
                                       ((1030, 700, 2100), (1000, 640, 256))])
def test_smaller_call_in_a_larger_call_s_workspace(big, small):
    """One workspace, exactly the size reported for the larger problem, serves both, with the bits of a workspace of their
    own (rank 16, no oversampling; and the layer form's factorization in it)."""
    import torch
    import paper_2409_18772_amd as L
    ws = L.Workspace(L.lrqmm_workspace_bytes(*big, 16, 0))
    for M, N, K in (big, small):
        A, B = to_dev(wl.random_matrix("normal", M, K, seed=61)), to_dev(wl.random_matrix("normal", K, N, seed=62))
        say("shared workspace", M, N, K)
        assert torch.equal(L.lrqmm_matmul(A, B, 8, 16, 0, 1, seed=4, workspace=ws), L.lrqmm_matmul(A, B, 8, 16, 0, 1, seed=4))
        _, amax = L.lrqmm_quantize(A, L.AXIS_ROW, 8)
        for x, y in zip(L.lrqmm_rsvd(A, amax, 0, 8, 16, 0, 1, seed=4, workspace=ws), L.lrqmm_rsvd(A, amax, 0, 8, 16, 0, 1, seed=4)):
            assert torch.equal(x, y)


FULL = ["c2_4096_int8_r16", "c3_4096_int4_r32_outliers"]


@pytest.mark.parametrize("name", FULL)
def test_full_size_sampled_rows(name):
    """Full-size run in the benchmark's launch configuration, checked on sampled rows of C."""
    w = wl.CONFIGS[name]
    A, B = wl.make_inputs(w)
    say("matmul full", w.name)
    C = _run_gpu(w, A, B)
    rows = np.random.default_rng(5).choice(w.M, size=24, replace=False)
    say("oracle on", len(rows), "rows")
    ref = o.lrqmm(A, B, w.bits, w.rank, w.oversample, w.power_iters, seed=w.sketch_seed, row_sample=rows,
                  want_cint=False)
    d = rel_fro(ref["C"], C[rows])
    say(name, "gpu vs oracle", d, "tol", tol_for(ref))
    assert d < tol_for(ref)
    check_elementwise(C[rows], ref, w.rank, rows, what=name)
    exact = o.exact_product(A[rows], B)
    e_lr, e_dq = o.rel_err(exact, C[rows]), o.rel_err(exact, ref["C0"])
    say(name, "err lrqmm", e_lr, "err direct quant", e_dq)
    assert e_lr < e_dq
    if "int4" in name:
        assert e_dq / e_lr >= 10.0        # the headline claim on the outlier workload


@pytest.mark.parametrize("oversample,power_iters", [(0, 0), (8, 1)])
def test_resnet_conv_shape_sampled_rows(oversample, power_iters):
    """The conv-shaped workload at full size (100352 x 64 x 576), with the configured sketch (no oversampling, no
    power iteration) and with the alternative setting p = 8, q = 1."""
    import paper_2409_18772_amd as L
    w = wl.CONFIGS["c5_resnet50_conv_int4_r8"]
    A, B = wl.make_inputs(w)
    say("matmul full", w.name, "p", oversample, "q", power_iters)
    C = to_np(L.lrqmm_matmul(to_dev(A), to_dev(B), w.bits, w.rank, oversample, power_iters, seed=w.sketch_seed))
    rows = np.random.default_rng(6).choice(w.M, size=512, replace=False)
    ref = o.lrqmm(A, B, w.bits, w.rank, oversample, power_iters, seed=w.sketch_seed, row_sample=rows,
                  want_cint=False)
    d = rel_fro(ref["C"], C[rows])
    say(w.name, "gpu vs oracle", d, "tol", tol_for(ref))
    if (oversample, power_iters) == (0, 0):
        assert d < tol_for(ref)
        check_elementwise(C[rows], ref, w.rank, rows, what=w.name)
        return
    # With p = 8, q = 1 the cut at r = 8 falls between two singular values of R_A that agree to 0.13 %
    # (test_rsvd_truncation_between_nearly_equal_singular_values in test_gpu_rsvd_gemm.py): the rank-8 part is
    # then fixed only to ~2e-4 of its norm at float32 resolution, and C inherits that through the compensation.
    # What is unique is compared tightly -- the error against the exact product, which must equal the
    # oracle's -- and the distance itself against the factorization's own tolerance carried to C.
    exact = o.exact_product(A[rows], B)
    e_gpu, e_ref = o.rel_err(exact, C[rows]), o.rel_err(exact, ref["C"])
    comp = np.linalg.norm(ref["C"] - ref["C0"]) / np.linalg.norm(ref["C"])
    say(w.name, "err vs exact: gpu", e_gpu, "oracle", e_ref, "compensation / C", comp)
    assert abs(e_gpu - e_ref) <= 1e-4 * e_ref
    assert d < tol_for(ref) + 2 * 2e-4 * comp


# Rows of C checked against the oracle at 16384^3.  The 64 x 64 grid of 256 x 256 tiles is dealt to the 8 XCDs as
# rectangles of 32 x 16 tiles, each worked through in 16 rounds of 32 tiles; tile rows 31 and 63 (rows 7936-8191
# and 16128-16383) are the last rows of the two bands of rectangles, i.e. tiles of the last round, next to the
# band boundary.  The sample takes three rows from each and eight drawn at random.  (At this size the early
# product is not cut along K: that happens only below four rounds, and is covered at 4096^3.)
C4_ROWS = np.concatenate([[7936, 8050, 8191, 16128, 16250, 16383],
                          np.random.default_rng(7).choice(16384, size=8, replace=False)])


def test_largest_config_oracle_rows():
    """c4 (16384^3, int4, r = 64, l = 80, two power iterations) at full size, in the benchmark's launch
    configuration, against the oracle: both residual factorizations in full, C on sampled rows (rows of C
    are independent given the factors)."""
    import torch
    import paper_2409_18772_amd as L
    w = wl.CONFIGS["c4_16384_int4_r64"]
    say("inputs", w.name)
    A, B = wl.make_inputs(w)
    dA, dB = to_dev(A), to_dev(B)
    ws = L.Workspace.for_problem(w.M, w.N, w.K, w.rank, w.oversample)
    say("matmul full", w.name)
    C = L.lrqmm_matmul(dA, dB, w.bits, w.rank, w.oversample, w.power_iters, seed=w.sketch_seed, workspace=ws)
    rows = np.sort(C4_ROWS)
    Cr = C[torch.from_numpy(rows).cuda()].cpu().numpy()
    del C, dA, dB, ws
    torch.cuda.empty_cache()
    say("oracle: factorizations in full, C on", len(rows), "rows")
    ref = o.lrqmm(A, B, w.bits, w.rank, w.oversample, w.power_iters, seed=w.sketch_seed, row_sample=rows,
                  want_cint=False)
    d = rel_fro(ref["C"], Cr)
    say(w.name, "gpu vs oracle", d, "tol", tol_for(ref))
    assert d < tol_for(ref)
    check_elementwise(Cr, ref, w.rank, rows, what=w.name)
    exact = o.exact_product(A[rows], B)
    e_lr, e_dq = o.rel_err(exact, Cr), o.rel_err(exact, ref["C0"])
    say(w.name, "err lrqmm", e_lr, "err direct quant", e_dq)
    # against floor rounding, the quantizer of the method (Eq. (get_ra2)); against round-to-nearest direct
    # quantization of zero-mean data the two errors are about equal
    assert e_lr * 10.0 < e_dq


RAGGED_LARGE = [
    # shapes on the 256 x 256 tile kernel that are no multiples of its tile: guarded loads, guarded
    # epilogue, clamped rows and columns of the rank update
    (4100, 2052, 528),      # K % 16 == 0: 16-byte operand loads with guards
    (4100, 2052, 500),      # byte-wise operand loads
]


@pytest.mark.parametrize("M,N,K", RAGGED_LARGE)
@pytest.mark.parametrize("fused", [False, True])
def test_ragged_large_tile_shapes(M, N, K, fused):
    """fused = False: beta = 0 and a dense D, the schedule with the early integer product and the rank
    update as a kernel of its own; fused = True: a strided D with beta != 0, the GEMM with the fused
    epilogue.  Oracle on sampled rows, including the last (partial) tile row."""
    import torch
    import paper_2409_18772_amd as L
    bits, r, p, q = 4, 28, 4, 1      # a sketch of 32 columns: the width from which the early-product schedule is used
    A = wl.random_matrix("normal", M, K, seed=41)
    B = wl.random_matrix("uniform01", K, N, seed=42)
    rows = np.sort(np.concatenate([[0, 255, 256, 4095, 4096, M - 1],
                                   np.random.default_rng(8).choice(M, size=10, replace=False)]))
    say("ragged large tiles", M, N, K, "fused" if fused else "early product")
    ref = o.lrqmm(A, B, bits, r, p, q, seed=11, row_sample=rows, want_cint=False)
    if not fused:
        C = to_np(L.lrqmm_matmul(to_dev(A), to_dev(B), bits, r, p, q, seed=11))
        d = rel_fro(ref["C"], C[rows])
        say("gpu vs oracle", d, "tol", tol_for(ref))
        assert d < tol_for(ref)
        check_elementwise(C[rows], ref, r, rows, what="ragged early")
        return
    alpha, beta = 1.5, -0.5
    D0 = wl.random_matrix("normal", M, N, seed=43)
    big = torch.full((M, N + 3), -7.0, dtype=torch.float32, device="cuda")
    dD = big[:, :N]
    dD.copy_(torch.from_numpy(D0))
    L.lrqmm_matmul_ex(to_dev(A), to_dev(B), dD, bits, r, p, q, seed=11, alpha=alpha, beta=beta)
    got = to_np(dD)[rows].astype(np.float64)
    want = o.scaled_update(ref["C"], alpha, beta, D0[rows])
    # the update of the plain product: |alpha| times its error plus three roundings (see test_gpu_update_strides.py)
    nc, nd = np.linalg.norm(ref["C"]), np.linalg.norm(D0[rows])
    bound = abs(alpha) * tol_for(ref) * nc + 3 * 2.0 ** -24 * (abs(alpha) * nc + abs(beta) * nd)
    err = np.linalg.norm(got - want)
    say("gpu vs oracle", err, "bound", bound)
    assert err < bound
    # element-wise: the product's budget scaled by |alpha| plus the three roundings of the update
    from gpu_util import elementwise_budget
    budget, _ = elementwise_budget(ref, r, rows)
    lim = abs(alpha) * budget + 3 * 2.0 ** -24 * (abs(alpha) * np.abs(ref["C"]) + abs(beta) * np.abs(D0[rows]))
    assert np.all(np.abs(got - want) <= lim)
    assert np.all(to_np(big)[:, N:] == -7.0)


def test_wide_panels_large_tiles_sampled_rows():
    """Rank 64 on the large-tile schedule (early integer product, rank update as its own kernel): panels of
    2r = 128 columns take the update kernel that forms the panel products from bfloat16 planes.  Oracle on
    sampled rows, Frobenius and element-wise."""
    import paper_2409_18772_amd as L
    M, N, K, bits, r, p, q = 4096, 2048, 512, 4, 64, 16, 1
    A = wl.random_matrix("normal", M, K, seed=61)
    B = wl.random_matrix("normal", K, N, seed=62)
    rows = np.sort(np.random.default_rng(9).choice(M, size=16, replace=False))
    say("wide panels", M, N, K, r)
    C = to_np(L.lrqmm_matmul(to_dev(A), to_dev(B), bits, r, p, q, seed=13))
    ref = o.lrqmm(A, B, bits, r, p, q, seed=13, row_sample=rows, want_cint=False)
    d = rel_fro(ref["C"], C[rows])
    say("gpu vs oracle", d, "tol", tol_for(ref))
    assert d < tol_for(ref)
    check_elementwise(C[rows], ref, r, rows, what="wide panels")


def test_three_stream_schedule_is_repeatable():
    """The two factorization chains, the early integer product on the third stream and the K-cut tiles involve
    no atomics on floating-point data and no order that depends on timing: 300 calls at the headline shape,
    with other calls through the same workspace in between, all give the first call's bits.  (A missing event
    wait between the three streams would show up here as an occasional difference.)"""
    import torch
    import paper_2409_18772_amd as L
    w = wl.CONFIGS["c3_4096_int4_r32_outliers"]
    A, B = wl.make_inputs(w)
    dA, dB = to_dev(A), to_dev(B)
    ws = L.Workspace.for_problem(w.M, w.N, w.K, w.rank, w.oversample)
    C = torch.empty((w.M, w.N), dtype=torch.float32, device="cuda")
    first, differing = None, 0
    for it in range(300):
        L.lrqmm_matmul(dA, dB, w.bits, w.rank, w.oversample, w.power_iters, seed=w.sketch_seed, workspace=ws, C=C)
        if first is None:
            first = C.clone()
        elif not torch.equal(first, C):
            differing += 1
        if it % 7 == 3:     # a direct-quantization call and another sketch seed through the same workspace
            L.lrqmm_matmul(dA, dB, w.bits, 0, workspace=ws, C=C)
            L.lrqmm_matmul(dA, dB, w.bits, w.rank, w.oversample, w.power_iters, seed=it, workspace=ws, C=C)
    say("calls differing from the first:", differing)
    assert differing == 0


def test_call_is_ordered_like_one_stream_on_a_caller_stream():
    """On a caller's stream the call must wait for earlier work of that stream (its operands may still be in
    the making) and later work of that stream must see its result, although two library streams do part of it:
    the operands are produced by kernels enqueued on the stream right before the call, the result is copied on
    the stream right after it, nothing is synchronized in between, and the copy must equal the result of the
    same call on settled inputs, bit for bit."""
    import torch
    import paper_2409_18772_amd as L
    w = wl.CONFIGS["c3_4096_int4_r32_outliers"]
    A, B = wl.make_inputs(w)
    dA, dB = to_dev(A), to_dev(B)
    ws = L.Workspace.for_problem(w.M, w.N, w.K, w.rank, w.oversample)
    want = L.lrqmm_matmul(dA, dB, w.bits, w.rank, w.oversample, w.power_iters, seed=w.sketch_seed, workspace=ws).clone()
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    A2, B2 = torch.empty_like(dA), torch.empty_like(dB)
    C = torch.empty((w.M, w.N), dtype=torch.float32, device="cuda")
    with torch.cuda.stream(s):
        for _ in range(3):
            # operands rebuilt on the stream just before the call (x * 0.5 + x * 0.5 is exact in binary)
            torch.add(dA * 0.5, dA * 0.5, out=A2)
            torch.add(dB * 0.5, dB * 0.5, out=B2)
            L.lrqmm_matmul(A2, B2, w.bits, w.rank, w.oversample, w.power_iters, seed=w.sketch_seed, workspace=ws, C=C)
            got = C.clone()             # consumer on the same stream
            A2.zero_(); B2.zero_()      # and the operands are destroyed right behind the call
        s.synchronize()
    assert torch.equal(got, want)


def test_empty_reduction_reads_no_operand():
    """K = 0 with M, N > 0: C_F = 0, so D <- beta D (zeros when beta = 0); the GEMM kernels are not
    launched at all (they load their first operand tile unconditionally)."""
    import torch
    import paper_2409_18772_amd as L
    M, N = 300, 260
    A = torch.empty((M, 0), dtype=torch.float32, device="cuda")
    B = torch.empty((0, N), dtype=torch.float32, device="cuda")
    say("K = 0: matmul")
    C = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    L.lrqmm_matmul(A, B, 8, 0, C=C)
    assert torch.all(C == 0)
    D0 = wl.random_matrix("normal", M, N, seed=3)
    D = to_dev(D0)
    L.lrqmm_matmul_ex(A, B, D, 4, 0, alpha=2.0, beta=-1.5)
    assert np.array_equal(to_np(D), np.float32(-1.5) * D0)
    say("K = 0: gemm")
    Aq = torch.empty((M, 0), dtype=torch.int8, device="cuda")
    BqT = torch.empty((N, 0), dtype=torch.int8, device="cuda")
    am, an = torch.ones(M, device="cuda"), torch.ones(N, device="cuda")
    C2, Cint = L.lrqmm_gemm(Aq, am, BqT, an, 8, want_cint=True)
    assert torch.all(C2 == 0) and torch.all(Cint == 0)
    say("K = 0: residual_matmul")
    D = to_dev(D0)
    L.lrqmm_residual_matmul(A, B, D, 4, 4, alpha=1.0, beta=1.0)
    assert np.array_equal(to_np(D), D0)
    # large enough for the 256 x 256 tile kernel's dispatch
    M, N = 4096, 2048
    C = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    L.lrqmm_matmul(torch.empty((M, 0), dtype=torch.float32, device="cuda"),
                   torch.empty((0, N), dtype=torch.float32, device="cuda"), 4, 0, C=C)
    assert torch.all(C == 0)


def test_largest_config_properties():
    """c4 (16384^3, l = 80, two power iterations) at full size, properties beside the oracle comparison
    above: finite output, bit-identical repeat, and on sampled rows an error against the exact float64
    product far below that of direct (floor) quantization computed by the same library."""
    import torch
    import paper_2409_18772_amd as L
    w = wl.CONFIGS["c4_16384_int4_r64"]
    say("inputs", w.name)
    A, B = wl.make_inputs(w)
    dA, dB = to_dev(A), to_dev(B)
    ws = L.Workspace.for_problem(w.M, w.N, w.K, w.rank, w.oversample)
    say("matmul full", w.name)
    C = L.lrqmm_matmul(dA, dB, w.bits, w.rank, w.oversample, w.power_iters, seed=w.sketch_seed, workspace=ws)
    rows = np.random.default_rng(7).choice(w.M, size=12, replace=False)
    ridx = torch.from_numpy(rows).cuda()
    Cr = C[ridx].cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(Cr))
    C2 = L.lrqmm_matmul(dA, dB, w.bits, w.rank, w.oversample, w.power_iters, seed=w.sketch_seed, workspace=ws)
    assert torch.equal(C, C2)
    del C2
    C0 = L.lrqmm_matmul(dA, dB, w.bits, 0, workspace=ws)
    C0r = C0[ridx].cpu().numpy().astype(np.float64)
    say("exact product on", len(rows), "rows")
    exact = A[rows].astype(np.float64) @ B.astype(np.float64)
    e_lr, e_dq = o.rel_err(exact, Cr), o.rel_err(exact, C0r)
    say(w.name, "err lrqmm", e_lr, "err direct quant", e_dq)
    assert e_lr * 10.0 < e_dq


@pytest.mark.parametrize("shape", [(4096, 2048, 512, 28, 4, 1), (300, 200, 260, 28, 4, 1), (3000, 64, 576, 8, 0, 0),
                                   (8300, 64, 576, 8, 0, 0), (4096, 1024, 3000, 16, 8, 0), (4096, 2100, 3000, 28, 4, 0)])
def test_call_can_be_captured_in_a_graph(shape):
    """The call only enqueues kernels and event waits (its clears are fill kernels), so it may be recorded
    into a HIP graph, side streams included; every replay must reproduce the eager result, with eager work
    and synchronizations between the replays.  First shape: both factorizations on the caller's stream, the integer product
    on another (sketch of 32 columns, large-tile kernel); second: one stream; third and fourth: short rows of A in one stream;
    fifth: two chains; sixth: one stream and the early product."""
    import torch
    import paper_2409_18772_amd as L
    M, N, K, r, p, q = shape
    A = to_dev(wl.random_matrix("normal", M, K, seed=31))
    B = to_dev(wl.random_matrix("normal", K, N, seed=32))
    ws = L.Workspace.for_problem(M, N, K, r, p)
    C = torch.empty((M, N), dtype=torch.float32, device="cuda")

    def step():
        L.lrqmm_matmul(A, B, 4, r, p, q, seed=7, workspace=ws, C=C)

    step()
    torch.cuda.synchronize()
    ref = C.clone()
    say("capture", shape)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        step()                       # first use of the library's streams and events outside the capture
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        step()
    torch.cuda.synchronize()
    for i in range(3):
        C.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(C, ref), i
        step()                       # eager work between replays
        torch.cuda.synchronize()
        assert torch.equal(C, ref), i


@pytest.mark.parametrize("shape", [(33000, 64, 576, 8, 0, 0), (33000, 64, 576, 8, 4, 0), (5000, 2100, 3000, 28, 4, 0)])
def test_calls_on_several_streams_can_be_captured(shape):
    """The same for the kernels that read a tall A once, B's chain on the side stream, and for two chains with the early product."""
    test_call_can_be_captured_in_a_graph(shape)


def test_captured_call_judges_the_operand_of_each_replay():
    """Whether R^T Q is formed again is decided on the device: a captured call follows the values that A holds when it is replayed."""
    import torch
    import paper_2409_18772_amd as L
    M, N, K, r = 33000, 40, 576, 8
    kinds = [torch.from_numpy(_tall_operand(k, M, K)).cuda() for k in ("scaled 1", "factor 1e-4", "scaled 1e19")]
    B = to_dev(wl.random_matrix("normal", K, N, seed=32))
    ws = L.Workspace.for_problem(M, N, K, r, 0)
    A, C = kinds[0].clone(), torch.empty((M, N), dtype=torch.float32, device="cuda")
    refs = [L.lrqmm_matmul(x, B, 4, r, seed=7, workspace=ws).clone() for x in kinds]
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        L.lrqmm_matmul(A, B, 4, r, seed=7, workspace=ws, C=C)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        L.lrqmm_matmul(A, B, 4, r, seed=7, workspace=ws, C=C)
    torch.cuda.synchronize()
    for i in (0, 1, 0, 2, 1, 0):
        A.copy_(kinds[i])
        C.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(C, refs[i]), i


def test_capture_with_profiling_on_is_refused():
    """Timing events do not belong in a graph: a call under stream capture with stage timing enabled
    returns LRQMM_ERR_UNSUPPORTED before it enqueues anything, and the capture stays valid (empty)."""
    import torch
    import paper_2409_18772_amd as L
    M, N, K = 300, 200, 260
    A = to_dev(wl.random_matrix("normal", M, K, seed=31))
    B = to_dev(wl.random_matrix("normal", K, N, seed=32))
    ws = L.Workspace.for_problem(M, N, K, 28, 4)
    C = torch.empty((M, N), dtype=torch.float32, device="cuda")
    L.lrqmm_matmul(A, B, 4, 28, 4, 1, seed=7, workspace=ws, C=C)      # library streams exist from here on
    torch.cuda.synchronize()
    ref = C.clone()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    tmp = torch.ones(16, device="cuda")
    L.lrqmm_profile_enable(True)
    status = None
    try:
        with torch.cuda.graph(g, stream=s):
            tmp.zero_()                  # (the graph is not empty)
            try:
                L.lrqmm_matmul(A, B, 4, 28, 4, 1, seed=7, workspace=ws, C=C)
            except L.LrqmmError as e:
                status = e.status
    finally:
        L.lrqmm_profile_enable(False)
    torch.cuda.synchronize()
    assert status == -2
    L.lrqmm_matmul(A, B, 4, 28, 4, 1, seed=7, workspace=ws, C=C)      # the library still works
    torch.cuda.synchronize()
    assert torch.equal(C, ref)


def test_gemm_only_profiling_mode():
    import torch
    import paper_2409_18772_amd as L
    M, N, K = 4096, 2048, 512
    A = to_dev(wl.random_matrix("normal", M, K, seed=33))
    B = to_dev(wl.random_matrix("normal", K, N, seed=34))
    ws = L.Workspace.for_problem(M, N, K, 28, 4)
    L.lrqmm_profile_enable(L.PROF_GEMM_ONLY)
    try:
        for _ in range(3):
            L.lrqmm_matmul(A, B, 4, 28, 4, 1, workspace=ws)         # early product: stage int_gemm
        torch.cuda.synchronize()
        st, n = L.lrqmm_profile_read()
        assert n == 3 and st["int_gemm"] > 0 and st["gemm"] == 0 and st["rsvd_a"] == 0
        L.lrqmm_matmul(A, B, 4, 0, workspace=ws)                    # rank 0: fused kernel, stage gemm
        torch.cuda.synchronize()
        st, n = L.lrqmm_profile_read()
        assert n == 1 and st["gemm"] > 0 and st["int_gemm"] == 0
    finally:
        L.lrqmm_profile_enable(False)


# Panels prepared straight from the last products (sketches of up to 16 columns without oversampling, K up to 2048) and, from one k block
# more on, through the factors: both sides of the limit, k blocks and columns that end early, one k block and none whole, one chain
# and two (the last shape), few and many ranges of the last product.  The oracle forms the SVD.
@pytest.mark.parametrize("M,N,K,bits,r,q", [(40, 33, 17, 8, 1, 0), (65, 63, 64, 8, 16, 1), (130, 70, 65, 4, 5, 0), (300, 260, 1000, 8, 10, 1),
                                            (90, 515, 1025, 8, 16, 1), (260, 130, 2048, 8, 9, 1), (260, 130, 2049, 8, 9, 1), (9000, 40, 300, 8, 8, 1),
                                            (6700, 40, 2000, 8, 10, 1)])
def test_panels_from_the_last_products(M, N, K, bits, r, q):
    import paper_2409_18772_amd as L
    A, B = wl.random_matrix("uniform01", M, K, seed=95), wl.random_matrix("uniform01", K, N, seed=96)
    say("panels from the last products", M, N, K, bits, r, q)
    C = to_np(L.lrqmm_matmul(to_dev(A), to_dev(B), bits, r, 0, q, seed=7))
    ref = o.lrqmm(A, B, bits, r, 0, q, seed=7)
    assert rel_fro(ref["C"], C) < tol_for(ref)


# Column maxima by strips over all rows (up to 512) and by slabs (from 513): columns at the edges of the 64-column strips, of the
# 256-column slabs and below one load; the separate calls' quantizer has kernels of its own.
@pytest.mark.parametrize("K", [17, 127, 129, 512, 513])
@pytest.mark.parametrize("N", [17, 63, 64, 66, 257])
def test_column_maxima_in_strips_and_slabs(N, K):
    import paper_2409_18772_amd as L
    dA, dB = to_dev(wl.random_matrix("normal", 90, K, seed=97)), to_dev(wl.random_matrix("normal", K, N, seed=98))
    say("column maxima", N, K)
    C = to_np(L.lrqmm_matmul(dA, dB, 8, 17, 0, 1, seed=9))
    assert np.array_equal(to_np(_separate_calls(L, dA, dB, 8, 17, 0, 1, 9)), C)
