// Internal launch functions of the LRQMM library (one per step of the hot path).
// All pointers are device pointers; every function only enqueues work on `st`
// and returns LRQMM_OK or LRQMM_ERR_HIP.
#pragma once
#include "common.h"
#include "../../include/lrqmm.h"

// ---- quantize.hip -------------------------------------------------------
// X is rows x cols with row stride ldx (>= cols).  per_tensor: one scale for the whole matrix,
// i.e. every entry of amax holds the global maximum.  amax0 != null: quantize the residual of a
// first quantization whose group maxima are amax0 (second level of Eq. (gemm_r_split)).
int launch_quantize_rows(const float* X, int ldx, int rows, int cols, QuantParams q, bool per_tensor,
                         const float* amax0, int8_t* codes, float* amax, hipStream_t st);
int launch_quantize_cols(const float* X, int ldx, int rows, int cols, QuantParams q, bool per_tensor,
                         const float* amax0, int8_t* codesT, float* amax, hipStream_t st);
// Both operands of a product, one scale per row of A and per column of B: the same codes and maxima in fewer launches and
// reads than the two calls above (see quant_pair_kernel).  codesRA ... not null: their residuals too, quantized a second time.
bool quantize_pair_usable(int M, int N, int K);
struct QuantPair {
    int8_t *codesA, *codesB;                // M x K; N x K (transposed)
    float *amaxA, *amaxB;
    int8_t *codesRA, *codesRB;
    float *amaxRA, *amaxRB;
};
// packed: the format of packed codes (see PK8, PK6), or PK_NONE for rows of bytes.
int launch_quantize_pair(const float* A, int lda, const float* B, int ldb, int M, int N, int K, QuantParams q, QuantPair o,
                         hipStream_t st, int packed = PK_NONE);
// The group maxima alone, and sketches beside them (what a quantization followed by a factorization starts from): row maxima of A
// (M x K), column maxima of B (K x N), up to two sketches in one launch (long columns are cleared in one before it), and with
// per_tensor the matrices' maxima in another.  M or N may be 0: the other operand alone.
struct SketchJob {
    uint64_t seed;
    int stream_id, rows, cols, ld;          // (as for launch_fill_sketch)
    float* omega;
};
int launch_absmax_pair(const float* A, int lda, int M, int K, float* amaxA, const float* B, int ldb, int N,
                       float* amaxB, QuantParams q, bool per_tensor, const SketchJob* fill, int nfill, hipStream_t st);
// lam[n], s[n] from amax[n]; entries n..npad-1 are zero-filled.
// A minimal kernel (writes one zero word): used as a few microseconds of delay on a stream.
int launch_tick(uint32_t* word, hipStream_t st);
int launch_scales(const float* amax, int n, int npad, float qmaxf, float* lam, float* s,
                  hipStream_t st);

// ---- sketch.hip ---------------------------------------------------------
// omega[i*ld + j] for i < rows, j < ld; columns j >= cols are zero.
int launch_fill_sketch(uint64_t seed, int stream_id, int rows, int cols, int ld, float* omega,
                       hipStream_t st);
// The same plus, in the same launch, the step vectors of the operand: lam[i] = qmax/amax[i],
// s[i] = amax[i]/qmax for i < n, zero up to npad (skipped when amax is null).
int launch_sketch_and_scales(uint64_t seed, int stream_id, int rows, int cols, int ld, float* omega,
                             const float* amax, int n, int npad, float qmaxf, float* lam, float* s,
                             hipStream_t st);
// dst[i*ld + j] = (j < cols) ? src[i*cols + j] : 0
int launch_pad_copy(const float* src, int rows, int cols, int ld, float* dst, hipStream_t st);

// ---- passes.hip ---------------------------------------------------------
#define MAX_SPLITS 8      // upper bound on the splits of plan_pass_n from 1025 rows on; launch_reduce_gram sums so many at a time
#define MAX_SPLITS_FEW 32 // ... up to 1024 rows
#define MAX_SPLITS_T 64   // upper bound for plan_pass_t
struct PassPlan {
    int splits;   // number of partial results
    int chunk;    // reduction-index range per split (multiple of 64)
};
PassPlan plan_pass_n(int rows, int cols, int LP);
PassPlan plan_pass_t(int rows, int cols, int LP);
// Room for the partial results of both passes: at least what the plans need, and no less
// for a larger problem (a plan takes fewer ranges where there are more rows), so that a workspace serves smaller ones.
size_t pass_partial_floats(int rows, int cols, int LP);
int codes_splits(int rows, int K);          // (of lrqmm_gemm_static's limit alone)
// One operand of a factorization, as the passes see it.  X is rows x cols with row stride ldx (>= cols); axis 0: scales
// by row, 1: by column (lam, s: the step vectors).
struct PassOperand {
    const float* X;
    int ldx, rows, cols, axis;
    float *lam, *s;
    float* W;           // cols x LP: operand of the N pass, result of the T pass
    float* Y;           // rows x LP: operand of the T pass, result of the N pass
    float* partial;     // [splits][rows or cols][LP]
    const float* amax;  // group maxima and codes, used by the quantizing pass
    int8_t* codes;
    PassPlan pn, pt;
    void* steps;        // for passes_full_*.hip: W (N pass) or Y (T pass) in the order of its steps
    double* gpart;      // ... Gram partials of the result
    int fn, ft;         // pass_full_ranges of the N pass, the T pass
    const int* run;     // T pass of 16 columns in float32: does nothing where *run is 0 (null: runs)
};
// A tall operand of a residual product in the order of the matrix cores' operands, zero padded, lane 16 g + c holding rows 4 g + (e & 3)
// + 16 (e >> 2) (e < 8) of column c of a 32-row step: STEPS_PLANES [step][column tile of 16][plane][lane][8], three bfloat16 planes;
// STEPS_FLOAT [step][lane][8] float32, one column tile (the passes on the float32 matrix cores, see launch_resid_mul_n).
enum { STEPS_NONE = 0, STEPS_PLANES = 1, STEPS_FLOAT = 2 };
#define STEP_PIECE 512
static inline size_t steps_bytes(int n, int LP) { return (size_t)ceil_div(n, 32) * (LP / 16) * 3 * STEP_PIECE * sizeof(uint16_t); }
static inline int steps_format(int LP, int planes) { return LP == 16 && planes == 3 ? STEPS_FLOAT : STEPS_PLANES; }
// Both passes take one operand, or two of different axes in one launch.
// planes: bfloat16 planes per float32 operand in the matrix-core products (3: float32 accuracy, the default;
// 2: relative error 2^-16 per product; 1: plain bfloat16 operands) -- the reduced-precision compensation of the
// Methodology (text after Eq. (gemm_r_split)).  With planes == 3 sketches of up to 16 columns use the float32
// matrix-core kernels, except in the quantizing N pass, which is on bfloat16 planes at every width.
// N pass: partial[s][rows][LP] = R[:, chunk s] . W[chunk s, :].
// quantize: the same launch quantizes the operands from their group maxima (amax): it writes the codes (row-major for
// axis 0, transposed for axis 1) and the step vectors, then read by the later passes.
// packed: the format in which the codes leave (not PK_NONE: codes is then 16-byte aligned and holds pk_bytes).
int launch_resid_mul_n(const PassOperand* op, int nop, QuantParams q, int LP, bool quantize, hipStream_t st,
                       int planes = 3, int packed = PK_NONE);
// T pass: partial[s][cols][LP] = R[chunk s, :]^T . Y[chunk s, :].
int launch_resid_mul_t(const PassOperand* op, int nop, QuantParams q, int LP, hipStream_t st, int planes = 3);
// ---- passes_full_n.hip, passes_full_t.hip ----
// The same products, the other factor in the order of steps, for the operands with fn > 0 (N pass), ft > 0 (T pass): in that many
// ranges of the reduction, a single one without partial results: Y (rows x LP) = R W, or W (cols x LP) = R^T Y, and
// full_blocks(results, LP) Gram partials of it.  One operand or two of different axes.
#define FULL_ELEMENTS 16200000      // of an operand with sides of up to 4096 (see two_chains)
int pass_full_ranges(bool t_type, int rows, int cols, int ldx, int LP);     // 0: the products above
size_t full_steps_bytes(int rows, int cols, int LP);   // of the longest factor in the order of steps; does not fall when an argument grows
int full_blocks(int n, int LP);
int full_blocks_most(int n, int LP);        // of any result of up to n rows
int launch_pass_full_n(const PassOperand* op, int nop, QuantParams q, int LP, hipStream_t st, int planes = 3);
int launch_pass_full_t(const PassOperand* op, int nop, QuantParams q, int LP, hipStream_t st, int planes = 3);
// Row quantization and the sketch product from one read, for operands quantized by rows whose rows are short
// (cols <= 576, a multiple of 16) and sketches padded to 16 columns: writes the row maxima amax[rows], the step
// vectors, the codes (rows x cols), Y = R.W (rows x 16) and gpart[quant_sketch_rows_blocks(rows)][16][16], the
// float64 Gram matrices of the workgroups' rows of Y (to be added by launch_gram_sum).  Maxima, steps and codes
// carry the bits of launch_quantize_rows; Y is the float32 matrix-core product of launch_resid_mul_n with the
// reduction cut into eight parts that are added in a fixed order.  Otherwise LRQMM_ERR_UNSUPPORTED and nothing is
// launched.
#define LRQ_QSR_MAX_BLOCKS 512
#define LRQ_QSR_MAX_COLS 576
// Where lrqmm_matmul takes it, or quant_project_rows_kernel.  Below, both operands advance together in half the launches and on
// one stream: a call on two streams takes 95 us and more whatever its size.  Together / one read, us per call (64 columns of B
// unless stated, sketch of 8, no power iteration):
//   K = 64   80000 rows 88 / 98, 100352 99 / 100 (16 columns of B 111 / 100, 512 172 / 167)
//   K = 144  52000 88 / 97, 60000 94 / 98 (512 columns 129 / 119), 80000 115 / 99
//   K = 288  36000 84 / 103, 44000 90 / 103, 52000 110 / 103
//   K = 432  28000 80 / 104, 34000 103 / 101 (512 columns 141 / 131), 40000 108 / 105
//   K = 576  24000 88 / 108, 30000 93 / 106, 33000 106 / 109, 40000 115 / 109
// One power iteration: 80000 x 64 157 / 150, 60000 x 144 169 / 164, 44000 x 288 159 / 158, 34000 x 432 183 / 174, 30000 x 576 172 / 168.
// Above 13 million elements the joint passes leave partial results, above 32768 rows their Gram workgroups take 128 rows.
#define LRQ_ONE_READ_ROWS 25000     // more than these in any case
static inline bool one_read_pays(int rows, int cols) {
    return (long long)(rows - LRQ_ONE_READ_ROWS) * (cols < 64 ? 64 : cols) >= 4600000 ||
           (rows > 32768 && (long long)rows * cols > 13000000);
}
bool quant_sketch_rows_usable(const float* X, int ldx, int rows, int cols, int LP, const int8_t* codes);
int quant_sketch_rows_blocks(int rows);
int launch_quant_sketch_rows(const float* X, int ldx, int rows, int cols, QuantParams q, const float* W, int LP,
                             float* Y, double* gpart, float* amax, float* lam_out, float* s_out, int8_t* codes,
                             hipStream_t st);
// The same (one_read.hip) with R^T Y from that read as well, for the same operands: Y = R.(W H) with a reflection H (see there), and
// mpart[quant_project_blocks(rows)][cols][16] the workgroups' R^T Y, to be added by launch_project_sum.
#define LRQ_QPR_MAX_BLOCKS 480      // two on every CU of 256 but one in eight, which the other operand's small
// launches find half free (496: they waited for the end, the call 180 us in place of 168)
int quant_project_blocks(int rows);
int launch_quant_project_rows(const float* X, int ldx, int rows, int cols, QuantParams q, const float* W, int LP, float* Y, double* gpart,
                              float* mpart, float* amax, float* lam_out, float* s_out, int8_t* codes, hipStream_t st);
// The panels of the rank-2r update from the codes of both operands, in one launch (RP: r rounded up to 16).  Wf, Vf: the K x r
// factors W and Vt^T as three bfloat16 planes in operand order, zero padded: [k block of 64][column tile of 16][plane][step][lane][8],
// a piece (k block, tile, plane, step) being an operand of v_mfma_f32_16x16x32_bf16.  Every codes format gives the same bits.
#define FACTOR_PIECE 512            // bfloat16 values
struct PanelArgs {
    const int8_t *codesA, *codesB;          // of A and of B transposed
    const uint16_t *Wf, *Vf;
    const float *U, *Sig, *sA, *sB, *Xp, *Gam, *Zt;
    float *Lp, *Rp;
    int M, N, K, r, R2P, nslices;           // nslices: of Xp
    int ldu;                                // row stride of U
    int nbR;                                // (set by launch_panels)
};
int launch_panels(const PanelArgs& a, int RP, int planes, int packed, hipStream_t st);

// ---- orth.hip -----------------------------------------------------------
// Every launch below takes one job or two (the two operands of a product, in one launch).
int gram_blocks(int n, int LP);
int gram_blocks_most(int n, int LP);        // of any factor with up to n rows
struct GramJob {
    const float* partial;       // [splits][n][LP]
    int splits, n;
    float* Y;                   // n x LP: sum of the partials
    double* gpart;              // [blocks][LP][LP]
    double* gram;               // LP x LP: Gram matrix of Y
    int blocks;                 // Gram partials; 0: gram_blocks(n, LP)
    int rows_per_block;         // (set by launch_reduce_gram)
    void* steps;                // launch_orth_apply: Q in the order of steps too
    int steps_fmt;
    const double* M;            // launch_orth_apply (16 columns): Z <- (sum of M's PROJECT_GROUPS parts) T as well, m x LP
    float* Z;
    int m;
    int* again;                 // ... and whether R^T Q has to be formed from Q instead (see PROJECT_AMPLIFICATION)
};
// Y = sum_s partial[s]; gpart[b] = Gram of the b-th block of rows of Y in float64.
int launch_reduce_gram(const GramJob* job, int njob, int LP, hipStream_t st);
// gram = sum over the blocks of gpart, in fixed order.
int launch_gram_sum(const GramJob* job, int njob, int LP, hipStream_t st);
// What `blocks` workgroups of quant_project_rows_kernel have left, added in PROJECT_GROUPS groups: gsum[group][16][16] (Gram partials for
// launch_orth_apply, with sum) and msum[group][cols][16].
#define PROJECT_GROUPS 16
// Where Z = (R^T Y) T takes the place of R^T Q.  R^T Y is a float32 sum in the square of the operand's scale, and T multiplies the error of its
// columns: column j of Z by sum_i |T_ij| |y_i|, next to 1 for columns of Y that are far from dependent, 10^5 at the limit of a live
// pivot.  Relative distance of Z from float64, 28800 x 576, 8 columns, 4 bits (float32 emulation on the CPU), R^T Q / (R^T Y) T: independent values
// (1.2 to 1.4) 7e-8 / 3e-8, values about a mean of each column's own (3.9) 7.4e-8 / 7.0e-8, at 8 bits (4.5) 8.1e-8 / 8.1e-8; rank 1 plus 1e-3
// noise (19) 7e-8 / 3.6e-7, rank 1 times 1 + 1e-4 noise (2500) 8e-8 / 4e-5.  The lengths of live columns keep the squares inside float32's
// range with as much room as R^T Q has (2^-20 to 2^40; those of 28800 rows of order 1 are 10 to 10^4).
#define PROJECT_AMPLIFICATION 4.0
#define PROJECT_LEAST 0x1p-40       // of the squared lengths
#define PROJECT_MOST 0x1p80
int launch_project_sum(const double* gpart, const float* mpart, int blocks, int cols, double* gsum, double* msum, hipStream_t st);
// Y <- Y T, T upper triangular with (Y T)^T (Y T) = I on the live columns, from gram; sum: from the Gram partials (as many
// as orth_apply_sums allows) instead.
bool orth_apply_sums(int blocks, int LP);
int launch_orth_apply(const GramJob* job, int njob, int ell, int LP, bool sum, hipStream_t st);
// out = In[n x LP] . Mat[LP x cm]; normal: out[i*ldo + c]; transposed: out[c*ldo + i].  Up to four jobs.
struct ApplyJob {
    const float* In;
    const double* Mat;
    float* out;
    int n, cm, ldm, ldo, transposed;
};
int launch_apply(const ApplyJob* job, int njob, int LP, hipStream_t st);
// Eigen-decomposition of the Gram matrix (l x l, leading dimension LP): Sigma[r] = sqrt of
// the r largest eigenvalues, Ur (LP x r) their eigenvectors, Mv = Ur diag(1/Sigma).
struct SvdJob {
    const double* gram;
    float* Sigma;
    double *Ur, *Mv;
};
int launch_small_svd(const SvdJob* job, int njob, int ell, int LP, int rank, hipStream_t st);
// Factors without the small SVD, for sketches padded to 16 columns: U (rows x rank) = the leading columns of Q, Sigma = 1,
// Vt (rank x cols) = (sum_s partial[s])^T, the T pass's result Q^T R.  U diag(Sigma) Vt is Q Q^T R.
struct BasisJob {
    const float* partial;       // [splits][cols][LP]
    int splits, cols;
    const float* Q;             // rows x LP
    int rows;
    float *U, *Sigma, *Vt;
};
int launch_take_basis(const BasisJob* job, int njob, int LP, int rank, hipStream_t st);
// The same for both operands, as the panels need it (see PanelArgs; U is A's Q, ldu = 16): Vf from A's partials, Wf from B's Q, Zt
// from B's partials, the slices Xp of V^T W, Sig = Gam = 1, in one launch.  basis_slices: of Xp; 0: K is too long.
int basis_slices(int K);
struct BasisPanels {
    const float *partialA, *partialB, *QB;      // [splitsA][K][16], [splitsB][N][16], K x 16
    int splitsA, splitsB, N, K, r;
    const int* again;                           // where *again is not 0 (may be null), A's are these
    const float* partialA2;
    int splitsA2;
    uint16_t *Wf, *Vf;
    float *Zt, *Xp, *Sig, *Gam;
    int slices, per, nkb;                       // (set by launch_basis_panels)
};
int launch_basis_panels(const BasisPanels& a, hipStream_t st);

// ---- gemm.hip -----------------------------------------------------------
// X = V^T W is kept as vtw_slices(K) k-slices Xp[ks][t][u] that are summed where X is used.
#define LRQ_VTW_MAX_SLICES 16
int vtw_slices(int K);      // (at most)
// One launch (r > 0): step vectors lamX/sX (padded to a multiple of 4) of both operands, Wf / Vf: the planes of W and Vt^T (see PanelArgs), and the slices
// Xp of V^T W.
int launch_panel_prep(int M, int N, int K, int r, int RP, float qmaxf, const float* amaxA, const float* amaxB,
                      const float* W, const float* Vt, float* lamA, float* sA, float* lamB, float* sB,
                      uint16_t* Wf, uint16_t* Vf, float* Xp, hipStream_t st);
// Destination of the GEMM: D (row stride ldc) <- alpha * result + beta * D; D is not read when beta == 0.
struct GemmOut {
    float* C;
    int ldc;
    float alpha, beta;
};
// result = diag(sA) (Aq . BqT^T) diag(sB) [+ Lp . Rp^T when Lp != null]; optional raw int32 output
// (M x N, dense).  Without panels (Lp == null) sA, sB are the group maxima, turned into steps with qmaxf.
int launch_int8_gemm(int M, int N, int K, const int8_t* Aq, const int8_t* BqT, const float* sA,
                     const float* sB, const float* Lp, const float* Rp, int R2P, GemmOut C,
                     int32_t* Cint, float qmaxf, hipStream_t st, int packed = PK_NONE);
// packed (here and below): the format of both code matrices; same results.  Packed codes: no Cint beside a result; Cint without one
// (out.C == null) holds the raw sums.
// The format in which codes travel inside a call with factorizations, and in one without (there also PK_NONE: rows of bytes).
int packed_format(int bits, int K);
int direct_format(int M, int N, int K, int bits);
// D <- alpha (A0 B0 + A0 B1 + A1 B0 [+ A1 B1]) + beta D, the products of the operands' codes (0) and of their residuals' (1),
// each dequantized by the steps of its group maxima: terms = 3 or 4 products in one launch, where int8_terms_usable.
bool int8_terms_usable(int M, int N, int K);
int terms_format(int M, int N, int K, int bits);        // of the codes of four products in one launch
int launch_int8_terms(int M, int N, int K, const int8_t* const A[2], const float* const amaxA[2], const int8_t* const B[2],
                      const float* const amaxB[2], int terms, float qmaxf, GemmOut out, hipStream_t st, int packed = PK_NONE);
// The product with an empty reduction (K == 0): D <- alpha * 0 + beta * D (D not read when beta == 0) and,
// when Cint is given, zeros in Cint.  Reads no operand.
int launch_empty_product(int M, int N, GemmOut C, int32_t* Cint, hipStream_t st);
// The raw int32 sums alone (C_int, row stride N), for a chip on which only `resident` CUs are
// free (0: unknown): with one 256x256 tile per workgroup, the tiles beyond a whole number of
// rounds over those CUs would cost a full extra round; they are cut along K instead, one
// workgroup per range, which leave partial sums in `part` (int8_gemm_sums_scratch_bytes; null:
// no cut), and launch_int8_gemm_sums_finish (same arguments, later on the same stream) adds
// them up into C_int.  Integer sums: the result is bit-identical to the plain kernel's.
#define LRQ_SUMS_MAX_PARTS 64       // (tile, range) pairs at most
size_t int8_gemm_sums_scratch_bytes(int M, int N, int K);
int launch_int8_gemm_sums(int M, int N, int K, const int8_t* Aq, const int8_t* BqT, int32_t* Cint, int resident,
                          int32_t* part, hipStream_t st, int packed);
int launch_int8_gemm_sums_finish(int M, int N, int K, const int8_t* Aq, const int8_t* BqT, int32_t* Cint, int resident,
                                 const int32_t* part, hipStream_t st);
// True when the large-tile kernel may be asked for raw int32 sums: launch_int8_gemm with C == null and Cint != null (sA, sB are
// then not read).  With C given launch_int8_gemm takes it from a few more tiles on (large_tiles_into_c).
bool int8_gemm_large_tiles(int M, int N);
long long int8_gemm_tiles(int M, int N);       // of 256 x 256, how many cover the output
// True when the integer product may run early and launch_rank_update finish the job: the
// large-tile kernel applies, N % 4 == 0 and C is 16-byte aligned.
bool rank_update_usable(int M, int N, const float* C);
// C (dense, holding raw int32 sums in its memory) <- alpha (float(Cint) sA_i sB_j + Lp . Rp^T), in place.
int launch_rank_update(int M, int N, float* C, const float* sA, const float* sB, const float* Lp, const float* Rp,
                       int R2P, float alpha, hipStream_t st);
