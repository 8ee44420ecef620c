// C-ABI entry points of the LRQMM library: argument validation, workspace
// carving and the launch sequence of each call (paper: Algorithm 2; Algorithm 1
// for lrqmm_rsvd).  No device memory is allocated here; everything lives in the
// caller's buffers and workspace.
#include "kernels.h"
#include <cstdio>
#include <algorithm>
#include <cstdlib>
#include <functional>
#include <memory>
#include <vector>

namespace {

struct Arena {
    char* base;
    size_t off;
    explicit Arena(void* b) : base(static_cast<char*>(b)), off(0) {}
    template <typename T>
    T* take(size_t count) {
        off = align_up(off, 256);
        T* p = base ? reinterpret_cast<T*>(base + off) : nullptr;
#ifdef LRQMM_CHECK      // checked host build: sizes must not wrap, regions must stay aligned and ordered
        size_t bytes = 0, end = 0;
        if (__builtin_mul_overflow(count, sizeof(T), &bytes) || __builtin_add_overflow(off, bytes, &end) ||
            (base && ((uintptr_t)p & 255) != 0) || end < off) {
            std::fprintf(stderr, "LRQMM_CHECK: workspace region overflows (count %zu x %zu bytes at offset %zu)\n", count,
                         sizeof(T), off);
            std::abort();
        }
#endif
        off += count * sizeof(T);
        return p;
    }
};

inline int pad_to(int x, int m) { return (x + m - 1) / m * m; }

struct RsvdWs {
    float *lam, *s, *Wc, *Yr, *partial;
    double *gpart, *gram, *Ur, *Mv, *M;
    char* steps;
    float* mpart;               // one-read kernel: partial R^T Y (tall operands, like M)
    int* again;                 // ... and whether a pass for R^T Q follows
};

// Every region of carve_rsvd and carve_matmul is at least as large for a larger problem, so that one workspace, sized for the
// largest, serves them all.
size_t carve_rsvd(Arena& a, int rows, int cols, int axis, int LP, int rank, RsvdWs* w) {
    const int nscale = axis == LRQMM_AXIS_ROW ? rows : cols;
    const int npad = pad_to(nscale, 4);
    // (the one-read quantization kernel for row-quantized operands leaves one Gram partial per workgroup)
    int nb = gram_blocks_most(rows > cols ? rows : cols, LP);
    if (axis == LRQMM_AXIS_ROW && LP == 16 && quant_sketch_rows_blocks(rows) > nb) nb = quant_sketch_rows_blocks(rows);
    nb = std::max(nb, full_blocks_most(rows > cols ? rows : cols, LP));
    RsvdWs t = {};
    t.lam = a.take<float>(npad);
    t.s = a.take<float>(npad);
    t.Wc = a.take<float>((size_t)cols * LP);
    t.Yr = a.take<float>((size_t)rows * LP);
    // (the one-read kernel's Gram matrices and R^T Y, then their sums, lie where a pass leaves its partial results later)
    const size_t partial = pass_partial_floats(rows, cols, LP) * sizeof(float);
    const bool tall = axis == LRQMM_AXIS_ROW && rows > LRQ_ONE_READ_ROWS;       // (used for sketches of 16 columns alone)
    const size_t values = (size_t)std::min(cols, LRQ_QSR_MAX_COLS) * 16, sums = PROJECT_GROUPS * (256 + values) * sizeof(double);
    const size_t project = tall ? sums + quant_project_blocks(rows) * values * sizeof(float) : 0;
    char* const shared = a.take<char>(std::max(partial, project));
    t.partial = reinterpret_cast<float*>(shared);
    t.M = reinterpret_cast<double*>(shared);            // Gram matrices, then R^T Y
    t.mpart = shared ? reinterpret_cast<float*>(shared + sums) : nullptr;
    t.gpart = a.take<double>((size_t)nb * LP * LP);
    t.gram = a.take<double>((size_t)LP * LP);
    t.Ur = a.take<double>((size_t)LP * rank);
    t.Mv = a.take<double>((size_t)LP * rank);
    t.steps = a.take<char>(full_steps_bytes(rows, cols, LP));
    if (tall) t.again = a.take<int>(1);
    if (w) *w = t;
    return a.off;
}

struct GemmWs {
    float *lamA, *sA, *lamB, *sB, *X, *Lp, *Rp;
    uint16_t *Wf, *Vf;
};

size_t carve_gemm(Arena& a, int M, int N, int K, int rank, GemmWs* w) {
    GemmWs t = {};
    const int Mp = pad_to(M, 4), Np = pad_to(N, 4);
    t.lamA = a.take<float>(Mp);
    t.sA = a.take<float>(Mp);
    t.lamB = a.take<float>(Np);
    t.sB = a.take<float>(Np);
    if (rank > 0) {
        const int RP = pad_to(rank, 16), R2P = pad_to(2 * rank, 8);
        t.Wf = a.take<uint16_t>((size_t)3 * RP * pad_to(K, 64));
        t.Vf = a.take<uint16_t>((size_t)3 * RP * pad_to(K, 64));
        t.X = a.take<float>((size_t)rank * rank * LRQ_VTW_MAX_SLICES);
        t.Lp = a.take<float>((size_t)M * R2P);
        t.Rp = a.take<float>((size_t)N * R2P);
    }
    if (w) *w = t;
    return a.off;
}

struct MatmulWs {
    int8_t *Aq, *BqT;
    float *amaxA, *amaxB, *U, *Sig, *Vt, *W, *Gam, *Zt;
    uint32_t* tick;
    int32_t* parts;                   // partial sums of the early integer product's K ranges
    void *sub, *subA, *subB;          // scratch of the products and of the two factorizations
    size_t sub_bytes, subA_bytes, subB_bytes;
};

size_t carve_matmul(Arena& a, int M, int N, int K, int rank, int oversample, MatmulWs* w) {
    MatmulWs t = {};
    t.Aq = a.take<int8_t>(pk_bytes(M, K, PK8));         // (the most of any format)
    t.BqT = a.take<int8_t>(pk_bytes(N, K, PK8));
    t.amaxA = a.take<float>(M);
    t.amaxB = a.take<float>(N);
    t.tick = a.take<uint32_t>(64);
    t.parts = nullptr;
    if (rank > 0 && int8_gemm_sums_scratch_bytes(M, N, K) > 0)
        t.parts = a.take<int32_t>(int8_gemm_sums_scratch_bytes(M, N, K) / sizeof(int32_t));
    if (rank > 0) {
        t.U = a.take<float>((size_t)M * rank);
        t.Sig = a.take<float>(rank);
        t.Vt = a.take<float>((size_t)rank * K);
        t.W = a.take<float>((size_t)K * rank);
        t.Gam = a.take<float>(rank);
        t.Zt = a.take<float>((size_t)rank * N);
    }
    a.off = align_up(a.off, 256);
    size_t sub = 0, sa = 0, sb = 0;
    {
        Arena g(nullptr);
        sub = carve_gemm(g, M, N, K, rank, nullptr);
    }
    if (rank > 0) {
        // the two residual factorizations run concurrently: each gets its own region
        const int LP = pad_to(rank + oversample, 16);
        Arena ra(nullptr), rb(nullptr);
        sa = align_up(carve_rsvd(ra, M, K, LRQMM_AXIS_ROW, LP, rank, nullptr), 256);
        sb = align_up(carve_rsvd(rb, K, N, LRQMM_AXIS_COL, LP, rank, nullptr), 256);
    }
    t.subA = a.base ? a.base + a.off : nullptr;
    t.subA_bytes = sa;
    t.subB = a.base ? a.base + a.off + sa : nullptr;
    t.subB_bytes = sb;
    a.off += sa + sb;
    t.sub = a.base ? a.base + a.off : nullptr;
    t.sub_bytes = sub;
    a.off += sub;
    if (w) *w = t;
    return a.off;
}

// Optional stage timing of lrqmm_matmul with HIP events recorded on the caller's stream.
constexpr int kProfStages = LRQMM_PROF_STAGES;
constexpr int kProfEvents = 11;
constexpr int kProfMaxCalls = 512;
// event indices: 0-2 main stream (quantize A, RSVD A), 3-5 side stream (quantize B, RSVD B),
// 6-8 main stream after the join (panels, GEMM or rank update), 9-10 the early integer GEMM on
// the third stream (recorded back to back on the main stream when that schedule is not used)
constexpr int kStageBegin[kProfStages] = {0, 1, 3, 4, 6, 7, 9};
constexpr int kStageEnd[kProfStages] = {1, 2, 4, 5, 7, 8, 10};
constexpr int kLastMainEvent = 8;
struct Prof {
    bool on = false;
    bool gemm_only = false;             // record only the pair of events around the integer GEMM
    bool early[kProfMaxCalls] = {};     // per recorded call: the GEMM ran on the third stream
    int ncalls = 0;
    hipEvent_t ev[kProfMaxCalls][kProfEvents];
    bool created = false;
} g_prof;

// Streams and events that lrqmm_matmul needs beyond the caller's stream, one set per device (created on
// the first call on that device, never destroyed: they live as long as the process).  `stream` carries
// B's quantization and factorization where they run next to A's on the caller's stream; `gemm_stream` the early integer
// product.  All at default priority.
struct Side {
    hipStream_t stream = nullptr;        // B's chain where it runs beside A's
    hipStream_t gemm_stream = nullptr;   // early integer GEMM
    hipEvent_t fork = nullptr, join = nullptr;
    hipEvent_t gate = nullptr, gate_b = nullptr, gdone = nullptr;
    int cus = 0;                         // compute units of the device
    bool ok = false;
};
constexpr int kMaxDevices = 16;
Side g_side_dev[kMaxDevices];

// The current device's set, or null when it does not exist yet and `create` is false (a call under
// stream capture must not create streams) or when creating it failed.
Side* side_state(bool create) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    Side& s = g_side_dev[dev];
    if (s.ok) return &s;
    if (!create) return nullptr;
    if (hipStreamCreateWithFlags(&s.stream, hipStreamNonBlocking) != hipSuccess) return nullptr;
    if (hipStreamCreateWithFlags(&s.gemm_stream, hipStreamNonBlocking) != hipSuccess) return nullptr;
    for (hipEvent_t* e : {&s.gate, &s.gate_b, &s.gdone, &s.fork, &s.join})
        if (hipEventCreateWithFlags(e, hipEventDisableTiming) != hipSuccess) return nullptr;
    if (hipDeviceGetAttribute(&s.cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return nullptr;
    s.ok = true;
    return &s;
}

// Scratch memory of lrqmm_gemm_static: a fixed array in the library's device image (every GPU that loads
// the library holds its own copy, at its own address, until the process ends).  In host code the array's
// name is only a handle for hipGetSymbolAddress; the device address is looked up once per device, with
// that device current, and kept.
static __device__ __align__(256) unsigned char scratch[LRQMM_STATIC_SCRATCH_BYTES];
void* g_scratch_ptr[kMaxDevices] = {};

int static_scratch(void** out) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return LRQMM_ERR_HIP;
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return LRQMM_ERR_HIP;
        if ((uintptr_t)ptr & 255) return LRQMM_ERR_HIP;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return LRQMM_OK;
}

inline void prof_mark(int slot, int i, hipStream_t st) {
    if (slot < 0) return;
    if (g_prof.gemm_only) {     // events 9, 10 bracket the early product, 7, 8 the fused kernel
        const bool early = g_prof.early[slot];
        if (!(early ? (i == 9 || i == 10) : (i == 7 || i == 8))) return;
    }
    (void)hipEventRecord(g_prof.ev[slot][i], st);
}

// arithmetic of the entry points that take no precision argument (lrqmm_rsvd, lrqmm_matmul)
#ifndef LRQMM_DEFAULT_PREC
#define LRQMM_DEFAULT_PREC LRQMM_PREC_FP32
#endif
bool bits_ok(int bits) { return bits >= 2 && bits <= 8; }
// Host-side size arithmetic (padding, block counts) is done in int: dimensions stay well below 2^31.
bool dims_ok(int a, int b, int c = 0) { return a <= LRQMM_MAX_DIM && b <= LRQMM_MAX_DIM && c <= LRQMM_MAX_DIM; }
// ... and an M x N output must leave the number of 128 x 128 tiles (a grid size) below 2^31
bool output_ok(int M, int N) { return (long long)((M + 127) / 128) * ((N + 127) / 128) < (1ll << 31); }
bool precision_ok(int p) {
    return p == LRQMM_PREC_FP32 || p == LRQMM_PREC_BF16X2 || p == LRQMM_PREC_BF16 || p == LRQMM_PREC_SUBSPACE_BF16X2;
}
// bfloat16 planes per operand: in the products that only shape the subspace (sketch and power iterations) and in
// the products whose values enter C directly (the projection Q^T R and the code products of the panels)
int planes_subspace(int p) { return p == LRQMM_PREC_BF16 ? 1 : (p == LRQMM_PREC_FP32 ? 3 : 2); }
int planes_values(int p) { return p == LRQMM_PREC_BF16 ? 1 : (p == LRQMM_PREC_BF16X2 ? 2 : 3); }

// Whether the two operands' factorizations run as two chains on two streams instead of advancing together, one launch
// per step for both.  Together they need half the launches, which bound small problems, and no events; as two chains the
// single-workgroup steps of one fall beside the other's passes, which pays once the passes are as long as those steps.
// Measured, together / two chains, us, sketches of 24, 40 and 80 columns (one power iteration): 1024^3 143 / 193 (24);
// 2048^3 196 / 212, 271 / 285, 497 / 508; 3072^3 279 / 283, 368 / 357, 618 / 614; 4096^3 351 / 348, 445 / 434, 688 / 690;
// 8192^3 1387 / 1366 (24), 2017 / 1958 (80).
// Those are the passes of passes.hip.  With whole reductions a pass of both operands is short enough on its own up to sides of
// 4096.  Two chains / together, us, inputs from memory, by sketch columns:
//   2600^3              10 181 / 166    24 239 / 229    40 311 / 301
//   3300^3                              24 287 / 278    40 364 / 341    80 592 / 570
//   3700^3                              24 328 / 309    40 400 / 377    80 636 / 614
//   4000^3                              24 338 / 332    40 415 / 413    80 658 / 649
//   4096 x 4096 x 2048                  24 269 / 241    40 359 / 328
//   2048 x 2048 x 4096                  24 248 / 228
//   4096^3              10 280 / 271    24 333 / 335    40 400 / 408    80 633 / 650
// and not with a short or a longer side: 4096 x 1024 x 4096 10 182 / 191, 1500 x 1500 x 6000 24 259 / 269, 6000 x 3000 x 1600
// 24 270 / 278.  Sides between 1500 and 2000: 4096 x 4096 x 1700 40 321 / 316, 3500 x 1700 x 3500 40 318 / 317, 4000 x 1500 x 3500 24
// 248 / 248.
// Few rows of A (a batch through a layer) keep the large operand's chain waiting at every one of its launches; N = K = 4096:
//   128 rows     8 172 / 158    24 232 / 218    40 310 / 291    80 523 / 518
//   512          8 178 / 168    24 242 / 233    40 313 / 306    80 535 / 534
//   768          8 186 / 175    24 247 / 241    40 320 / 320    80 545 / 548
//   1024         8 193 / 183    24 255 / 251    40 324 / 329    80 565 / 563
// A narrow B does not: 4096 x 512 x 4096 8 163 / 171, 24 230 / 230, 40 292 / 300.
bool two_chains(int M, int N, int K, int LP, int planes) {
    const long long a = (long long)M * K, b = (long long)K * N;
    if (a + b <= 13000000) return false;
    if (planes < 2 || std::max(std::max(M, N), K) > 4096) return true;
    if (M <= 768) return false;
    return !(std::min(std::min(M, N), K) >= 2000 && (LP == 16 || std::max(a, b) <= FULL_ELEMENTS));
}

// Whether the integer product (`tiles` tiles of 256 x 256, one per CU at a time) runs early, beside the small SVDs and the
// panel kernels, with the update as a kernel of its own, or with its fused epilogue after the panels.  Early it saves a last
// round that leaves most CUs idle, and the time of the SVDs where the product is one round and not much longer than they
// are; it writes and reads C once more, and a long product holds the CUs that the panel kernels need.  The lines lie alike for both
// formats of packed codes.  Measured, early / fused, us per call (one power iteration), by the sketch's width, 4 bits; 8 bits.  Whole
// rounds: one, 4096^3, 24 342 / 302; 356 / 327, 32 344 / 326; 367 / 352, 40 391 / 384; 405 / 407, 56 504 / 501; 507 / 527, 80 684 / 680; 693 / 708;
// two, 8192 x 4096 x 4096, 40 558 / 538; 591 / 578, 56 653 / 648; 682 / 691, 64 692 / 705; 743 / 752, 80 836 / 864; 851 / 906; four, 8192^3, 56
// 1436 / 1416; 1652 / 1603, 64 1485 / 1481; 1689 / 1661, 80 1680 / 1733; 1873 / 1906.  Rounds filled to 0.50 (half of one, 4096 x 2048 x 4096) 32
// 299 / 285; 298 / 293, 80 626 / 626; 626 / 629; 0.56 (one, 3072^3) 32 287 / 284; 286 / 295, 40 341 / 340; 341 / 353; 0.63 (two, 4608^3) 24 411 /
// 406; 449 / 444, 32 422 / 435; 451 / 477, 40 477 / 514; 506 / 550; 0.75 (three, 6144^3) 32 683 / 719; 779 / 819; 0.77 (four, 7168^3) 32 940 / 958; 1073 /
// 1107.  From 0.85 on widths up to 48 part with little on either side: 0.88 (three, 6656^3) 32 807 / 812; 916 / 918, 48 914 / 927; 1015 / 1025,
// (four, 7680^3) 40 1147 / 1139; 1326 / 1297, 48 1197 / 1174; 1346 / 1330, 0.94 (four, 7936^3) 48 1262 / 1230; 1435 / 1402; wider ones gain, 0.88
// 7680^3 56 1292 / 1309; 1442 / 1459, 64 1339 / 1368; 1490 / 1518, 0.94 7936^3 56 1384 / 1381; 1555 / 1536, 64 1434 / 1447; 1604 / 1594, 80 1608 / 1676; 1781 /
// 1814, 0.90 (five, 8704^3) 56 1689 / 1714; 1910 / 1931, 64 1756 / 1781; 1967 / 1991, 0.89 (seven, 10240^3) 56 2238 / 2218; 2604 / 2581, 64 2306 / 2301;
// 2672 / 2660, 80 2583 / 2633; 2975 / 2999.
bool early_product(long long tiles, int cus, int ell) {
    const long long rounds = (tiles + cus - 1) / cus;
    if (ell < 32) return false;
    const int fill = ell >= 64 || (ell > 48 && rounds <= 5) ? 95 : 85;
    return 100 * tiles <= fill * rounds * cus || rounds <= (ell > 64 ? 2 : (ell >= 40 ? 1 : 0));
}

// int32 accumulation is safe when K * (qmax+1)^2 < 2^31.
bool k_fits_int32(int K, int bits) {
    const long long lim = 1ll << (2 * (bits - 1));
    return (long long)K * lim < (1ll << 31);
}

// A factorization is first planned as a list of kernel launches and then issued, so that lrqmm_matmul can put the
// early integer product between them and, where the two operands' factorizations run on two streams, issue their
// launches alternately: both streams then receive work at the same pace.
using LaunchList = std::vector<std::function<int()>>;

// Issues a[a0 .. a1) and b[b0 .. b1) alternately.
static int run_interleaved(const LaunchList& a, size_t a0, size_t a1, const LaunchList& b, size_t b0, size_t b1) {
    while (a0 < a1 || b0 < b1) {
        if (a0 < a1) {
            const int rc = a[a0++]();
            if (rc != LRQMM_OK) return rc;
        }
        if (b0 < b1) {
            const int rc = b[b0++]();
            if (rc != LRQMM_OK) return rc;
        }
    }
    return LRQMM_OK;
}
static int run_interleaved(const LaunchList& a, const LaunchList& b) {
    return run_interleaved(a, 0, a.size(), b, 0, b.size());
}

// One operand's factorization R ~ U diag(Sigma) Vt: the operand as the passes see it, scratch, destinations.
struct Factor {
    PassOperand op;
    RsvdWs w;
    float *U, *Sigma, *Vt;
};
static int make_factor(Factor* f, const float* X, int ldx, int rows, int cols, int axis, int LP, int rank,
                       const float* amax, int8_t* codes, float* U, float* Sigma, float* Vt, void* workspace,
                       size_t workspace_bytes) {
    Arena a(workspace);
    if (carve_rsvd(a, rows, cols, axis, LP, rank, &f->w) > workspace_bytes) return LRQMM_ERR_WORKSPACE;
    f->op = {X, ldx, rows, cols, axis, f->w.lam, f->w.s, f->w.Wc, f->w.Yr, f->w.partial, amax, codes,
             plan_pass_n(rows, cols, LP), plan_pass_t(rows, cols, LP), f->w.steps, f->w.gpart,
             pass_full_ranges(false, rows, cols, ldx, LP), pass_full_ranges(true, rows, cols, ldx, LP)};
    f->U = U; f->Sigma = Sigma; f->Vt = Vt;
    return LRQMM_OK;
}

// The partial results of the last transposed product: a single one where the pass leaves none.  projected: formed beside the first
// product (see one_read_projects); where *again is set, a pass has left `p2` instead.
struct TPartials { const float* p; int splits; const int* again; const float* p2; int splits2; };
static TPartials t_partials(const Factor& f, int planes, bool projected = false) {
    if (projected) return {f.op.W, 1, f.w.again, f.op.partial, f.op.pt.splits};
    if (planes >= 2 && f.op.ft == 1) return {f.op.W, 1};
    return {f.op.partial, planes >= 2 && f.op.ft > 1 ? f.op.ft : f.op.pt.splits};
}

// Whether the one-read kernel forms R^T Y as well: where R^T Q is the only other product and only its sums are asked for, and not
// where Y is likely to be turned down (PROJECT_AMPLIFICATION): the columns of R Omega are as dependent as those of Omega, whose
// amplification is above 4 in 5 % of the sketches of 16 columns with 64 rows, in 43 % of 8 with 16, and in none of 3000 with six
// times as many rows as columns.  Both products / R Omega alone, 100352 rows, 64 columns of B, us: 16 values a row l = 4 98 / 107, 8
// 124 / 111; 32 l = 8 97 / 111, 16 128 / 115; 64 l = 8 98 / 99; 112 l = 8 99 / 110; 576 l = 8 169 / 204.
static bool one_read_projects(int power_iters, bool stop_at_basis, int cols, int rank) {
    return power_iters == 0 && stop_at_basis && cols >= 6 * rank;
}

// How the first residual product of a factorization is formed.
enum class FirstPass {
    plain,          // codes and step vectors exist: Y = R Omega
    quantize,       // only the group maxima exist: the same pass leaves the codes and the step vectors too
    one_read        // nothing exists: maxima, codes, Y and the Gram partials of Y from one read (short rows of A)
};

// Appends the launches of one factorization, or of two that advance together (one launch per step for both; their
// operands have different axes), to `ops`.  The sketches are in place.  svd_index: position of the small SVD.
// stop_at_basis: the list ends with the last product's partials (see launch_basis_panels).  basis_suffices: the caller only uses the
// product U diag(Sigma) Vt, and nothing is truncated (oversample == 0): U = Q, Sigma = 1, Vt = Q^T R carry the same product as the
// SVD's factors.  packed: the format of the quantizing pass's codes.
static void factor_launches(LaunchList& ops, const Factor* factors, int n, FirstPass first, QuantParams q, int rank,
                            int oversample, int power_iters, int planes_first, int planes, int planes_last, hipStream_t st,
                            size_t* svd_index, float* one_read_amax = nullptr, bool basis_suffices = false,
                            int packed = PK_NONE, bool stop_at_basis = false) {
    struct Pair { Factor f[2]; PassOperand op[2]; };
    auto p = std::make_shared<Pair>();
    for (int i = 0; i < n; ++i) { p->f[i] = factors[i]; p->op[i] = factors[i].op; }
    const int ell = rank + oversample, LP = pad_to(ell, 16);
    // A product and the Gram partials of its result, and then, unless it is the last, Q = orth(result) in place: Gram (float64),
    // Cholesky and Q = Y T.  An operand whose pass leaves no partial results (launch_pass_full) needs its other factor in the order
    // of steps, from the orthonormalization before.
    struct Jobs { GramJob g[2]; };
    auto in_steps = [=](bool t_type, int pl, int i) { return pl >= 2 ? (t_type ? p->op[i].ft : p->op[i].fn) : 0; };
    auto product = [&](bool t_type, int pl) {
        Jobs j = {};
        Pair part[2];                       // [1]: the operands whose pass takes the order of steps
        int np[2] = {0, 0};
        for (int i = 0; i < n; ++i) {
            const Factor& f = p->f[i];
            const PassOperand& o = f.op;
            const int rows = t_type ? o.cols : o.rows, ranges = in_steps(t_type, pl, i);
            part[ranges > 0].op[np[ranges > 0]++] = o;
            j.g[i] = {f.w.partial, ranges > 0 ? ranges : (t_type ? o.pt.splits : o.pn.splits), rows, t_type ? o.W : o.Y, f.w.gpart, f.w.gram,
                      ranges == 1 ? full_blocks(rows, LP) : 0, 0};
        }
        for (int k = 0; k < 2; ++k) {
            if (np[k] == 0) continue;
            const Pair a = part[k];
            const int na = np[k];
            if (k) ops.push_back([=] { return (t_type ? launch_pass_full_t : launch_pass_full_n)(a.op, na, q, LP, st, pl); });
            else ops.push_back([=] { return (t_type ? launch_resid_mul_t(a.op, na, q, LP, st, pl)
                                                    : launch_resid_mul_n(a.op, na, q, LP, false, st, pl)); });
        }
        return j;
    };
    auto reduce = [&](const Jobs& j) {      // of the partial results
        Jobs a = {};
        int na = 0;
        for (int i = 0; i < n; ++i) if (j.g[i].blocks == 0) a.g[na++] = j.g[i];
        if (na > 0) ops.push_back([=] { return launch_reduce_gram(a.g, na, LP, st); });
    };
    // next_t, next_pl: the product that takes Q
    auto gram_to_basis = [&](Jobs j, bool next_t, int next_pl) {
        bool sums = true;           // few partials: added where they are used
        for (int i = 0; i < n; ++i) {
            sums = sums && orth_apply_sums(j.g[i].blocks > 0 ? j.g[i].blocks : gram_blocks(j.g[i].n, LP), LP);
            if (in_steps(next_t, next_pl, i)) { j.g[i].steps = p->f[i].w.steps; j.g[i].steps_fmt = steps_format(LP, next_pl); }
        }
        if (!sums) ops.push_back([=] { return launch_gram_sum(j.g, n, LP, st); });
        ops.push_back([=] { return launch_orth_apply(j.g, n, ell, LP, sums, st); });
    };
    auto orth = [&](const Jobs& j, bool next_t, int next_pl) {
        reduce(j);
        gram_to_basis(j, next_t, next_pl);
    };
    const int t_first = power_iters > 0 ? planes : planes_last;      // planes of the first transposed product
    // Y = R Omega
    if (first == FirstPass::one_read) {
        const Factor f = p->f[0];
        if (one_read_projects(power_iters, stop_at_basis, f.op.cols, rank)) {
            // R^T Q = (R^T Y) T: nothing reads the operand again, unless Y shows that this would be less accurate than R^T Q
            const int blocks = quant_project_blocks(f.op.rows);
            double *const gsum = f.w.M, *const msum = gsum + PROJECT_GROUPS * 256;
            GramJob g = {nullptr, 0, f.op.rows, f.op.Y, gsum, f.w.gram, PROJECT_GROUPS, 0};
            g.M = msum; g.Z = f.op.W; g.m = f.op.cols; g.again = f.w.again;
            PassOperand rtq = f.op;
            rtq.run = f.w.again;
            ops.push_back([=] {
                return launch_quant_project_rows(f.op.X, f.op.ldx, f.op.rows, f.op.cols, q, f.op.W, LP, f.op.Y, f.w.gpart, f.w.mpart,
                                                 one_read_amax, f.w.lam, f.w.s, f.op.codes, st);
            });
            ops.push_back([=] { return launch_project_sum(f.w.gpart, f.w.mpart, blocks, f.op.cols, gsum, msum, st); });
            ops.push_back([=] { return launch_orth_apply(&g, 1, ell, LP, true, st); });
            ops.push_back([=] { return launch_resid_mul_t(&rtq, 1, q, LP, st); });
            return;
        }
        ops.push_back([=] {
            return launch_quant_sketch_rows(f.op.X, f.op.ldx, f.op.rows, f.op.cols, q, f.op.W, LP, f.op.Y, f.w.gpart,
                                            one_read_amax, f.w.lam, f.w.s, f.op.codes, st);
        });
        Jobs j = {};
        j.g[0] = {nullptr, 0, f.op.rows, f.op.Y, f.w.gpart, f.w.gram, quant_sketch_rows_blocks(f.op.rows), 0};
        gram_to_basis(j, true, t_first);
    } else {
        const bool quantizing = first == FirstPass::quantize;
        // (the sketch is not in the order of steps)
        Jobs j = {};
        for (int i = 0; i < n; ++i) {
            const Factor& f = p->f[i];
            j.g[i] = {f.w.partial, f.op.pn.splits, f.op.rows, f.op.Y, f.w.gpart, f.w.gram, 0, 0};
        }
        ops.push_back([=] { return launch_resid_mul_n(p->op, n, q, LP, quantizing, st, planes_first, packed); });
        orth(j, true, t_first);
    }
    for (int it = 0; it < power_iters; ++it) {
        // Z = orth(R^T Q); Q = orth(R Z)
        orth(product(true, planes), false, planes);
        orth(product(false, planes), true, it + 1 < power_iters ? planes : planes_last);
    }
    // B^T = R^T Q (cols x l), its Gram B B^T, small SVD, U = Q U', V = B^T U' / sigma
    const Jobs j = product(true, planes_last);
    if (stop_at_basis) return;
    if (basis_suffices) {
        ops.push_back([=] {
            BasisJob bj[2];
            for (int i = 0; i < n; ++i) {
                const Factor& f = p->f[i];
                const TPartials t = t_partials(f, planes_last);
                bj[i] = {t.p, t.splits, f.op.cols, f.op.Y, f.op.rows, f.U, f.Sigma, f.Vt};
            }
            return launch_take_basis(bj, n, LP, rank, st);
        });
        return;
    }
    reduce(j);
    ops.push_back([=] { return launch_gram_sum(j.g, n, LP, st); });
    if (svd_index) *svd_index = ops.size();         // the GPU is nearly idle from this launch to its end
    ops.push_back([=] {
        SvdJob sj[2];
        for (int i = 0; i < n; ++i) sj[i] = {p->f[i].w.gram, p->f[i].Sigma, p->f[i].w.Ur, p->f[i].w.Mv};
        return launch_small_svd(sj, n, ell, LP, rank, st);
    });
    ops.push_back([=] {
        ApplyJob aj[4];
        for (int i = 0; i < n; ++i) {
            const Factor& f = p->f[i];
            aj[2 * i] = {f.op.Y, f.w.Ur, f.U, f.op.rows, rank, rank, rank, 0};
            aj[2 * i + 1] = {f.op.W, f.w.Mv, f.Vt, f.op.cols, rank, rank, f.op.cols, 1};
        }
        return launch_apply(aj, 2 * n, LP, st);
    });
}

#define LRQ_TRY(x)                  \
    do {                            \
        rc = (x);                   \
        if (rc != LRQMM_OK) return rc; \
    } while (0)

}  // namespace

extern "C" {

const char* lrqmm_status_string(int status) {
    switch (status) {
        case LRQMM_OK: return "ok";
        case LRQMM_ERR_INVALID_ARG: return "invalid argument";
        case LRQMM_ERR_UNSUPPORTED: return "unsupported configuration";
        case LRQMM_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
        case LRQMM_ERR_HIP: return "HIP launch failed";
        case LRQMM_ERR_STATIC_LIMIT: return "problem needs more scratch memory than the library's static buffer holds";
        default: return "unknown status";
    }
}

size_t lrqmm_workspace_bytes(int M, int N, int K, int rank, int oversample) {
    if (M < 0 || N < 0 || K < 0 || rank < 0 || oversample < 0 || !dims_ok(M, N, K) || !output_ok(M, N)) return 0;
    if (rank + oversample > LRQMM_MAX_SKETCH) return 0;
    Arena a(nullptr);
    return carve_matmul(a, M, N, K, rank, oversample, nullptr) + 256;
}

int lrqmm_quantize(const float* X, int rows, int cols, int axis, int bits, int round_mode, int8_t* codes,
                   float* amax, void* stream) {
    return lrqmm_quantize_ex(X, cols, rows, cols, axis, bits, round_mode, LRQMM_SCALE_VECTOR, codes, amax, stream);
}

int lrqmm_quantize_ex(const float* X, int ldx, int rows, int cols, int axis, int bits, int round_mode,
                      int scale_mode, int8_t* codes, float* amax, void* stream) {
    if (rows < 0 || cols < 0 || ldx < cols) return LRQMM_ERR_INVALID_ARG;
    if (!dims_ok(rows, cols)) return LRQMM_ERR_UNSUPPORTED;
    if (scale_mode != LRQMM_SCALE_VECTOR && scale_mode != LRQMM_SCALE_TENSOR) return LRQMM_ERR_INVALID_ARG;
    if (axis != LRQMM_AXIS_ROW && axis != LRQMM_AXIS_COL) return LRQMM_ERR_INVALID_ARG;
    if (round_mode != LRQMM_ROUND_FLOOR && round_mode != LRQMM_ROUND_NEAREST) return LRQMM_ERR_INVALID_ARG;
    if (!bits_ok(bits)) return LRQMM_ERR_UNSUPPORTED;
    if (rows == 0 || cols == 0) return LRQMM_OK;
    if (!X || !codes || !amax) return LRQMM_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const QuantParams q = make_quant_params(bits, round_mode);
    const bool per_tensor = scale_mode == LRQMM_SCALE_TENSOR;
    if (axis == LRQMM_AXIS_ROW) return launch_quantize_rows(X, ldx, rows, cols, q, per_tensor, nullptr, codes, amax, st);
    return launch_quantize_cols(X, ldx, rows, cols, q, per_tensor, nullptr, codes, amax, st);
}

int lrqmm_quantize_residual(const float* X, int ldx, const float* amax0, int rows, int cols, int axis, int bits,
                            int round_mode, int scale_mode, int8_t* codesR, float* amaxR, void* stream) {
    if (rows < 0 || cols < 0 || ldx < cols) return LRQMM_ERR_INVALID_ARG;
    if (!dims_ok(rows, cols)) return LRQMM_ERR_UNSUPPORTED;
    if (scale_mode != LRQMM_SCALE_VECTOR && scale_mode != LRQMM_SCALE_TENSOR) return LRQMM_ERR_INVALID_ARG;
    if (axis != LRQMM_AXIS_ROW && axis != LRQMM_AXIS_COL) return LRQMM_ERR_INVALID_ARG;
    if (round_mode != LRQMM_ROUND_FLOOR && round_mode != LRQMM_ROUND_NEAREST) return LRQMM_ERR_INVALID_ARG;
    if (!bits_ok(bits)) return LRQMM_ERR_UNSUPPORTED;
    if (rows == 0 || cols == 0) return LRQMM_OK;
    if (!X || !amax0 || !codesR || !amaxR || amax0 == amaxR) return LRQMM_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const QuantParams q = make_quant_params(bits, round_mode);
    const bool per_tensor = scale_mode == LRQMM_SCALE_TENSOR;
    if (axis == LRQMM_AXIS_ROW) return launch_quantize_rows(X, ldx, rows, cols, q, per_tensor, amax0, codesR, amaxR, st);
    return launch_quantize_cols(X, ldx, rows, cols, q, per_tensor, amax0, codesR, amaxR, st);
}

int lrqmm_fill_sketch(uint64_t seed, int stream_id, int rows, int cols, float* omega, void* stream) {
    if (rows < 0 || cols < 0 || stream_id < 0) return LRQMM_ERR_INVALID_ARG;
    if (!dims_ok(rows, cols)) return LRQMM_ERR_UNSUPPORTED;
    if (rows == 0 || cols == 0) return LRQMM_OK;
    if (!omega) return LRQMM_ERR_INVALID_ARG;
    return launch_fill_sketch(seed, stream_id, rows, cols, cols, omega, static_cast<hipStream_t>(stream));
}

int lrqmm_rsvd(const float* X, const float* amax, int rows, int cols, int axis, int bits, int round_mode,
               int rank, int oversample, int power_iters, uint64_t seed, const float* omega_or_null, float* U,
               float* Sigma, float* Vt, void* workspace, size_t workspace_bytes, void* stream) {
    return lrqmm_rsvd_ex(X, cols, amax, rows, cols, axis, bits, round_mode, rank, oversample, power_iters, seed,
                         omega_or_null, LRQMM_DEFAULT_PREC, U, Sigma, Vt, workspace, workspace_bytes, stream);
}

int lrqmm_rsvd_ex(const float* X, int ldx, const float* amax, int rows, int cols, int axis, int bits, int round_mode,
                  int rank, int oversample, int power_iters, uint64_t seed, const float* omega_or_null, int precision,
                  float* U, float* Sigma, float* Vt, void* workspace, size_t workspace_bytes, void* stream) {
    if (rows < 0 || cols < 0 || rank < 1 || oversample < 0 || power_iters < 0 || ldx < cols) return LRQMM_ERR_INVALID_ARG;
    if (!dims_ok(rows, cols)) return LRQMM_ERR_UNSUPPORTED;
    if (!precision_ok(precision)) return LRQMM_ERR_INVALID_ARG;
    if (axis != LRQMM_AXIS_ROW && axis != LRQMM_AXIS_COL) return LRQMM_ERR_INVALID_ARG;
    if (round_mode != LRQMM_ROUND_FLOOR && round_mode != LRQMM_ROUND_NEAREST) return LRQMM_ERR_INVALID_ARG;
    if (!bits_ok(bits)) return LRQMM_ERR_UNSUPPORTED;
    if (rows == 0 || cols == 0) return LRQMM_OK;
    const int ell = rank + oversample;
    if (ell > rows || ell > cols) return LRQMM_ERR_INVALID_ARG;
    if (ell > LRQMM_MAX_SKETCH) return LRQMM_ERR_UNSUPPORTED;
    if (!X || !amax || !U || !Sigma || !Vt) return LRQMM_ERR_INVALID_ARG;
    if (!workspace || ((uintptr_t)workspace & 255)) return LRQMM_ERR_WORKSPACE;
    const int LP = pad_to(ell, 16);
    Factor f;
    const int rc = make_factor(&f, X, ldx, rows, cols, axis, LP, rank, amax, nullptr, U, Sigma, Vt, workspace, workspace_bytes);
    if (rc != LRQMM_OK) return rc;
    const QuantParams q = make_quant_params(bits, round_mode);
    const int nscale = axis == LRQMM_AXIS_ROW ? rows : cols;
    hipStream_t st = static_cast<hipStream_t>(stream);
    LaunchList ops;
    if (omega_or_null) {
        ops.push_back([=] { return launch_scales(amax, nscale, pad_to(nscale, 4), q.qmaxf, f.w.lam, f.w.s, st); });
        ops.push_back([=] { return launch_pad_copy(omega_or_null, cols, ell, LP, f.w.Wc, st); });
    } else {
        ops.push_back([=] {
            return launch_sketch_and_scales(seed, axis, cols, ell, LP, f.w.Wc, amax, nscale, pad_to(nscale, 4), q.qmaxf,
                                            f.w.lam, f.w.s, st);
        });
    }
    factor_launches(ops, &f, 1, FirstPass::plain, q, rank, oversample, power_iters, planes_subspace(precision),
                    planes_subspace(precision), planes_values(precision), st, nullptr);
    return run_interleaved(ops, LaunchList());
}

static int gemm_impl(int M, int N, int K, int bits, int rank, const int8_t* Aq, const float* amaxA,
                     const int8_t* BqT, const float* amaxB, const float* U, const float* Sig, const float* Vt,
                     const float* W, const float* Gam, const float* Zt, GemmOut out, int32_t* Cint_or_null,
                     void* workspace, size_t workspace_bytes, void* stream, int prof_slot,
                     hipEvent_t raw_sums_ready = nullptr, int planes = 3, int packed = PK_NONE, const PanelArgs* ready = nullptr) {
    float* const C = out.C;
    if (M < 0 || N < 0 || K < 0 || rank < 0 || out.ldc < N) return LRQMM_ERR_INVALID_ARG;
    if (!dims_ok(M, N, K) || !output_ok(M, N)) return LRQMM_ERR_UNSUPPORTED;
    if (!bits_ok(bits)) return LRQMM_ERR_UNSUPPORTED;
    if (!k_fits_int32(K, bits)) return LRQMM_ERR_UNSUPPORTED;
    if (M == 0 || N == 0) return LRQMM_OK;
    if (rank > K || rank > M || rank > N) return LRQMM_ERR_INVALID_ARG;
    if (rank > LRQMM_MAX_SKETCH) return LRQMM_ERR_UNSUPPORTED;
    if (!C || !amaxA || !amaxB || (K > 0 && (!Aq || !BqT))) return LRQMM_ERR_INVALID_ARG;
    if (rank > 0 && (!U || !Sig || !Vt || !W || !Gam || !Zt)) return LRQMM_ERR_INVALID_ARG;
    if (!workspace || ((uintptr_t)workspace & 255)) return LRQMM_ERR_WORKSPACE;
    GemmWs w;
    Arena a(workspace);
    if (carve_gemm(a, M, N, K, rank, &w) > workspace_bytes) return LRQMM_ERR_WORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (K == 0) {
        // An empty reduction: C_F = 0 (rank <= K leaves no compensation either), so only the update
        // D <- alpha * 0 + beta * D remains.  No operand is read and no GEMM kernel is launched.
        prof_mark(prof_slot, 7, st);
        const int r0 = launch_empty_product(M, N, out, Cint_or_null, st);
        for (int e = 8; e <= 10; ++e) prof_mark(prof_slot, e, st);
        return r0;
    }
    const QuantParams q = make_quant_params(bits, 0);
    int rc;
    int R2P = 0;
    const int RP = pad_to(rank, 16);
    if (rank > 0) {
        R2P = pad_to(2 * rank, 8);
        PanelArgs pa = {Aq, BqT, w.Wf, w.Vf, U, Sig, w.sA, w.sB, w.X, Gam, Zt, w.Lp, w.Rp, M, N, K, rank, R2P};
        pa.nslices = ceil_div(K, ceil_div(K, vtw_slices(K)));
        pa.ldu = rank;
        if (ready) pa = *ready;
        else LRQ_TRY(launch_panel_prep(M, N, K, rank, RP, q.qmaxf, amaxA, amaxB, W, Vt, w.lamA, w.sA, w.lamB, w.sB, w.Wf, w.Vf, w.X, st));
        w.sA = const_cast<float*>(pa.sA);
        w.sB = const_cast<float*>(pa.sB);
        LRQ_TRY(launch_panels(pa, RP, K % 16 == 0 ? planes : 3, packed, st));       // (as the interface states)
    }
    if (raw_sums_ready) {
        // the integer product ran early on another stream and left its int32 sums in C
        if (hipStreamWaitEvent(st, raw_sums_ready, 0) != hipSuccess) return LRQMM_ERR_HIP;
        prof_mark(prof_slot, 7, st);
        rc = launch_rank_update(M, N, C, w.sA, w.sB, w.Lp, w.Rp, R2P, out.alpha, st);
        prof_mark(prof_slot, 8, st);
        return rc;
    }
    prof_mark(prof_slot, 7, st);
    rc = launch_int8_gemm(M, N, K, Aq, BqT, rank > 0 ? w.sA : amaxA, rank > 0 ? w.sB : amaxB, rank > 0 ? w.Lp : nullptr,
                          rank > 0 ? w.Rp : nullptr, R2P, out, Cint_or_null, q.qmaxf, st, packed);
    prof_mark(prof_slot, 8, st);
    prof_mark(prof_slot, 9, st);
    prof_mark(prof_slot, 10, st);
    return rc;
}

int lrqmm_gemm(int M, int N, int K, int bits, int rank, const int8_t* Aq, const float* amaxA,
               const int8_t* BqT, const float* amaxB, const float* U, const float* Sig, const float* Vt,
               const float* W, const float* Gam, const float* Zt, float* C, int32_t* Cint_or_null,
               void* workspace, size_t workspace_bytes, void* stream) {
    return lrqmm_gemm_ex(M, N, K, bits, rank, Aq, amaxA, BqT, amaxB, U, Sig, Vt, W, Gam, Zt, 1.0f, 0.0f, C, N,
                         Cint_or_null, workspace, workspace_bytes, stream);
}

int lrqmm_gemm_ex(int M, int N, int K, int bits, int rank, const int8_t* Aq, const float* amaxA,
                  const int8_t* BqT, const float* amaxB, const float* U, const float* Sig, const float* Vt,
                  const float* W, const float* Gam, const float* Zt, float alpha, float beta, float* D, int ldd,
                  int32_t* Cint_or_null, void* workspace, size_t workspace_bytes, void* stream) {
    const GemmOut out = {D, ldd, alpha, beta};
    return gemm_impl(M, N, K, bits, rank, Aq, amaxA, BqT, amaxB, U, Sig, Vt, W, Gam, Zt, out, Cint_or_null,
                     workspace, workspace_bytes, stream, -1);
}

int lrqmm_gemm_static(int M, int N, int K, int bits, int rank, const int8_t* Aq, const float* amaxA,
                      const int8_t* BqT, const float* amaxB, const float* U, const float* Sig, const float* Vt,
                      const float* W, const float* Gam, const float* Zt, float alpha, float beta, float* D, int ldd,
                      int32_t* Cint_or_null, void* stream) {
    if (M < 0 || N < 0 || K < 0 || rank < 0 || ldd < N) return LRQMM_ERR_INVALID_ARG;
    if (!dims_ok(M, N, K) || !output_ok(M, N)) return LRQMM_ERR_UNSUPPORTED;
    if (rank > LRQMM_MAX_SKETCH) return LRQMM_ERR_UNSUPPORTED;
    if (M == 0 || N == 0) return LRQMM_OK;
    // (which problems fit is part of the interface: the limit still counts regions that the kernels no longer need, two of K x
    // RP float32 values and the partial results of the code products)
    Arena a(nullptr);
    const int RP = pad_to(rank, 16);
    a.take<float>((size_t)K * RP);
    a.take<float>((size_t)K * RP);
    if (rank > 0) {
        a.take<float>((size_t)codes_splits(M, K) * M * RP);
        a.take<float>((size_t)codes_splits(N, K) * N * RP);
    }
    if (carve_gemm(a, M, N, K, rank, nullptr) > (size_t)LRQMM_STATIC_SCRATCH_BYTES) return LRQMM_ERR_STATIC_LIMIT;
    void* ws = nullptr;
    const int rc = static_scratch(&ws);
    if (rc != LRQMM_OK) return rc;
    const GemmOut out = {D, ldd, alpha, beta};
    return gemm_impl(M, N, K, bits, rank, Aq, amaxA, BqT, amaxB, U, Sig, Vt, W, Gam, Zt, out, Cint_or_null, ws,
                     LRQMM_STATIC_SCRATCH_BYTES, stream, -1);
}

int lrqmm_matmul(int M, int N, int K, int bits, int rank, int oversample, int power_iters, uint64_t seed,
                 int round_mode, const float* A, const float* B, float* C, void* workspace,
                 size_t workspace_bytes, void* stream) {
    return lrqmm_matmul_ex(M, N, K, bits, rank, oversample, power_iters, seed, round_mode, LRQMM_SCALE_VECTOR,
                           LRQMM_DEFAULT_PREC, A, K, B, N, 1.0f, 0.0f, C, N, workspace, workspace_bytes, stream);
}

int lrqmm_matmul_ex(int M, int N, int K, int bits, int rank, int oversample, int power_iters, uint64_t seed,
                    int round_mode, int scale_mode, int precision, const float* A, int lda, const float* B, int ldb,
                    float alpha, float beta, float* D, int ldd, void* workspace, size_t workspace_bytes, void* stream) {
    float* const C = D;
    if (M < 0 || N < 0 || K < 0 || rank < 0 || oversample < 0 || power_iters < 0) return LRQMM_ERR_INVALID_ARG;
    if (!dims_ok(M, N, K) || !output_ok(M, N)) return LRQMM_ERR_UNSUPPORTED;
    if (!precision_ok(precision)) return LRQMM_ERR_INVALID_ARG;
    if (lda < K || ldb < N || ldd < N) return LRQMM_ERR_INVALID_ARG;
    if (scale_mode != LRQMM_SCALE_VECTOR && scale_mode != LRQMM_SCALE_TENSOR) return LRQMM_ERR_INVALID_ARG;
    if (round_mode != LRQMM_ROUND_FLOOR && round_mode != LRQMM_ROUND_NEAREST) return LRQMM_ERR_INVALID_ARG;
    if (!bits_ok(bits)) return LRQMM_ERR_UNSUPPORTED;
    if (!k_fits_int32(K, bits)) return LRQMM_ERR_UNSUPPORTED;
    if (M == 0 || N == 0) return LRQMM_OK;
    if (rank > 0) {
        const int ell = rank + oversample;
        if (ell > M || ell > N || ell > K) return LRQMM_ERR_INVALID_ARG;
        if (ell > LRQMM_MAX_SKETCH) return LRQMM_ERR_UNSUPPORTED;
    }
    if (!C || (K > 0 && (!A || !B))) return LRQMM_ERR_INVALID_ARG;
    if (!workspace || ((uintptr_t)workspace & 255)) return LRQMM_ERR_WORKSPACE;
    MatmulWs w;
    Arena a(workspace);
    if (carve_matmul(a, M, N, K, rank, oversample, &w) > workspace_bytes) return LRQMM_ERR_WORKSPACE;
    hipStream_t pst = static_cast<hipStream_t>(stream);
    // Under stream capture the call may only enqueue kernels, event records and event waits: it cannot
    // create its streams and events, and timing events do not belong in a graph.
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(pst, &capture) != hipSuccess) return LRQMM_ERR_HIP;
    const bool capturing = capture != hipStreamCaptureStatusNone;
    if (capturing && g_prof.on) return LRQMM_ERR_UNSUPPORTED;
    const bool factored = rank > 0 && K > 0;
    const QuantParams qp = make_quant_params(bits, round_mode);
    const bool per_tensor = scale_mode == LRQMM_SCALE_TENSOR;
    const int ell = rank + oversample, LP = pad_to(ell, 16);
    Side* const side = factored ? side_state(!capturing) : nullptr;
    if (factored && !side) return capturing ? LRQMM_ERR_UNSUPPORTED : LRQMM_ERR_HIP;
    // The two operands' factorizations advance together on the caller's stream, one launch per step for both, or (see
    // two_chains) B's runs on the side stream beside A's.  A tall operand with short rows (an im2col'd convolution:
    // K = 576) keeps its rows in registers -- maxima, codes and Y from a single read -- in a chain of its own.
    // (in every precision mode: the one-read pass runs in float32, which the reduced modes allow; see the row limit)
    const bool short_rows = factored && !per_tensor && quant_sketch_rows_usable(A, lda, M, K, LP, w.Aq);
    const bool one_read = short_rows && one_read_pays(M, K);
    // (Such an operand that is not tall enough stays in one stream whatever its size: its passes are short beside the 95 us of two.  Two
    // chains / together, us, l = 8: 24000 x 64 x 576 104 / 87, 24000 x 4096 x 576 266 / 264, 4000 x 24000 x 576 297 / 278, 300 x 24000 x 576 136 /
    // 113; one power iteration 24000 x 64 x 576 156 / 155, 24000 x 4096 x 576 336 / 339, 30000 x 1024 x 432 211 / 204, 300 x 24000 x 576 204 / 186.)
    const bool overlap = one_read || (factored && !short_rows && two_chains(M, N, K, LP, planes_subspace(precision)));
    // The one-read kernel leaves rows of bytes: its products are short and bound by the store of C.
    const bool pair = !factored && !per_tensor && quantize_pair_usable(M, N, K);
    const int packed = pair ? direct_format(M, N, K, bits) : (factored && !one_read ? packed_format(bits, K) : PK_NONE);
    const int slot = (g_prof.on && g_prof.ncalls < kProfMaxCalls) ? g_prof.ncalls++ : -1;
    hipStream_t bst = overlap ? side->stream : pst;
    // Early integer GEMM: with both factorizations in their single-workgroup SVD the GPU is
    // nearly idle, so the int8 product (which needs only the codes) runs there on a third
    // stream, leaves raw int32 sums in C, and the epilogue follows the panels as a kernel of
    // its own.  Used for problems on the large-tile kernel.
    // (the raw sums need D's memory: only when its old contents are not an input and it is dense)
    const bool early = factored && rank_update_usable(M, N, C) && beta == 0.0f && ldd == N &&
                       early_product(int8_gemm_tiles(M, N), side->cus, ell);
    // Nothing to truncate: C needs no more of a factorization than U diag(Sigma) Vt = Q (Q^T R), and the small SVD falls
    // away.  Up to 16 columns; a call with a wider sketch gives the bits of the separate quantize, rsvd and gemm calls (a
    // narrow one's first product differs from them anyway).
    const bool basis_suffices = oversample == 0 && LP == 16;
    const bool basis_panels = factored && basis_suffices && basis_slices(K) > 0;
    if (slot >= 0) g_prof.early[slot] = early;
    hipStream_t gst = early ? side->gemm_stream : pst;
    // Planned first and then issued (see LaunchList): opsA holds the chain of both operands, or A's beside opsB with B's.
    LaunchList opsA, opsB;
    Factor f[2] = {};
    size_t svd = 0, svdB = 0;       // positions of the small-SVD launches in opsA (and opsB)
    int rc;
    auto mark = [&](LaunchList& ops, int event, hipStream_t st) {
        if (slot >= 0) ops.push_back([=] { prof_mark(slot, event, st); return LRQMM_OK; });
    };
    // (the first product of such an operand is float32-accurate in every precision mode, on either path)
    const int pl = planes_subspace(precision), pl_last = planes_values(precision), pl_first = short_rows ? 3 : pl;
    mark(opsA, 0, pst);
    mark(overlap ? opsB : opsA, 3, bst);
    if (!factored) {
        if (pair) {
            opsA.push_back([=] {
                return launch_quantize_pair(A, lda, B, ldb, M, N, K, qp, QuantPair{w.Aq, w.BqT, w.amaxA, w.amaxB}, pst, packed);
            });
        } else if (K > 0) {
            opsA.push_back([=] { return lrqmm_quantize_ex(A, lda, M, K, LRQMM_AXIS_ROW, bits, round_mode, scale_mode, w.Aq, w.amaxA, pst); });
            opsA.push_back([=] { return lrqmm_quantize_ex(B, ldb, K, N, LRQMM_AXIS_COL, bits, round_mode, scale_mode, w.BqT, w.amaxB, pst); });
        } else {
            opsA.push_back([=] { return launch_pad_copy(nullptr, M, 0, 1, w.amaxA, pst); });
            opsA.push_back([=] { return launch_pad_copy(nullptr, N, 0, 1, w.amaxB, pst); });
        }
        for (int e : {1, 4, 2, 5}) mark(opsA, e, pst);
    } else {
        // The group maxima come first (one read of the operands); the operand's second read yields codes, step vectors and
        // the sketch product Y = R.Omega in one launch.  The sketches are filled beside the maxima.
        LRQ_TRY(make_factor(&f[0], A, lda, M, K, LRQMM_AXIS_ROW, LP, rank, w.amaxA, w.Aq, w.U, w.Sig, w.Vt, w.subA,
                            w.subA_bytes));
        LRQ_TRY(make_factor(&f[1], B, ldb, K, N, LRQMM_AXIS_COL, LP, rank, w.amaxB, w.BqT, w.W, w.Gam, w.Zt, w.subB,
                            w.subB_bytes));
        float *const WcA = f[0].w.Wc, *const WcB = f[1].w.Wc;
        float *const amaxA = w.amaxA, *const amaxB = w.amaxB;
        const FirstPass quant = FirstPass::quantize;
        if (overlap) {
            if (one_read) {
                opsA.push_back([=] { return launch_fill_sketch(seed, LRQMM_AXIS_ROW, K, ell, LP, WcA, pst); });
            } else {
                opsA.push_back([=] {
                    const SketchJob sk = {seed, LRQMM_AXIS_ROW, K, ell, LP, WcA};
                    return launch_absmax_pair(A, lda, M, K, amaxA, nullptr, 0, 0, nullptr, qp, per_tensor, &sk, 1, pst);
                });
            }
            mark(opsA, 1, pst);
            factor_launches(opsA, &f[0], 1, one_read ? FirstPass::one_read : quant, qp, rank, oversample, power_iters, pl_first,
                            pl, pl_last, pst, &svd, amaxA, basis_suffices, packed, basis_panels);
            opsB.push_back([=] {
                const SketchJob sk = {seed, LRQMM_AXIS_COL, N, ell, LP, WcB};
                return launch_absmax_pair(nullptr, 0, 0, K, nullptr, B, ldb, N, amaxB, qp, per_tensor, &sk, 1, bst);
            });
            mark(opsB, 4, bst);
            factor_launches(opsB, &f[1], 1, quant, qp, rank, oversample, power_iters, pl, pl, pl_last, bst, &svdB, nullptr,
                            basis_suffices, packed, basis_panels);
            mark(opsB, 5, bst);
        } else {
            opsA.push_back([=] {
                const SketchJob sk[2] = {{seed, LRQMM_AXIS_ROW, K, ell, LP, WcA}, {seed, LRQMM_AXIS_COL, N, ell, LP, WcB}};
                return launch_absmax_pair(A, lda, M, K, amaxA, B, ldb, N, amaxB, qp, per_tensor, sk, 2, pst);
            });
            mark(opsA, 1, pst);
            mark(opsA, 4, pst);
            factor_launches(opsA, f, 2, quant, qp, rank, oversample, power_iters, pl_first, pl, pl_last, pst, &svd, nullptr,
                            basis_suffices, packed, basis_panels);
            mark(opsA, 5, pst);
        }
        mark(opsA, 2, pst);
    }

    // Nothing has been enqueued so far.  From the fork on, every path -- errors included -- joins the
    // library's streams back into the caller's, so that a capture is never left with an open branch
    // and a later call never meets work of a failed one.
    bool forked = false, gemm_forked = false;
    auto issue = [&]() -> int {
        int rc;
        if (overlap) {
            if (hipEventRecord(side->fork, pst) != hipSuccess) return LRQMM_ERR_HIP;
            forked = true;
            if (hipStreamWaitEvent(bst, side->fork, 0) != hipSuccess) return LRQMM_ERR_HIP;
        }
        if (!early) return run_interleaved(opsA, opsB);
        // everything that precedes the small SVDs
        LRQ_TRY(run_interleaved(opsA, 0, svd, opsB, 0, svdB));
        // The gates are recorded before anything waits on them: the integer product needs both operands' codes, and
        // starting it behind the kernels that precede the SVDs keeps it out of the passes' way.
        if (hipEventRecord(side->gate, pst) != hipSuccess) return LRQMM_ERR_HIP;
        if (overlap && hipEventRecord(side->gate_b, bst) != hipSuccess) return LRQMM_ERR_HIP;
        LRQ_TRY(opsA[svd]());
        if (overlap) LRQ_TRY(opsB[svdB]());
        gemm_forked = true;
        if (hipStreamWaitEvent(gst, side->gate, 0) != hipSuccess) return LRQMM_ERR_HIP;
        if (overlap && hipStreamWaitEvent(gst, side->gate_b, 0) != hipSuccess) return LRQMM_ERR_HIP;
        // The product must not take the CUs before the two SVD workgroups have theirs: a few minimal
        // kernels give the SVD launches (one dependent launch behind the gates) a head start.  The
        // two SVD workgroups hold a CU each while the product runs.
        const int resident = side->cus - 2;
        for (int t = 0; t < 3; ++t) LRQ_TRY(launch_tick(w.tick, gst));
        prof_mark(slot, 9, gst);
        rc = launch_int8_gemm_sums(M, N, K, w.Aq, w.BqT, reinterpret_cast<int32_t*>(C), resident, w.parts, gst, packed);
        prof_mark(slot, 10, gst);
        if (rc != LRQMM_OK) return rc;
        LRQ_TRY(launch_int8_gemm_sums_finish(M, N, K, w.Aq, w.BqT, reinterpret_cast<int32_t*>(C), resident, w.parts, gst));
        if (hipEventRecord(side->gdone, gst) != hipSuccess) return LRQMM_ERR_HIP;
        return run_interleaved(opsA, svd + 1, opsA.size(), opsB, overlap ? svdB + 1 : 0, opsB.size());
    };
    rc = issue();
    if (forked) {
        if (hipEventRecord(side->join, bst) != hipSuccess || hipStreamWaitEvent(pst, side->join, 0) != hipSuccess)
            rc = rc != LRQMM_OK ? rc : LRQMM_ERR_HIP;
    }
    if (rc == LRQMM_OK) {
        prof_mark(slot, 6, pst);
        PanelArgs ready = {};
        if (basis_panels) {
            GemmWs g;
            Arena ga(w.sub);
            carve_gemm(ga, M, N, K, rank, &g);
            const TPartials ta = t_partials(f[0], pl_last, one_read && one_read_projects(power_iters, basis_panels, K, rank)), tb = t_partials(f[1], pl_last);
            rc = launch_basis_panels({ta.p, tb.p, f[1].op.Y, ta.splits, tb.splits, N, K, rank, ta.again, ta.p2, ta.splits2,
                                      g.Wf, g.Vf, w.Zt, g.X, w.Sig, w.Gam}, pst);
            ready = {w.Aq, w.BqT, g.Wf, g.Vf, f[0].op.Y, w.Sig, f[0].w.s, f[1].w.s, g.X, w.Gam, w.Zt, g.Lp, g.Rp, M, N, K, rank,
                     pad_to(2 * rank, 8), basis_slices(K), LP};
        }
        if (rc == LRQMM_OK) rc = gemm_impl(M, N, K, bits, rank, w.Aq, w.amaxA, w.BqT, w.amaxB, w.U, w.Sig, w.Vt, w.W, w.Gam, w.Zt,
                       GemmOut{D, ldd, alpha, beta}, nullptr, w.sub, w.sub_bytes, stream, slot,
                       early ? side->gdone : nullptr, planes_values(precision), packed, basis_panels ? &ready : nullptr);
    }
    if (rc != LRQMM_OK && gemm_forked) {
        // failed somewhere behind the fork of the third stream: join it too (a second record of the
        // event after a successful first one is harmless)
        (void)hipEventRecord(side->gdone, gst);
        (void)hipStreamWaitEvent(pst, side->gdone, 0);
    }
    return rc;
}

namespace {
struct ResidualWs {
    int8_t *Aq, *RAq, *BqT, *RBqT;
    float *amaxA, *amaxRA, *amaxB, *amaxRB;
    void* sub;
    size_t sub_bytes;
};
size_t carve_residual(Arena& a, int M, int N, int K, ResidualWs* w) {
    ResidualWs t = {};
    t.Aq = a.take<int8_t>(pk_bytes(M, K, PK8));
    t.RAq = a.take<int8_t>(pk_bytes(M, K, PK8));
    t.BqT = a.take<int8_t>(pk_bytes(N, K, PK8));
    t.RBqT = a.take<int8_t>(pk_bytes(N, K, PK8));
    t.amaxA = a.take<float>(M);
    t.amaxRA = a.take<float>(M);
    t.amaxB = a.take<float>(N);
    t.amaxRB = a.take<float>(N);
    a.off = align_up(a.off, 256);
    Arena g(nullptr);
    t.sub_bytes = carve_gemm(g, M, N, K, 0, nullptr);
    t.sub = a.base ? a.base + a.off : nullptr;
    a.off += t.sub_bytes;
    if (w) *w = t;
    return a.off;
}
}  // namespace

size_t lrqmm_residual_workspace_bytes(int M, int N, int K) {
    if (M < 0 || N < 0 || K < 0 || !dims_ok(M, N, K) || !output_ok(M, N)) return 0;
    Arena a(nullptr);
    return carve_residual(a, M, N, K, nullptr) + 256;
}

int lrqmm_residual_matmul(int M, int N, int K, int bits, int terms, int round_mode, int scale_mode, const float* A,
                          int lda, const float* B, int ldb, float alpha, float beta, float* D, int ldd,
                          void* workspace, size_t workspace_bytes, void* stream) {
    if (M < 0 || N < 0 || K < 0 || lda < K || ldb < N || ldd < N) return LRQMM_ERR_INVALID_ARG;
    if (!dims_ok(M, N, K) || !output_ok(M, N)) return LRQMM_ERR_UNSUPPORTED;
    if (terms != 1 && terms != 3 && terms != 4) return LRQMM_ERR_INVALID_ARG;
    if (round_mode != LRQMM_ROUND_FLOOR && round_mode != LRQMM_ROUND_NEAREST) return LRQMM_ERR_INVALID_ARG;
    if (scale_mode != LRQMM_SCALE_VECTOR && scale_mode != LRQMM_SCALE_TENSOR) return LRQMM_ERR_INVALID_ARG;
    if (!bits_ok(bits)) return LRQMM_ERR_UNSUPPORTED;
    if (!k_fits_int32(K, bits)) return LRQMM_ERR_UNSUPPORTED;
    if (M == 0 || N == 0) return LRQMM_OK;
    if (!D || (K > 0 && (!A || !B))) return LRQMM_ERR_INVALID_ARG;
    if (!workspace || ((uintptr_t)workspace & 255)) return LRQMM_ERR_WORKSPACE;
    ResidualWs w;
    Arena a(workspace);
    if (carve_residual(a, M, N, K, &w) > workspace_bytes) return LRQMM_ERR_WORKSPACE;
    if (K == 0) terms = 1;
    int rc, packed = PK_NONE;
    if (scale_mode == LRQMM_SCALE_VECTOR && quantize_pair_usable(M, N, K)) {
        if (terms == 4 && int8_terms_usable(M, N, K)) packed = terms_format(M, N, K, bits);
        QuantPair o = {w.Aq, w.BqT, w.amaxA, w.amaxB};
        if (terms >= 3) { o.codesRA = w.RAq; o.codesRB = w.RBqT; o.amaxRA = w.amaxRA; o.amaxRB = w.amaxRB; }
        LRQ_TRY(launch_quantize_pair(A, lda, B, ldb, M, N, K, make_quant_params(bits, round_mode), o,
                                     static_cast<hipStream_t>(stream), packed));
    } else if (K > 0) {
        LRQ_TRY(lrqmm_quantize_ex(A, lda, M, K, LRQMM_AXIS_ROW, bits, round_mode, scale_mode, w.Aq, w.amaxA, stream));
        LRQ_TRY(lrqmm_quantize_ex(B, ldb, K, N, LRQMM_AXIS_COL, bits, round_mode, scale_mode, w.BqT, w.amaxB, stream));
        if (terms >= 3) {
            LRQ_TRY(lrqmm_quantize_residual(A, lda, w.amaxA, M, K, LRQMM_AXIS_ROW, bits, round_mode, scale_mode, w.RAq,
                                            w.amaxRA, stream));
            LRQ_TRY(lrqmm_quantize_residual(B, ldb, w.amaxB, K, N, LRQMM_AXIS_COL, bits, round_mode, scale_mode, w.RBqT,
                                            w.amaxRB, stream));
        }
    } else {
        LRQ_TRY(launch_pad_copy(nullptr, M, 0, 1, w.amaxA, static_cast<hipStream_t>(stream)));
        LRQ_TRY(launch_pad_copy(nullptr, N, 0, 1, w.amaxB, static_cast<hipStream_t>(stream)));
    }
    if (terms >= 3 && int8_terms_usable(M, N, K)) {
        const int8_t *const Acodes[2] = {w.Aq, w.RAq}, *const Bcodes[2] = {w.BqT, w.RBqT};
        const float *const amA[2] = {w.amaxA, w.amaxRA}, *const amB[2] = {w.amaxB, w.amaxRB};
        return launch_int8_terms(M, N, K, Acodes, amA, Bcodes, amB, terms, make_quant_params(bits, round_mode).qmaxf,
                                 GemmOut{D, ldd, alpha, beta}, static_cast<hipStream_t>(stream), packed);
    }
    // one integer GEMM per term of Eq. (gemm_r_split), each dequantized with the scales of its two
    // operands and accumulated into D through the GEMM's own alpha/beta update
    auto term = [&](const int8_t* Lq, const float* amaxL, const int8_t* RqT, const float* amaxR, float b) {
        return gemm_impl(M, N, K, bits, 0, Lq, amaxL, RqT, amaxR, nullptr, nullptr, nullptr, nullptr, nullptr,
                         nullptr, GemmOut{D, ldd, alpha, b}, nullptr, w.sub, w.sub_bytes, stream, -1);
    };
    LRQ_TRY(term(w.Aq, w.amaxA, w.BqT, w.amaxB, beta));
    if (terms >= 3) {
        // alpha * term is added to what D holds now: beta = 1 from here on
        LRQ_TRY(term(w.Aq, w.amaxA, w.RBqT, w.amaxRB, 1.0f));
        LRQ_TRY(term(w.RAq, w.amaxRA, w.BqT, w.amaxB, 1.0f));
    }
    if (terms == 4) LRQ_TRY(term(w.RAq, w.amaxRA, w.RBqT, w.amaxRB, 1.0f));
    return LRQMM_OK;
}

int lrqmm_profile_enable(int on) {
    if (on && !g_prof.created) {
        for (int c = 0; c < kProfMaxCalls; ++c)
            for (int i = 0; i < kProfEvents; ++i)
                if (hipEventCreate(&g_prof.ev[c][i]) != hipSuccess) return LRQMM_ERR_HIP;
        g_prof.created = true;
    }
    g_prof.on = on != 0;
    g_prof.gemm_only = on == LRQMM_PROF_GEMM_ONLY;
    g_prof.ncalls = 0;
    return LRQMM_OK;
}

int lrqmm_profile_read(float* stage_ms, int* ncalls) {
    if (!stage_ms || !ncalls) return LRQMM_ERR_INVALID_ARG;
    const int n = g_prof.ncalls;
    *ncalls = n;
    for (int i = 0; i < kProfStages; ++i) stage_ms[i] = 0.f;
    if (n == 0) return LRQMM_OK;
    if (g_prof.gemm_only) {
        // the caller has synchronized the stream of the calls (see the header); each call
        // contributes its GEMM to stage 6 (early product) or 5 (fused kernel)
        for (int c = 0; c < n; ++c) {
            const int b = g_prof.early[c] ? 9 : 7, stage = g_prof.early[c] ? 6 : 5;
            float ms = 0.f;
            if (hipEventSynchronize(g_prof.ev[c][b + 1]) != hipSuccess) return LRQMM_ERR_HIP;
            if (hipEventElapsedTime(&ms, g_prof.ev[c][b], g_prof.ev[c][b + 1]) != hipSuccess) return LRQMM_ERR_HIP;
            stage_ms[stage] += ms / (float)n;
        }
        g_prof.ncalls = 0;
        return LRQMM_OK;
    }
    if (hipEventSynchronize(g_prof.ev[n - 1][kLastMainEvent]) != hipSuccess) return LRQMM_ERR_HIP;
    for (int c = 0; c < n; ++c)
        for (int i = 0; i < kProfStages; ++i) {
            float ms = 0.f;
            if (hipEventElapsedTime(&ms, g_prof.ev[c][kStageBegin[i]], g_prof.ev[c][kStageEnd[i]]) != hipSuccess)
                return LRQMM_ERR_HIP;
            stage_ms[i] += ms / (float)n;
        }
    g_prof.ncalls = 0;
    return LRQMM_OK;
}

}  // extern "C"
