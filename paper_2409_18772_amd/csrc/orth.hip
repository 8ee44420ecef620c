// Orthonormalization and the small SVD of the randomized range finder (paper:
// Background 2.1 stage 1 "Q with orthogonal columns", Algorithm 1 (range basis and small SVD),
// truncation Eq. (k-svd)).
//
// The tall factors are l <= 80 columns wide, so all O(l^3) work happens on an
// l x l Gram matrix held in LDS by a single workgroup, in float64 (full-rate on
// this chip).  Orthonormalization is Cholesky-QR with the Gram matrix, the
// Cholesky factor, its inverse and the application Q = Y T all in float64; the
// small SVD is an eigen-solve of B B^T, by tridiagonalization (with a check of its result) and
// by cyclic Jacobi below five columns or where the check fails.  Accumulating the Gram in
// float64 keeps the squared condition number harmless (residual sketches have
// cond ~ 1e2..1e4).  Columns whose pivot vanishes (rank-deficient sketch, e.g. a
// zero residual) are dropped: the corresponding columns of Q are zero.
#include "kernels.h"
#include <type_traits>

// The kernels of this file are short links of a dependent chain and share the chip with the other operand's
// streaming passes or with the integer product, whose waves keep every SIMD busy.  Their waves ask for the
// highest issue priority on their SIMD (a property of the wave, set by an instruction of the kernel itself: the
// streams all stay at the default priority).  Measured: 4096^3, l = 40: 0.509 -> 0.494 ms per step; 16384^3,
// l = 80: 10.04 -> 9.97 ms.
__device__ __forceinline__ void raise_wave_priority() { __builtin_amdgcn_s_setprio(3); }

#define MAXL LRQMM_MAX_SKETCH
// Workgroups of orth_apply_kernel per job, at most: 100352 rows, 64 220 us per call, 256 210, 512 209; 8192 1878, 1855, 1855
#define ORTH_BLOCKS 256
#define ORTH_PER 2            // orth_apply_kernel adds up to 8 ORTH_PER Gram partials itself

// Workgroups of the Gram kernel, at most: 64 for wide sketches (each leaves an LP x LP float64 partial that a later
// kernel has to add up: ~1 MB in all at LP = 48), more for narrow sketches, whose partials are small -- a tall
// operand (10^5 rows at LP = 16) would otherwise keep 64 compute units busy for 25 tiles each.
static int gram_max_blocks(int LP) { return LP <= 16 ? 512 : (LP <= 32 ? 128 : 64); }

// 16-row workgroups as long as there are not too many of them (a few thousand rows: the kernel is one chain of load
// latency, sum, product, store, and short on a workgroup's share of the partials), whole 64-row tiles beyond.
static int gram_rows_per_block(int n, int LP) {
    const int cap = gram_max_blocks(LP);
    if (ceil_div(n, 16) <= cap) return 16;
    return ceil_div(ceil_div(n, cap), 64) * 64;
}

int gram_blocks(int n, int LP) { return max(1, ceil_div(n, gram_rows_per_block(n, LP))); }
int gram_blocks_most(int n, int LP) { return max(1, min(ceil_div(n, 16), gram_max_blocks(LP))); }

// Y = sum of the pass partials (fixed order); gpart[block] = float64 Gram matrix of the block's rows, formed on the
// float64 matrix cores (v_mfma_f64_16x16x4, layout as at apply_kernel) from a TR-row tile in LDS: the 16 x 16 blocks
// on and above the diagonal are dealt to the four waves, the rest is their mirror image.  Where a tile has fewer
// 16-byte groups than the workgroup has threads, SG threads share a group and add SG runs of the splits, combined in
// order.  The sums of a factor do not depend on the other job of the launch.
template <int NT, int TR>
__global__ __launch_bounds__(256) void reduce_gram_kernel(GramJob a, GramJob b, int nb0) {
    constexpr int LP = NT * 16;
    raise_wave_priority();
    constexpr int ld = LP + 1;
    constexpr int Q4 = LP / 4, Q = TR * Q4;                 // 16-byte groups per row and per tile
    constexpr int SG = Q >= 256 ? 1 : 256 / Q;
    constexpr int ITER = (Q * SG + 255) / 256;
    constexpr int NP = NT * (NT + 1) / 2, PW = (NP + 3) / 4;    // 16 x 16 blocks of the Gram matrix, per wave
    typedef double v4d __attribute__((ext_vector_type(4)));
    __shared__ float tile[TR * ld];
    __shared__ float4 runs[SG > 1 ? SG * Q : 1];
    const bool first = (int)blockIdx.x < nb0;
    const GramJob job = first ? a : b;
    const int blk = first ? blockIdx.x : blockIdx.x - nb0;
    const float* __restrict__ const partial = job.partial;
    const int n = job.n, splits = job.splits;
    const int rb = blk * job.rows_per_block;
    const int re = min(n, rb + job.rows_per_block);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int li = lane & 15, kq = lane >> 4;
    v4d acc[PW];
#pragma unroll
    for (int i = 0; i < PW; ++i) acc[i] = (v4d){0.0, 0.0, 0.0, 0.0};
    const size_t plane = (size_t)n * LP;
    for (int r0 = rb; r0 < re; r0 += TR) {
        if (r0 > rb) __syncthreads();
        // The splits are summed MAX_SPLITS at a time; the loads of a batch, over all of the thread's groups, are issued
        // before its first add (branch free: clamped row and split indices, masked afterwards).  SG == 1: split and tile
        // are the same for the whole workgroup, so an address is a scalar base and one 32-bit lane offset per group.
        // 158 registers at 48 columns and 64 rows: with 174 the kernel did not start beside two workgroups of the other
        // chain's R^T W pass (176 registers each of a SIMD's 512) and waited for one to end: 8192^3, 40 columns, 28 -> 18 us
        // per launch on average, the call 1.57 -> 1.49 ms.
        float4 v[ITER];
#pragma unroll
        for (int it = 0; it < ITER; ++it) v[it] = make_float4(0.f, 0.f, 0.f, 0.f);
        if constexpr (SG == 1) {
            uint32_t off[ITER];
#pragma unroll
            for (int it = 0; it < ITER; ++it) {
                const int e = min((int)threadIdx.x + 256 * it, Q - 1);
                off[it] = (uint32_t)(min(e / Q4, re - 1 - r0) * LP + (e % Q4) * 4);
            }
            // A short factor whose partner forces the 64-row tiles keeps the order of its own 16-row ones: nrun runs of the
            // splits, each summed from zero, added in order.  (All splits still load in one batch: run by run, the second
            // run's latency made a call of 1537 x 1021 x 2311 with 24 columns 1.4 % slower.)
            constexpr int RUNS16 = 16 * Q4 >= 256 ? 1 : 256 / (16 * Q4);
            const int nrun = RUNS16 > 1 && job.rows_per_block == 16 ? RUNS16 : 1;
            int run = 0, run_end = splits / nrun;
            float4 t[ITER];
#pragma unroll
            for (int it = 0; it < ITER; ++it) t[it] = make_float4(0.f, 0.f, 0.f, 0.f);
            auto flush = [&] {
#pragma unroll
                for (int it = 0; it < ITER; ++it) {
                    v[it].x += t[it].x; v[it].y += t[it].y; v[it].z += t[it].z; v[it].w += t[it].w;
                }
            };
            for (int s0 = 0; s0 < splits; s0 += MAX_SPLITS) {
                float4 p[MAX_SPLITS][ITER];
#pragma unroll
                for (int it = 0; it < ITER; ++it)
#pragma unroll
                    for (int sp = 0; sp < MAX_SPLITS; ++sp)
                        p[sp][it] = *reinterpret_cast<const float4*>(partial + (size_t)min(s0 + sp, splits - 1) * plane +
                                                                     (size_t)r0 * LP + off[it]);
                if constexpr (RUNS16 == 1) {
#pragma unroll
                    for (int it = 0; it < ITER; ++it)
#pragma unroll
                        for (int sp = 0; sp < MAX_SPLITS; ++sp)
                            if (s0 + sp < splits) {
                                t[it].x += p[sp][it].x; t[it].y += p[sp][it].y;
                                t[it].z += p[sp][it].z; t[it].w += p[sp][it].w;
                            }
                } else {
#pragma unroll
                    for (int sp = 0; sp < MAX_SPLITS; ++sp)
                        if (s0 + sp < splits) {
                            if (s0 + sp >= run_end) {       // (the same for the whole workgroup; runs may be empty)
                                flush();
                                do { ++run; run_end = (run + 1) * splits / nrun; } while (run_end <= s0 + sp);
#pragma unroll
                                for (int it = 0; it < ITER; ++it) t[it] = make_float4(0.f, 0.f, 0.f, 0.f);
                            }
#pragma unroll
                            for (int it = 0; it < ITER; ++it) {
                                t[it].x += p[sp][it].x; t[it].y += p[sp][it].y;
                                t[it].z += p[sp][it].z; t[it].w += p[sp][it].w;
                            }
                        }
                }
            }
            flush();
        } else {
            const int sg = threadIdx.x / Q, e = threadIdx.x % Q;
            const int longest = (splits + SG - 1) / SG, se = (sg + 1) * splits / SG;
            const float* src = partial + (size_t)min(r0 + e / Q4, re - 1) * LP + (e % Q4) * 4;
            for (int s0 = 0; s0 < longest; s0 += MAX_SPLITS) {
                const int sb = sg * splits / SG + s0;
                float4 p[MAX_SPLITS];
#pragma unroll
                for (int sp = 0; sp < MAX_SPLITS; ++sp)
                    p[sp] = *reinterpret_cast<const float4*>(src + (size_t)max(0, min(sb + sp, se - 1)) * plane);
#pragma unroll
                for (int sp = 0; sp < MAX_SPLITS; ++sp)
                    if (sb + sp < se) { v[0].x += p[sp].x; v[0].y += p[sp].y; v[0].z += p[sp].z; v[0].w += p[sp].w; }
            }
        }
        if (SG > 1) {
            runs[threadIdx.x] = v[0];       // (Q SG == 256)
            __syncthreads();
            if ((int)threadIdx.x < Q) {
#pragma unroll
                for (int sg = 1; sg < SG; ++sg) {
                    const float4 t = runs[sg * Q + threadIdx.x];
                    v[0].x += t.x; v[0].y += t.y; v[0].z += t.z; v[0].w += t.w;
                }
            }
        }
#pragma unroll
        for (int it = 0; it < ITER; ++it) {
            const int e = (int)threadIdx.x + 256 * it;
            if (e < Q) {
                const int rr = e / Q4, c = (e % Q4) * 4;
                const bool in = r0 + rr < re;
                if (in) *reinterpret_cast<float4*>(job.Y + (size_t)(r0 + rr) * LP + c) = v[it];
                float* t = tile + rr * ld + c;
                t[0] = in ? v[it].x : 0.f; t[1] = in ? v[it].y : 0.f; t[2] = in ? v[it].z : 0.f; t[3] = in ? v[it].w : 0.f;
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < PW; ++i) {
            const int p = wave + 4 * i;
            if (p < NP) {
                int ta = 0, o = p;
                while (o >= NT - ta) { o -= NT - ta; ++ta; }        // row ta of the upper triangle
                const int tb = ta + o;
#pragma unroll
                for (int st = 0; st < TR / 4; ++st) {
                    const float* row = tile + (4 * st + kq) * ld + li;
                    acc[i] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)row[16 * ta], (double)row[16 * tb], acc[i], 0, 0, 0);
                }
            }
        }
    }
    double* gp = job.gpart + (size_t)blk * LP * LP;
#pragma unroll
    for (int i = 0; i < PW; ++i) {
        const int p = wave + 4 * i;
        if (p < NP) {
            int ta = 0, o = p;
            while (o >= NT - ta) { o -= NT - ta; ++ta; }
            const int tb = ta + o;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int gi = 16 * ta + 4 * v + kq, gj = 16 * tb + li;
                gp[gi * LP + gj] = acc[i][v];
                if (ta != tb) gp[gj * LP + gi] = acc[i][v];
            }
        }
    }
}

// Gram matrix = the nb block partials summed by eight threads per entry: thread (part, e) adds the partials
// [part per, (part + 1) per) in order, per = ceil(nb / 8), BATCH loads in flight at a time, and the eight sums are
// added in the order of the parts.  Lanes 8 part + e of a wave: the loads of a part are 8 adjacent entries.
// BATCH = 8 for up to 64 partials: one batch, and few enough registers (under 64) for the waves to start beside
// two resident workgroups of the other operand's pass kernels, which leave about 80 registers per lane free on
// a SIMD -- a kernel with one thread per entry and 64 partials in 128 registers waited for a pass workgroup to
// drain first (16384^3: 58-121 us on average against 4 us alone; the partials were written by other workgroups on
// other XCDs, so every load is a long-latency miss and all loads of a batch are issued before the first add).  BATCH = 16, 32 and 64 beyond that,
// so that up to 512 partials are one batch and no load of it is idle (125 partials with 64 loads a
// thread, 2000^3 l = 10 116.2 / 112.5 us per call; 1537 x 1021 x 2311 l = 24 172.5 / 168.2).
template <int BATCH>
__global__ __launch_bounds__(64) void gram_sum_parts_kernel(GramJob a, GramJob b, int entries) {
    raise_wave_priority();
    const GramJob job = blockIdx.y == 0 ? a : b;
    const double* __restrict__ const gpart = job.gpart;
    double* __restrict__ const gram = job.gram;
    const int nb = job.blocks;
    const int e = threadIdx.x & 7, part = threadIdx.x >> 3;
    const int idx = min((int)blockIdx.x * 8 + e, entries - 1);      // (past the end: the last entry again, not stored)
    const int per = (nb + 7) >> 3;
    const int b_begin = min(nb, part * per), b_end = min(nb, b_begin + per);
    const double* src = gpart + idx;
    double acc = 0.0;
    for (int b0 = b_begin; b0 < b_end; b0 += BATCH) {
        double v[BATCH];
#pragma unroll
        for (int blk = 0; blk < BATCH; ++blk) v[blk] = src[(size_t)min(b0 + blk, nb - 1) * entries];
#pragma unroll
        for (int blk = 0; blk < BATCH; ++blk) acc += (b0 + blk < b_end) ? v[blk] : 0.0;
    }
    double sum = __shfl(acc, e, 64);
#pragma unroll
    for (int p = 1; p < 8; ++p) sum += __shfl(acc, 8 * p + e, 64);
    if (part == 0 && (int)blockIdx.x * 8 + e < entries) gram[idx] = sum;
}

// Gram matrices and R^T Y of quant_project_rows_kernel's workgroups, added in float64 in PROJECT_GROUPS contiguous groups (orth_apply_kernel
// adds the groups): blockIdx.x 0 a group's Gram matrices, an entry a thread, the others 512 values of R^T Y each, two a thread.  480
// partials of 576 x 16: 5.3 us; a thread per 16 bytes of 16 partials, all groups at once, 24 us (128 bytes at a time of every partial).
__global__ __launch_bounds__(256) void project_sum_kernel(const double* __restrict__ gpart, const float* __restrict__ mpart, int blocks,
                                                          int values, double* __restrict__ gsum, double* __restrict__ msum) {
    constexpr int BATCH = 16;
    raise_wave_priority();
    const int b0 = (int)blockIdx.y * blocks / PROJECT_GROUPS, b1 = ((int)blockIdx.y + 1) * blocks / PROJECT_GROUPS;
    if (blockIdx.x == 0) {
        double acc = 0.0;
        for (int b = b0; b < b1; b += BATCH) {
            double v[BATCH];
#pragma unroll
            for (int u = 0; u < BATCH; ++u) v[u] = gpart[(size_t)min(b + u, b1 - 1) * 256 + threadIdx.x];
#pragma unroll
            for (int u = 0; u < BATCH; ++u) acc += b + u < b1 ? v[u] : 0.0;
        }
        gsum[(size_t)blockIdx.y * 256 + threadIdx.x] = acc;
        return;
    }
    const int at = ((int)blockIdx.x - 1) * 512 + 2 * threadIdx.x;
    if (at >= values) return;
    double ax = 0.0, ay = 0.0;
    for (int b = b0; b < b1; b += BATCH) {
        float2 v[BATCH];
#pragma unroll
        for (int u = 0; u < BATCH; ++u) v[u] = *reinterpret_cast<const float2*>(mpart + (size_t)min(b + u, b1 - 1) * values + at);
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            ax += b + u < b1 ? (double)v[u].x : 0.0;
            ay += b + u < b1 ? (double)v[u].y : 0.0;
        }
    }
    *reinterpret_cast<double2*>(msum + (size_t)blockIdx.y * values + at) = make_double2(ax, ay);
}

// out = In . Mat with float64 accumulation on the float64 matrix cores, one wavefront per 16
// rows.  v_mfma_f64_16x16x4 operand layout (lane l): A[i = l%16][k = l/16], B[k = l/16][j = l%16],
// D[i = 4v + l/16][j = l%16] for v = 0..3.  The reduction index may be visited in any order, so
// lane group l/16 takes the contiguous quarter [kq KQ, (kq+1) KQ) of the LP columns: a lane
// loads KQ consecutive floats of its row (the wavefront's 16 rows form one contiguous block)
// and, per step, one element of Mat.  Every wavefront reads all its rows before it writes any,
// so `out` may alias `In` (same leading dimension).
// Workgroups [0, nb[0]) work on job 0, the next nb[1] on job 1, and so on.
struct ApplyJobs {
    ApplyJob j[4];
    int nb[4];
};
template <int NT>
__global__ __launch_bounds__(64) void apply_kernel(ApplyJobs jobs) {
    constexpr int LP = NT * 16;
    raise_wave_priority();
    constexpr int KQ = LP / 4;
    int blk = blockIdx.x;
    ApplyJob job = jobs.j[0];
#pragma unroll
    for (int i = 1; i < 4; ++i)
        if (blk >= jobs.nb[i - 1]) { blk -= jobs.nb[i - 1]; job = jobs.j[i]; }
        else break;
    const float* __restrict__ In = job.In;
    const double* __restrict__ Mat = job.Mat;
    float* __restrict__ out = job.out;
    const int n = job.n, cm = job.cm, ldm = job.ldm, ldo = job.ldo, transposed = job.transposed;
    const int l = threadIdx.x, li = l & 15, kq = l >> 4;
    const int r0 = blk * 16;
    const int row = min(r0 + li, n - 1);
    const bool row_ok = r0 + li < n;
    float a[KQ];
    const float4* ip = reinterpret_cast<const float4*>(In + (size_t)row * LP + kq * KQ);
#pragma unroll
    for (int u = 0; u < KQ / 4; ++u) {
        const float4 t = ip[u];
        a[4 * u + 0] = row_ok ? t.x : 0.f;
        a[4 * u + 1] = row_ok ? t.y : 0.f;
        a[4 * u + 2] = row_ok ? t.z : 0.f;
        a[4 * u + 3] = row_ok ? t.w : 0.f;
    }
    typedef double v4d __attribute__((ext_vector_type(4)));
    v4d acc[NT];
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) acc[ct] = (v4d){0.0, 0.0, 0.0, 0.0};
    const int nct = (cm + 15) >> 4;         // column tiles that hold output
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) {
        if (ct < nct) {                     // uniform
            const int c = 16 * ct + li;
            const bool c_ok = c < cm;
            const double* mp = Mat + (size_t)(kq * KQ) * ldm + (c_ok ? c : 0);
            double b[KQ];
#pragma unroll
            for (int sidx = 0; sidx < KQ; ++sidx) {
                const double t = mp[(size_t)sidx * ldm];
                b[sidx] = c_ok ? t : 0.0;
            }
#pragma unroll
            for (int sidx = 0; sidx < KQ; ++sidx)
                acc[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)a[sidx], b[sidx], acc[ct], 0, 0, 0);
        }
    }
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) {
        const int c = 16 * ct + li;
        if (ct < nct && c < cm) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int orow = r0 + 4 * v + kq;
                if (orow < n) {
                    if (transposed) out[(size_t)c * ldo + orow] = (float)acc[ct][v];
                    else            out[(size_t)orow * ldo + c] = (float)acc[ct][v];
                }
            }
        }
    }
}

__device__ __forceinline__ double rcp_f64(double d) {       // hardware estimate and two Newton steps
    double q = __builtin_amdgcn_rcp(d);
    q = fma(fma(-d, q, 1.0), q, q);
    return fma(fma(-d, q, 1.0), q, q);
}

// Orthonormalization Q = Y T in one launch: every workgroup forms T = L^-T of the Gram matrix G = L L^T for itself, by
// symmetric elimination of the augmented matrix [G | I], and applies it to its rows of Y in place (on the float64 matrix
// cores, layout as at apply_kernel; the rows are loaded before the elimination starts).  Step j subtracts
// (M[i][j] / d_j) * (row j) from every row i > j, d_j the pivot M[j][j].  The left half is then L^T with rows unscaled (row j
// times sqrt(d_j)), the right half is L^-1 with row j unscaled the same way, so T[a][b] = M[b][LP + a] / sqrt(d_b).  A pivot
// below 1e-10 of its original diagonal (rank-deficient sketch) is dead: it eliminates nothing and its row and column of T
// are zero.
//
// 256 threads in a 16 x 16 grid (ti, tg) own rows ti + 16 ir and columns tg + 16 kc: pivot j = tj + 16 jr sits in register
// row and column jr, compile-time constants inside the unrolled jr loop.  Two pivots per step: pivots j and j + 1 share one
// publication in LDS (rows and columns j, j + 1 as they stand before pivot j; two generations) and one barrier, and every
// thread derives the effect of pivot j on row and column j + 1 itself before it applies both rank-1 updates; an odd l ends
// with a dead second pivot.  Updates that cannot change a value that is read later are left out at compile time (rows above
// the pivots, eliminated columns of G, columns of the identity half that are still zero).
//
// What bounds it: the chain of a step, LDS write -> barrier -> LDS read -> two reciprocals -> FMA, about 500 cycles.  T formed
// by one workgroup of l^2 / 16 workers in a launch of its own, and applied in another, took 10.5 + 4.7 us and a gap at 24
// columns, 15 + 6.4 at 40, 36 + 16 at 80 (those workers shared one to four SIMDs' LDS reads).  Calls with two launches / with
// one (one power iteration; the small SVD as it is now): 2048^3 l = 24 215 / 197 us, 40 296 / 270, 80 548 / 491; 4096^3 24
// 361 / 344, 40 444 / 417, 80 726 / 664; 8192^3 80 1902 / 1855; 16384^3 the same.  82 to 173 registers: the waves start
// beside resident workgroups of the other chain's passes (4096^3, l = 40, at 306 registers 433 us).
// parts > 0: G is still in that many partials (see gram_sum_parts_kernel, whose order of addition is kept).
struct OrthGrid { int nb, rows, parts, nbY; };  // workgroups of the job, rows per workgroup (a multiple of 64); [nbY, nb): 64 rows of M each
template <int NT>
__global__ __launch_bounds__(256, NT <= 2 ? 4 : (NT <= 4 ? 3 : 2)) void orth_apply_kernel(GramJob a0, GramJob a1, OrthGrid g0, OrthGrid g1, int ell) {
    constexpr int LP = 16 * NT, KC = 2 * NT, KQ = LP / 4, LDT = LP + 1;
    raise_wave_priority();
    const bool first = (int)blockIdx.x < g0.nb;
    const double* __restrict__ const gram = first ? a0.gram : a1.gram;
    const double* __restrict__ const gpart = first ? a0.gpart : a1.gpart;
    float* __restrict__ const Y = first ? a0.Y : a1.Y;
    const int n = first ? a0.n : a1.n, rows = first ? g0.rows : g1.rows, parts = first ? g0.parts : g1.parts;
    void* __restrict__ const steps = first ? a0.steps : a1.steps;
    const int steps_fmt = first ? a0.steps_fmt : a1.steps_fmt;
    const double* __restrict__ const M = first ? a0.M : a1.M;
    float* __restrict__ const Z = first ? a0.Z : a1.Z;
    const int nbY = first ? g0.nbY : g1.nbY, m = first ? a0.m : a1.m;
    int* __restrict__ const again = first ? a0.again : a1.again;
    const int blk = first ? blockIdx.x : blockIdx.x - g0.nb;
    __shared__ double rowb[2][2][2 * LP];
    __shared__ double colb[2][2][LP];
    __shared__ double thrb[2][2];
    __shared__ double Ts[LP * LDT];
    __shared__ double diag[NT == 1 ? LP : 1];           // squared lengths of Y's columns
    const int tid = threadIdx.x, ti = tid >> 4, tg = tid & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, li = lane & 15, kq = lane >> 4;
    const int row_end = min(steps_fmt ? (n + 31) & ~31 : n, (blk + 1) * rows);      // (steps end in zeros)
    // the wave's first 16 rows of Y: lane (li, kq) holds a quarter of row 4 (li % 4) + li / 4, so that the lane's four results are
    // adjacent rows
    float y[KQ];
    auto load_rows = [&](int r0) {
        const float4* ip = reinterpret_cast<const float4*>(Y + (size_t)min(r0 + 4 * (li & 3) + (li >> 2), n - 1) * LP + kq * KQ);
#pragma unroll
        for (int u = 0; u < KQ / 4; ++u) {
            const float4 t = ip[u];
            y[4 * u + 0] = t.x; y[4 * u + 1] = t.y; y[4 * u + 2] = t.z; y[4 * u + 3] = t.w;
        }
    };
    load_rows(blk * rows + wave * 16);
    double mreg[NT][KC];
    if (NT == 1 && parts > 0) {         // one entry per thread
        const int per = (parts + 7) >> 3;
        double v[8][ORTH_PER], sum = 0.0;
#pragma unroll
        for (int p = 0; p < 8; ++p)
#pragma unroll
            for (int u = 0; u < ORTH_PER; ++u) v[p][u] = gpart[(size_t)min(p * per + u, parts - 1) * (LP * LP) + tid];
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            double acc = 0.0;
#pragma unroll
            for (int u = 0; u < ORTH_PER; ++u) acc += (u < per && p * per + u < parts) ? v[p][u] : 0.0;
            sum = p == 0 ? acc : sum + acc;
        }
        mreg[0][0] = sum;
    } else {
#pragma unroll
        for (int ir = 0; ir < NT; ++ir)
#pragma unroll
            for (int kc = 0; kc < NT; ++kc) mreg[ir][kc] = gram[(ti + 16 * ir) * LP + tg + 16 * kc];
    }
    double thr[NT], pivot[NT];          // 1e-10 * original diagonal, on the threads that own it; pivots, 0 when dead
#pragma unroll
    for (int ir = 0; ir < NT; ++ir) {
        const int i = ti + 16 * ir;     // < LP; rows and columns >= ell enter as zeros
        thr[ir] = (i < ell && ti == tg) ? 1e-10 * mreg[ir][ir] : 0.0;
        pivot[ir] = 0.0;
        if (NT == 1 && ti == tg) diag[ti] = i < ell ? mreg[ir][ir] : 0.0;
#pragma unroll
        for (int kc = 0; kc < NT; ++kc) {
            const int c = tg + 16 * kc;
            if (i >= ell || c >= ell) mreg[ir][kc] = 0.0;
            mreg[ir][NT + kc] = (c == i && i < ell) ? 1.0 : 0.0;
        }
    }
    int par = 0;
    auto live_col = [](int kc, int jr) { return kc < NT ? kc >= jr : kc - NT <= jr; };
#pragma unroll
    for (int jr = 0; jr < NT; ++jr) {
        for (int tj = 0; tj < 16; tj += 2) {
            const int j = tj + 16 * jr;
            if (j >= ell) break;
            if (tg == tj || tg == tj + 1) {
#pragma unroll
                for (int ir = 0; ir < NT; ++ir)
                    if (ir >= jr) colb[par][tg - tj][ti + 16 * ir] = mreg[ir][jr];
            }
            if (ti == tj || ti == tj + 1) {
#pragma unroll
                for (int kc = 0; kc < KC; ++kc)
                    if (live_col(kc, jr)) rowb[par][ti - tj][tg + 16 * kc] = mreg[jr][kc];
                if (tg == ti) thrb[par][ti - tj] = thr[jr];
            }
            __syncthreads();
            double l[NT], x[NT], r0[KC], r1[KC];
            const double a = rowb[par][0][j], brow = rowb[par][0][j + 1], c11 = rowb[par][1][j + 1];
            const double lnext = colb[par][0][j + 1];
            const double thr0 = thrb[par][0], thr1 = thrb[par][1];
#pragma unroll
            for (int ir = 0; ir < NT; ++ir) {
                l[ir] = ir >= jr ? colb[par][0][ti + 16 * ir] : 0.0;
                x[ir] = ir >= jr ? colb[par][1][ti + 16 * ir] : 0.0;
            }
#pragma unroll
            for (int kc = 0; kc < KC; ++kc) {
                r0[kc] = live_col(kc, jr) ? rowb[par][0][tg + 16 * kc] : 0.0;
                r1[kc] = live_col(kc, jr) ? rowb[par][1][tg + 16 * kc] : 0.0;
            }
            const bool live0 = a > thr0 && a > 0.0;
            const double qa = live0 ? rcp_f64(a) : 0.0;
            const double f = -(lnext * qa);
            const double d1 = fma(f, brow, c11);
            const bool live1 = d1 > thr1 && d1 > 0.0;
            const double qd = live1 ? rcp_f64(d1) : 0.0;
            if (ti == tj) pivot[jr] = live0 ? a : 0.0;
            if (ti == tj + 1) pivot[jr] = live1 ? d1 : 0.0;
            double r1p[KC];
#pragma unroll
            for (int kc = 0; kc < KC; ++kc) r1p[kc] = live_col(kc, jr) ? fma(f, r0[kc], r1[kc]) : 0.0;
#pragma unroll
            for (int ir = 0; ir < NT; ++ir) {
                if (ir < jr) continue;          // rows above the pivots: nothing to eliminate
                const int i = ti + 16 * ir;
                const double lq = (i > j) ? -(l[ir] * qa) : 0.0;
                const double xi = fma(lq, brow, x[ir]);             // column j+1 after pivot j
                const double mq = (i > j + 1) ? -(xi * qd) : 0.0;
#pragma unroll
                for (int kc = 0; kc < KC; ++kc)
                    if (live_col(kc, jr)) mreg[ir][kc] = fma(mq, r1p[kc], fma(lq, r0[kc], mreg[ir][kc]));
            }
            par ^= 1;
        }
    }
#pragma unroll
    for (int ir = 0; ir < NT; ++ir) {
        const double pv = pivot[ir];
        double inv = 0.0;
        if (pv > 0.0) {      // 1/sqrt by the hardware estimate and three Newton steps
            inv = __builtin_amdgcn_rsq(pv);
            inv = inv * fma(-0.5 * pv, inv * inv, 1.5);
            inv = inv * fma(-0.5 * pv, inv * inv, 1.5);
            inv = inv * fma(-0.5 * pv, inv * inv, 1.5);
        }
#pragma unroll
        for (int kc = 0; kc < NT; ++kc) Ts[(tg + 16 * kc) * LDT + ti + 16 * ir] = mreg[ir][NT + kc] * inv;
    }
    __syncthreads();
    typedef double v4d __attribute__((ext_vector_type(4)));
    if (NT == 1 && again && blk == 0 && wave == 0) {
        double amp = 0.0;
#pragma unroll
        for (int s = 0; s < KQ; ++s) amp += fabs(Ts[(kq * KQ + s) * LDT + li]) * sqrt(diag[kq * KQ + s]);
        amp += __shfl_xor(amp, 16, 64);
        amp += __shfl_xor(amp, 32, 64);
        const double d = diag[li];              // (comparisons that fail for a NaN)
        const bool good = amp <= PROJECT_AMPLIFICATION && (d == 0.0 || (d >= PROJECT_LEAST && d <= PROJECT_MOST));
        const bool all = __all(good);
        if (lane == 0) *again = all ? 0 : 1;
    }
    if (NT == 1 && blk >= nbY) {
        const int r0 = (blk - nbY) * 64 + wave * 16;
        const double* mp = M + (size_t)min(r0 + li, m - 1) * LP + kq * KQ;
        double row[KQ];
#pragma unroll
        for (int s = 0; s < KQ; ++s) row[s] = 0.0;
#pragma unroll 4
        for (int p = 0; p < PROJECT_GROUPS; ++p)
#pragma unroll
            for (int s = 0; s < KQ; ++s) row[s] += mp[(size_t)p * m * LP + s];
        v4d acc = (v4d){0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < KQ; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(row[s], Ts[(kq * KQ + s) * LDT + li], acc, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (r0 + 4 * v + kq < m) Z[(size_t)(r0 + 4 * v + kq) * LP + li] = (float)acc[v];
        return;
    }
    for (int r0 = blk * rows + wave * 16; r0 < row_end; r0 += 64) {
#pragma unroll 1
        for (int ct = 0; ct < NT; ++ct) {           // (rolled: the elements of T of one column tile in registers at a time)
            v4d acc = (v4d){0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int s = 0; s < KQ; ++s)
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)y[s], Ts[(kq * KQ + s) * LDT + 16 * ct + li], acc, 0, 0, 0);
            float out[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int orow = r0 + 4 * kq + v;
                out[v] = orow < n ? (float)acc[v] : 0.f;
                if (orow < n) Y[(size_t)orow * LP + 16 * ct + li] = out[v];
            }
            const int half = (r0 >> 4) & 1;         // of the step
            if (NT == 1 && steps_fmt == STEPS_FLOAT) {
                *reinterpret_cast<float4*>(static_cast<float*>(steps) + (size_t)(r0 >> 5) * 512 + lane * 8 + 4 * half) =
                    make_float4(out[0], out[1], out[2], out[3]);
            } else if (steps_fmt == STEPS_PLANES) {
                uint16_t* dst = static_cast<uint16_t*>(steps) + ((size_t)(r0 >> 5) * NT + ct) * (3 * STEP_PIECE) + lane * 8 + 4 * half;
                uint32_t w[3][2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {       // (see split_planes)
                    const float a = out[2 * h], b = out[2 * h + 1];
                    w[0][h] = pack_bf16x2(a, b);
                    const float ra = a - __uint_as_float(w[0][h] << 16), rb = b - __uint_as_float(w[0][h] & 0xffff0000u);
                    w[1][h] = pack_bf16x2(ra, rb);
                    w[2][h] = pack_bf16x2(ra - __uint_as_float(w[1][h] << 16), rb - __uint_as_float(w[1][h] & 0xffff0000u));
                }
#pragma unroll
                for (int p = 0; p < 3; ++p) *reinterpret_cast<uint2*>(dst + p * STEP_PIECE) = make_uint2(w[p][0], w[p][1]);
            }
        }
        if (r0 + 64 < row_end) load_rows(r0 + 64);
    }
}

// Jacobi rotation that annihilates the off-diagonal entry of [[gpp, gpq], [gpq, gqq]]
// under G <- J^T G J with J = [[c, s], [-s, c]].  The angle is formed in float (an inexact
// angle still converges); c and s are then made orthonormal to float64 accuracy.
// Returns true when the entry was still "large" (|gpq| > 3e-4 sqrt(gpp gqq)) before the
// rotation: Jacobi converges quadratically, so a sweep that saw no large entry leaves
// off-diagonals of relative size ~1e-7 -- the resolution of the float32 factors that leave
// this kernel -- and is the last one (one sweep fewer than with a float64-level criterion,
// with the same distance to the float64 oracle).
__device__ __forceinline__ bool jacobi_rotation(double gpp, double gqq, double gpq, double gsc, double& c,
                                                double& s) {
    c = 1.0;
    s = 0.0;
    const float bf = (float)(2.0 * gpq * gsc);
    const double g2 = gpq * gpq, dd = fabs(gpp * gqq);
    if (!(g2 > 1e-24 * dd) || bf == 0.0f) return false;
    const bool large = g2 > 1e-7 * dd;
    const float th = (float)((gqq - gpp) * gsc) * __builtin_amdgcn_rcpf(bf);
    const float tf = copysignf(1.0f, th) * __builtin_amdgcn_rcpf(fabsf(th) + __builtin_amdgcn_sqrtf(th * th + 1.0f));
    const double t = (double)tf;
    const double x = fma(t, t, 1.0);
    double r = __builtin_amdgcn_rsq(x);
    r = r * fma(-0.5 * x, r * r, 1.5);
    r = r * fma(-0.5 * x, r * r, 1.5);
    c = r;
    s = t * r;
    return large;
}

// Cyclic Jacobi eigen-solve of the l x l matrix G = B B^T (B = Q^T R) with round-robin
// pairing, so l/2 disjoint rotations run per step.
//
// Tournament on m (even) players, circle method: positions 0..m-2 rotate, position m-1 is
// fixed, and slot i pairs positions (i, m-1-i); after a step the player at position c moves
// to c-1 (mod m-1), and position c holds player (step + c) mod (m-1).  G is stored BY SLOT
// (index i = first member of slot i, index half+i = its second member) and moved as part of
// the update (read from one LDS copy, written permuted to the other), so every read and
// write address of a thread is the same in every step: the loop carries no index
// arithmetic, and with a row stride = half (mod 32) consecutive threads hit consecutive
// LDS banks.  The eigenvector matrix is kept transposed and by player (Vt[player][component])
// and is updated in place with 16-byte accesses.  After a whole sweep the arrangement is
// the identity again.
//
// A step has one workgroup barrier:
//  * the update waves apply the step's rotations: thread (P, Q) updates the 2x2 block
//    (slot P rows, slot Q columns) of G <- J^T G J and two components of the column pair
//    of slot P of V <- V J;
//  * meanwhile the rotation wave (wave 0, one lane per pair of the NEXT step) forms the
//    three entries its next pair will have after this step's rotations, in registers, from
//    the copy being read, and derives the next rotation from them.
// Eigenvalues are the squared singular values of B, eigenvectors its left singular vectors.
#define SVD_UPDATE_THREADS 448
#define SVD_THREADS (64 + SVD_UPDATE_THREADS)
// Columns from which the tridiagonal solver is the faster one: l = 4 10.6 against 9.0 us (Jacobi), 5 11.1 / 12.6, 8 13.0 / 18.8
#define LRQ_TRI_MIN 5
// Below 32 columns a matrix whose diagonal spans more than this goes to the Jacobi solver at once: it keeps the small
// eigenvalues of a graded matrix to their own size, the tridiagonalization to roundings of the norm.  Largest entry of
// |V^T V - I| on 260 x 300 residuals, singular values down to 10^-x of the largest, tridiagonal / Jacobi: x = 4.75 1.9e-8 /
// 1.8e-8, 5 3.7e-8 / 1.9e-8, 5.5 4.2e-7 / 2.0e-8, 6 2.7e-6 / 1.5e-8; a flat tail at x = 4 1.6e-8 / 2.8e-7.  Time at 24 columns
// 109 / 123 us per factorization.  From 32 columns on the tridiagonal solver takes them all (5.5 at 64 and 80: 7.7e-7).
#define LRQ_TRI_GRADED 1e-9
#define LRQ_TRI_GRADED_BELOW 32

// Loop-invariant addresses of one 2x2 block task of an update thread.
struct SvdTask {
    int active;
    int P, Q;
    int o11, o12, o21, o22;     // read offsets in G (words)
    int w11, w12, w21, w22;     // write offsets in the other copy
    int v1, v2;                 // word offsets in Vt of the slot's two eigenvector columns
    int v1_wrap, v2_wrap, dv2;  // both run up one player (ldv words) per step and wrap after player m-2
};

// ---------------------------------------------------------------------------
// The small SVD proper: eigenpairs of the l x l matrix G = B B^T by tridiagonalization.
//   1. Householder tridiagonalization, G in the registers of one wave (above 40 columns two or four), see tridiagonalize.
//   2. Eigenvalues by multisection, four waves: every lane counts the eigenvalues below two points of its own (Sturm
//      sequence of the leading minors, rescaled every eighth row: one dependent FMA per row; the rows of T in registers up
//      to 40 columns), and ballots narrow all intervals by a factor 2 GL + 1 per round, to 2^-49 of the norm, and two rounds
//      further where an eigenvalue is small or two are close (a flat tail at 1e-2 of the top, whose vectors else failed the
//      check below: 24 columns 139 / 111 us per factorization, 80 columns 635 / 346).
//   3. Eigenvectors of the tridiagonal matrix by twisted factorization, one lane per vector: the LDU sweep from the top in
//      one wave, the one from the bottom in another; they meet at the index where the residual is smallest.
//   4. Back transformation by the Householder vectors, eight lanes per vector, no barrier.
//   5. S = U^T U on the float64 matrix cores.  Off I by more than 1e-11 (eigenvalues that nearly coincide): one step
//      U (3 I - S) / 2, which squares the deviation.  By more than 1e-4, or not a number (multiple eigenvalues, a
//      tridiagonal matrix that falls apart): the Jacobi solver below instead; zero rows and narrow graded matrices
//      (LRQ_TRI_GRADED) go there at once.
// Accuracy: eigenvalues to a few ulps of the largest one; ||G u - s u|| likewise.
// Alone, Jacobi (below 32 columns) or the earlier form with G in LDS and eight waves / this one, us: l = 16 34 / 17, 24
// 61 / 27, 40 96 / 54, 64 206 / 102, 80 277 / 147.  What bounds it: step 1's chain of about 1000 cycles per column (two sums
// over lanes at 130 cycles each, three LDS round trips at 80, about 25 dependent float64 operations) to 1700 at 40 columns,
// 40 to 50 % of the time; step 2 about 22 %.
// ---------------------------------------------------------------------------
__device__ __forceinline__ double readlane_f64(double x, int lane) {
    const uint64_t u = __double_as_longlong(x);
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)u, lane);
    const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
// x of another lane of the same 16-lane row (every lane has a source)
template <int CTRL>
__device__ __forceinline__ double dpp_row_f64(double x) {
    const uint64_t u = __double_as_longlong(x);
    const uint32_t lo = __builtin_amdgcn_mov_dpp((int)(uint32_t)u, CTRL, 0xf, 0xf, true);
    const uint32_t hi = __builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
__device__ __forceinline__ double wave_max_f64(double x) {
    x = fmax(x, dpp_row_f64<0xb1>(x));
    x = fmax(x, dpp_row_f64<0x4e>(x));
    x = fmax(x, dpp_row_f64<0x141>(x));
    x = fmax(x, dpp_row_f64<0x140>(x));
    return fmax(fmax(readlane_f64(x, 0), readlane_f64(x, 16)), fmax(readlane_f64(x, 32), readlane_f64(x, 48)));
}
// Sum over each group of eight lanes, in every lane of the group.
__device__ __forceinline__ double oct_sum_f64(double x) {
    x += dpp_row_f64<0xb1>(x);              // quad_perm 1,0,3,2
    x += dpp_row_f64<0x4e>(x);              // quad_perm 2,3,0,1
    x += dpp_row_f64<0x141>(x);             // row_half_mirror
    return x;
}

// Groups of lanes per wave and waves, by register columns.  Measured, us per call of the small SVD, (groups, waves): l = 16
// (2, 1) 18.3, (4, 1) 17.4; 24 26.7, 28.0; 32 35.8, 36.7; 40 55.1, 54.2, (2, 4) 54.7; 48 85.6, 74.5, (2, 2) 74.1, (2, 4)
// 72.5; 64 (2, 2) 102, (2, 4) 104; 80 (4, 2) 162, (2, 4) 147.
constexpr int tri_groups(int LW) { return LW == 16 || LW == 40 ? 4 : 2; }
constexpr int tri_waves(int LW) { return LW <= 40 ? 1 : (LW == 64 ? 2 : 4); }
// float64 words of LDS for up to LW columns: the tridiagonal solver's vectors (672), Householder vectors or S, and two
// matrices of eigenvectors; or the Jacobi solver's two copies of G and Vt
constexpr int svd_pool(int LW) {
    const int LP = (LW + 15) / 16 * 16, A = LW * (LW | 1) > LP * LP ? LW * (LW | 1) : LP * LP;
    int words = 672 + (A + 1) / 2 * 2 + 2 * LP * LP;
    for (int m = 2; m <= LW; m += 2) {
        const int need = 2 * m * (m + ((m / 2 - m) & 31)) + m * m;
        if (need > words && need <= 19968) words = need;
    }
    return words;
}
// 1/d: hardware estimate e, then q + q (e + e^2), e = 1 - d q
__device__ __forceinline__ double rcp3_f64(double d) {
    const double q = __builtin_amdgcn_rcp(d);
    const double e = fma(-d, q, 1.0);
    return fma(q, fma(e, e, e), q);
}


// The two results of a swap of 32-lane halves (D = 32) or of odd and even 16-lane rows (D = 16) of x with itself: their sum
// is x + (x of the lane D away), the same in both.
template <int D>
__device__ __forceinline__ double cross_sum_f64(double x) {
    const uint64_t u = __double_as_longlong(x);
    const uint32_t l = (uint32_t)u, h = (uint32_t)(u >> 32);
    typedef uint32_t v2u __attribute__((ext_vector_type(2)));
    v2u a, b;
    if (D == 32) {
        a = __builtin_bit_cast(v2u, __builtin_amdgcn_permlane32_swap(l, l, false, false));
        b = __builtin_bit_cast(v2u, __builtin_amdgcn_permlane32_swap(h, h, false, false));
    } else {
        a = __builtin_bit_cast(v2u, __builtin_amdgcn_permlane16_swap(l, l, false, false));
        b = __builtin_bit_cast(v2u, __builtin_amdgcn_permlane16_swap(h, h, false, false));
    }
    return __longlong_as_double((long long)((uint64_t)b.x << 32 | a.x)) + __longlong_as_double((long long)((uint64_t)b.y << 32 | a.y));
}
// Sum over each 16-lane row, in every lane of it.
__device__ __forceinline__ double row_sum_f64(double x) {
    x += dpp_row_f64<0xb1>(x);              // quad_perm 1,0,3,2
    x += dpp_row_f64<0x4e>(x);              // quad_perm 2,3,0,1
    x += dpp_row_f64<0x141>(x);             // row_half_mirror
    x += dpp_row_f64<0x140>(x);             // row_mirror
    return x;
}
template <int P>        // over the 64 / P lanes that hold the rows (every group of lanes holds the same values)
__device__ __forceinline__ double rows_sum_f64(double x) {
    x = row_sum_f64(x);
    if (P == 2) x = cross_sum_f64<16>(x);
    return x;
}
template <int P>        // over the P groups
__device__ __forceinline__ double groups_sum_f64(double x) {
    if (P == 4) x = cross_sum_f64<16>(x);
    return cross_sum_f64<32>(x);
}

// Householder tridiagonalization of the l x l matrix `gram` (leading dimension LP) by NW waves, the matrix in registers.
// Each wave's P groups of 64 / P lanes share the columns (pairs 2 P NW m + 2 g, + 1 to group g), a lane has R rows.  Step k
// forms u, beta and w = beta G u - kk u from column k and leaves G - u w^T - w u^T; that update is applied in the next
// step's sweep over the registers, which also forms the next G x: one pass over the matrix and one LDS round trip of (u, w)
// and x per step (and, with more than one wave, one barrier, at which the waves exchange their parts of G x).  The norm of
// x and what follows from it run beside that pass (G u = G x + (u0 - x0) G e).
// V: row k = u (zeros up to k and from l on); beta into tau, diagonal and off-diagonal into dia, off.
template <int LW, int P, int NW>
struct TriShape {
    static constexpr int G = 64 / P, R = (LW + G - 1) / G;              // lanes per group, rows per lane
    static constexpr int PT = P * NW, CW = (LW + 2 * PT - 1) / (2 * PT) * 2, LC = CW * PT;      // groups, columns per group, columns
    static constexpr int ROWS = R * G, VEC = ROWS > LC ? ROWS : LC;     // length of a vector in LDS
    static constexpr int WORDS = NW * 3 * VEC + (NW > 1 ? 2 * (1 + NW) : 1) * VEC;      // of LDS
};
template <int LW, int P, int NW>
__device__ __forceinline__ void tridiagonalize(const double* __restrict__ gram, int LP, int ell, int wave, int lane,
                                               double* __restrict__ V, int lda, double* __restrict__ dia,
                                               double* __restrict__ off, double* __restrict__ tau, double* __restrict__ lds) {
    using S = TriShape<LW, P, NW>;
    constexpr int G = S::G, R = S::R, CW = S::CW, PT = S::PT, VEC = S::VEC;
    const int li = lane & (G - 1), g = wave * P + lane / G;
    double2* const uw = reinterpret_cast<double2*>(lds) + wave * VEC;       // (u, w) and x, a copy per wave
    double* const xv = lds + (2 * NW + wave) * VEC;
    double* const cvs = lds + 3 * NW * VEC;                                 // column k + 1 (two generations where waves share it)
    double* const yxs = cvs + (NW > 1 ? 2 : 1) * VEC;                       // partial products of the waves
    double a[R][CW];
#pragma unroll
    for (int c = 0; c < CW; ++c) {
        const int j = min(2 * PT * (c / 2) + 2 * g + (c & 1), LP - 1);
#pragma unroll
        for (int r = 0; r < R; ++r) a[r][c] = gram[j * LP + min(li + G * r, LP - 1)];     // (symmetric: row j is column j)
    }
    double x[R], u[R], w[R], d[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        x[r] = gram[min(li + G * r, LP - 1)];
        u[r] = w[r] = d[r] = 0.0;
    }
    for (int t = lane; t < VEC; t += 64) {
        uw[t] = make_double2(0.0, 0.0);
        xv[t] = 0.0;
    }
#pragma unroll
    for (int c = 0; c < CW; ++c) {
        const int j = 2 * PT * (c / 2) + 2 * g + (c & 1);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            asm volatile("" : "+v"(a[r][c]));           // (all loads in flight before the first use)
            if (j >= ell || li + G * r >= ell) a[r][c] = 0.0;
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) x[r] = li + G * r < ell ? x[r] : 0.0;
    const double2* const uwg = uw + 2 * g;
    const double* const xvg = xv + 2 * g;
    // Step k; C0: the first register column with a column beyond k
    auto step = [&](int k, auto first) {
        constexpr int C0 = decltype(first)::value;
        // (values that several lanes hold alike are stored by all of them: no branch)
        double xm[R], s = 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i = li + G * r;
            d[r] = i == k ? x[r] : d[r];
            xm[r] = i > k ? x[r] : 0.0;
            xv[i] = xm[r];
            const double t = i > k + 1 ? xm[r] : 0.0;
            s = fma(t, t, s);
        }
        asm volatile("" ::: "memory");          // (read by other lanes)
        const double x0 = xv[k + 1];
        s = rows_sum_f64<P>(s);
        // G <- G - u w^T - w u^T of the previous step, y = G x
        double y[R][2];
#pragma unroll
        for (int r = 0; r < R; ++r) y[r][0] = y[r][1] = 0.0;
        constexpr int CH = 4, PAIRS = (CW - C0) / 2, NCH = (PAIRS + CH - 1) / CH;     // column pairs per batch of reads
        double2 q0[2][CH], q1[2][CH], xx[2][CH];
        auto fetch = [&](int ch) {
#pragma unroll
            for (int p = 0; p < CH; ++p) {
                if (ch * CH + p >= PAIRS) continue;
                const int c = C0 + 2 * (ch * CH + p);
                q0[ch & 1][p] = uwg[PT * c];
                q1[ch & 1][p] = uwg[PT * c + 1];
                xx[ch & 1][p] = *reinterpret_cast<const double2*>(xvg + PT * c);
            }
        };
        fetch(0);
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch) {
            if (ch + 1 < NCH) fetch(ch + 1);
            if (NCH > 3) asm volatile("" ::: "memory");          // (one batch ahead, not all of them)
#pragma unroll
            for (int p = 0; p < CH; ++p) {
                if (ch * CH + p >= PAIRS) continue;
                const int c = C0 + 2 * (ch * CH + p), f = ch & 1;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    a[r][c] = fma(-q0[f][p].x, w[r], fma(-q0[f][p].y, u[r], a[r][c]));
                    a[r][c + 1] = fma(-q1[f][p].x, w[r], fma(-q1[f][p].y, u[r], a[r][c + 1]));
                    y[r][0] = fma(a[r][c], xx[f][p].x, y[r][0]);
                    y[r][1] = fma(a[r][c + 1], xx[f][p].y, y[r][1]);
                }
            }
        }
        double* const cv = cvs + (NW > 1 ? (k & 1) * VEC : 0);
        double* const yx = yxs + (k & 1) * NW * VEC;
        // column k + 1 is row k + 1: its lanes publish their registers
        if (li == ((k + 1) & (G - 1))) {
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (R == 1 || r == (k + 1) / G) {
#pragma unroll
                    for (int c = C0; c < CW; c += 2)
                        *reinterpret_cast<double2*>(cv + PT * c + 2 * g) = make_double2(a[r][c], a[r][c + 1]);
                }
        }
        double ys[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            ys[r] = groups_sum_f64<P>(y[r][0] + y[r][1]);
            if (NW > 1) yx[wave * VEC + li + G * r] = ys[r];
        }
        if (NW > 1) __syncthreads();
        else asm volatile("" ::: "memory");          // (read by other lanes)
        const double n2 = fma(x0, x0, s);       // (0: the next off-diagonal is 0 or not a number, and the solver gives up)
        double rs = __builtin_amdgcn_rsq(n2);
        rs = rs * fma(-0.5 * n2, rs * rs, 1.5);
        rs = rs * fma(-0.5 * n2, rs * rs, 1.5);
        const double mu = n2 * rs;
        const double beta = rcp3_f64(fma(fabs(x0), mu, n2));
        const double dl = copysign(mu, x0), u0 = x0 + dl;
        double gu[R], c1[R], dot = 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i = li + G * r;
            c1[r] = i < S::LC ? cv[min(i, S::LC - 1)] : 0.0;
            if (NW > 1) {
                ys[r] = yx[i];
#pragma unroll
                for (int v = 1; v < NW; ++v) ys[r] += yx[v * VEC + i];
            }
            u[r] = i == k + 1 ? u0 : xm[r];
            gu[r] = fma(dl, c1[r], ys[r]);
            dot = fma(u[r], gu[r], dot);
        }
        dot = rows_sum_f64<P>(dot);
        const double kk = (0.5 * beta) * (beta * dot);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i = li + G * r;
            const double t = fma(beta, gu[r], -(kk * u[r]));
            w[r] = i > k ? t : 0.0;
            uw[i] = make_double2(u[r], w[r]);
            V[k * lda + min(i, lda - 1)] = u[r];
        }
        asm volatile("" ::: "memory");          // (read by other lanes)
        double w1;
        if constexpr (R == 1) w1 = readlane_f64(w[0], k + 1);
        else w1 = uw[k + 1].y;
        tau[k] = beta;
        off[k] = -dl;
#pragma unroll
        for (int r = 0; r < R; ++r) x[r] = fma(-u[r], w1, fma(-w[r], u0, c1[r]));
    };
    constexpr int CM = CW / 4 * 2;          // half of the column pairs; they hold columns up to CM PT - 1
    const int half = min(CM * PT, ell - 1);
    int k = 0;
    for (; k < half; ++k) step(k, std::integral_constant<int, 0>());
    for (; k + 1 < ell; ++k) step(k, std::integral_constant<int, CM>());
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = li + G * r;
        if (i < ell) dia[i] = i == ell - 1 ? x[r] : d[r];
    }
    off[ell - 1] = 0.0;
}

// Returns false, before anything is written, when the Jacobi solver has to take over.  pool: vectors (672 words), then A
// (l rows of LW columns, odd stride: the Householder vectors; later S), then Z1 and Z2 (LP x rank rounded up to 16 each).
template <int LW>
__device__ __forceinline__ bool tridiagonal_svd(const SvdJob& job, int ell, int LP, int rank, double* const pool,
                                                int* const flags, int* const twist) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lda = LW | 1, ldz = (rank + 15) & ~15;
    double* const dia = pool;               // diagonal, off-diagonal (below row i)
    double* const off = pool + 96;
    double* const tau = pool + 288;
    double* const ev = pool + 384;
    double* const A = pool + 672;
    double* const Z1 = A + ((max(ell * lda, ldz * ldz) + 1) & ~1);         // (even: pairs are 16-byte aligned)
    double* const Z2 = Z1 + LP * ldz;
    if (tid < 2) flags[tid] = 0;
    {   // zero rows (columns of the sketch that were dropped) split the matrix; narrow graded matrices see LRQ_TRI_GRADED
        double top = 0.0, low = 1e300;
        for (int i = lane; i < ell; i += 64) {
            const double d = job.gram[i * LP + i];
            top = fmax(top, d);
            low = d > 0.0 ? fmin(low, d) : 0.0;
        }
        top = wave_max_f64(top);
        low = -wave_max_f64(-low);
        if (!(low > (ell < LRQ_TRI_GRADED_BELOW ? LRQ_TRI_GRADED * top : 0.0))) return false;          // the same in every wave
    }
    // ---- 1. tridiagonalization ----
    static_assert(672 + LW * (LW | 1) + TriShape<LW, tri_groups(LW), tri_waves(LW)>::WORDS <= svd_pool(LW), "fits the pool");
    constexpr int P = tri_groups(LW), NW = tri_waves(LW);
    if (wave < NW) {
        tridiagonalize<LW, P, NW>(job.gram, LP, ell, wave, lane, A, lda, dia, off, tau, Z1);
    } else if (NW > 1) {
        for (int k = 0; k + 1 < ell; ++k) __syncthreads();
    }
    __syncthreads();
    // scale to a Gershgorin radius of 1; a split, empty or non-finite matrix goes to the other solver
    double radius, least = 1e300;
    {
        double r = 0.0;
#pragma unroll
        for (int h = 0; h < (LW > 64 ? 2 : 1); ++h) {
            const int i = lane + 64 * h;
            if (i < ell) {
                const double a0 = i > 0 ? fabs(off[i - 1]) : 0.0, b0 = fabs(off[i]);
                const double t = fabs(dia[i]) + a0 + b0;
                r = t > r || !(t == t) ? t : r;         // (a NaN stays)
                if (i + 1 < ell) least = fmin(least, b0);
                if (!(t == t)) least = -1.0;
            }
        }
        radius = wave_max_f64(r);
        least = -wave_max_f64(-least);
    }
    if (!(radius > 1e-280 && radius < 1e280) || !(least > 1e-14 * radius)) return false;      // the same in every thread
    const double inv = rcp_f64(radius);
    double2* const de = reinterpret_cast<double2*>(pool + 480);         // (d_i, e_{i-1}^2), padded with rows that change no sign
    const double d0 = tid < ell ? dia[min(tid, 95)] * inv : 2.0;
    const double o0 = tid < ell ? off[min(tid, 95)] * inv : 0.0, om = (tid > 0 && tid < ell) ? off[min(tid, 95) - 1] * inv : 0.0;
    __syncthreads();
    if (tid < 96) {
        de[tid] = make_double2(d0, om * om);
        dia[tid] = d0;
        off[tid] = o0;
    }
    __syncthreads();
    // ---- 2. the largest eigenvalues, ev[t] the t-th largest; four waves, GL lanes each, two points per lane ----
    if (wave < 4) {
        const int GL = rank <= 8 ? 32 : (rank <= 16 ? 16 : (rank <= 32 ? 8 : (rank <= 40 ? 6 : (rank <= 64 ? 4 : 3))));
        const int rounds = rank <= 8 ? 9 : (rank <= 16 ? 10 : (rank <= 32 ? 12 : (rank <= 40 ? 14 : (rank <= 64 ? 16 : 18))));     // (2 GL + 1)^rounds > 2^49
        const int per = 64 / GL, grp = lane / GL, g = lane - grp * GL;
        const int t = wave * per + grp;
        const int e = ell - 1 - t;              // eigenvalues below it
        const double step = rcp_f64(2.0 * GL + 1.0);
        const uint64_t mask = ((1ull << GL) - 1) << (grp * GL), live = __ballot(grp < per && t < rank);
        constexpr bool IN_REGS = LW <= 40;      // the rows of T stay in registers, or come from LDS in every round
        double2 rows[IN_REGS ? LW : 1];
        if constexpr (IN_REGS) {
#pragma unroll
            for (int i = 0; i < LW; ++i) rows[i] = de[1 + i];
        }
        double lo = -1e-6, hi = 1.0;
        if (wave * per < rank)
        for (int r = 0; r < rounds + 2; ++r) {
            // two more where an eigenvalue is far below the largest (V = B^T U' / sigma needs it relative to itself) or close to
            // the next one (whose vectors are then only as orthogonal as the two are apart)
            if (r >= rounds) {
                const double next = __shfl(hi, min(lane + GL, 63), 64);
                const bool close = grp + 1 < per && t + 1 < rank && hi - lo > 1e-6 * (lo - next);
                if (!(__ballot(close || hi - lo > 1e-11 * hi) & live)) break;
            }
            const double h = (hi - lo) * step;
            const double xa = fma(h, g + 1.0, lo), xb = fma(h, (double)(g + 1 + GL), lo);
            // leading minors p_i of T - x I, scaled: the number of sign changes is the number of eigenvalues below x
            double a0 = 1.0, a1 = de[0].x - xa, b0 = 1.0, b1 = de[0].x - xb;
            uint32_t sa = (uint32_t)__double2hiint(a1) >> 31, sb = (uint32_t)__double2hiint(b1) >> 31;     // signs, the last one in bit 0
            int ca = sa, cb = sb;
            auto row = [&](double2 q) {
                const double a2 = fma(q.x - xa, a1, -(q.y * a0));
                const double b2 = fma(q.x - xb, b1, -(q.y * b0));
                sa = __builtin_amdgcn_alignbit(sa, (uint32_t)__double2hiint(a2), 31);
                sb = __builtin_amdgcn_alignbit(sb, (uint32_t)__double2hiint(b2), 31);
                a0 = a1; a1 = a2;
                b0 = b1; b1 = b2;
            };
            auto eight = [&] {          // after eight rows: their sign changes, and a common scale for the minors
                ca += __builtin_popcount((sa ^ (sa >> 1)) & 0xffu);
                cb += __builtin_popcount((sb ^ (sb >> 1)) & 0xffu);
                const int ea = __builtin_amdgcn_frexp_exp(fmax(fabs(a0), fabs(a1)));
                const int eb = __builtin_amdgcn_frexp_exp(fmax(fabs(b0), fabs(b1)));
                a0 = __builtin_amdgcn_ldexp(a0, -ea); a1 = __builtin_amdgcn_ldexp(a1, -ea);
                b0 = __builtin_amdgcn_ldexp(b0, -eb); b1 = __builtin_amdgcn_ldexp(b1, -eb);
            };
            if constexpr (IN_REGS) {
#pragma unroll
                for (int i = 0; i < LW; ++i) {
                    row(rows[i]);
                    if (i % 8 == 7) eight();
                }
            } else {
                for (int i = 1; i < ell; i += 16) {
                    double2 q[8], p[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) q[u] = de[i + u];
#pragma unroll
                    for (int u = 0; u < 8; ++u) p[u] = de[i + 8 + u];      // (inside the padding at the end)
#pragma unroll
                    for (int u = 0; u < 8; ++u) row(q[u]);
                    eight();
#pragma unroll
                    for (int u = 0; u < 8; ++u) row(p[u]);
                    eight();
                }
            }
            // points at or below the eigenvalue (the counts rise with the point)
            const int j = __builtin_popcountll(~__ballot(ca > e) & mask) + __builtin_popcountll(~__ballot(cb > e) & mask);
            const double nlo = fma(h, (double)j, lo);
            hi = j == 2 * GL ? hi : fma(h, j + 1.0, lo);
            lo = nlo;
        }
        if (g == 0 && grp < per && t < rank) ev[t] = 0.5 * (lo + hi);
    }
    __syncthreads();
    // ---- 3. eigenvectors of the tridiagonal matrix; column t belongs to ev[t]: the LDU sweep from the top in one wave, the
    // one from the bottom in another ----
    const int t3 = (wave >> 1) * 64 + lane;
    const bool top_sweep = (wave & 1) == 0, on3 = wave < 4 && t3 < rank;
    if (on3) {
        const double lam = ev[t3], tiny = 1e-30;
        double* const L = Z1 + t3;
        double* const Uz = Z2 + t3;
        // (the operands of step i + 1 are read before step i writes: LDS reads stay off the recurrences)
        if (top_sweep) {
            double dp = dia[0] - lam, o = off[0], dn = dia[1];
            for (int i = 0; i + 1 < ell; ++i) {
                const double o2 = off[i + 1], dn2 = dia[min(i + 2, ell - 1)];
                if (fabs(dp) < tiny) dp = copysign(tiny, dp);
                const double l = o * rcp3_f64(dp);
                L[i * ldz] = l;
                dp = fma(-l, o, dn - lam);
                o = o2;
                dn = dn2;
            }
        } else {
            double dm = dia[ell - 1] - lam, o = off[ell - 2], dn = dia[ell - 2];
            for (int i = ell - 2; i >= 0; --i) {
                const int ip = max(i - 1, 0);
                const double o2 = off[ip], dn2 = dia[ip];
                if (fabs(dm) < tiny) dm = copysign(tiny, dm);
                const double u = o * rcp3_f64(dm);
                Uz[i * ldz] = u;
                dm = fma(-u, o, dn - lam);
                o = o2;
                dn = dn2;
            }
        }
    }
    __syncthreads();
    // where the two meet: the smallest |gamma_i| = |(d_i - lambda) - l_{i-1} e_{i-1} - u_i e_i|; eight lanes per vector
    for (int b = 8 * wave; b < rank; b += SVD_THREADS / 8) {
        const int t = min(b + (lane >> 3), rank - 1), sl = lane & 7;
        const double lam = ev[t];
        double best = 1e300;
        int r = 0;
#pragma unroll
        for (int u = 0; u < MAXL / 8; ++u) {
            if (8 * u < ell) {
                const int i = min(sl + 8 * u, ell - 1);
                const double lo = i > 0 ? Z1[max(i - 1, 0) * ldz + t] * off[max(i - 1, 0)] : 0.0;
                const double up = i + 1 < ell ? Z2[min(i, ell - 2) * ldz + t] * off[i] : 0.0;
                const double gam = fabs((dia[i] - lam) - lo - up);
                if (gam < best) { best = gam; r = i; }
            }
        }
#pragma unroll
        for (int o = 1; o < 8; o <<= 1) {
            const double ob = __shfl_xor(best, o, 64);
            const int orr = __shfl_xor(r, o, 64);
            if (ob < best || (ob == best && orr < r)) { best = ob; r = orr; }
        }
        if (sl == 0) twist[t] = r;
    }
    __syncthreads();
    if (on3) {
        double* const L = Z1 + t3;
        double* const Uz = Z2 + t3;
        const int r = twist[t3];
        double z = 1.0;
        if (top_sweep) {
            for (int i0 = ell - 2; i0 >= 0; i0 -= 4) {
                double m[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) m[u] = L[max(i0 - u, 0) * ldz];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int i = i0 - u;
                    if (i < r && i >= 0) {
                        z = -(m[u] * z);
                        L[i * ldz] = z;
                    }
                }
            }
            L[r * ldz] = 1.0;
        } else {
            for (int i0 = 0; i0 + 1 < ell; i0 += 4) {
                double m[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) m[u] = Uz[min(i0 + u, ell - 2) * ldz];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int i = i0 + u;
                    if (i >= r && i + 1 < ell) {
                        z = -(m[u] * z);
                        L[(i + 1) * ldz] = z;
                    }
                }
            }
        }
    }
    __syncthreads();
    // ---- 4. normalization and back transformation, eight lanes per vector; unused rows and columns become zeros ----
    constexpr int NU = LW / 8;
    for (int b = 8 * wave; b < ldz; b += SVD_THREADS / 8) {
        const int t = b + (lane >> 3), sl = lane & 7;
        double* const col = Z1 + t;
        double z[NU], n2 = 0.0;
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            z[u] = (sl + 8 * u < ell && t < rank) ? col[(sl + 8 * u) * ldz] : 0.0;
            n2 = fma(z[u], z[u], n2);
        }
        n2 = oct_sum_f64(n2);
        double sc = __builtin_amdgcn_rsq(n2);
        sc = sc * fma(-0.5 * n2, sc * sc, 1.5);
        sc = sc * fma(-0.5 * n2, sc * sc, 1.5);
        sc = t < rank ? sc : 0.0;
#pragma unroll
        for (int u = 0; u < NU; ++u) z[u] *= sc;
        double v[NU], tk = tau[ell - 2];
#pragma unroll
        for (int u = 0; u < NU; ++u) v[u] = A[(ell - 2) * lda + sl + 8 * u];
        for (int k = ell - 2; k >= 0; --k) {
            const int kn = max(k - 1, 0);
            double vn[NU];
            const double tn = tau[kn];
#pragma unroll
            for (int u = 0; u < NU; ++u) vn[u] = A[kn * lda + sl + 8 * u];
            double d0 = 0.0, d1 = 0.0;
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                if (u & 1) d1 = fma(v[u], z[u], d1);
                else       d0 = fma(v[u], z[u], d0);
            }
            const double d = tk * oct_sum_f64(d0 + d1);
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                z[u] = fma(-d, v[u], z[u]);
                v[u] = vn[u];
            }
            tk = tn;
        }
        if (t < ldz) {
#pragma unroll
            for (int u = 0; u < NU; ++u)
                if (sl + 8 * u < LP) col[(sl + 8 * u) * ldz] = z[u];
            if (LW + sl < LP) col[(LW + sl) * ldz] = 0.0;
        }
    }
    __syncthreads();
    // ---- 5. S = U^T U (kept as 3/2 I - S/2 in A's place), its distance from I, one correction step ----
    typedef double v4d __attribute__((ext_vector_type(4)));
    const int nt = ldz >> 4, li = lane & 15, kq = lane >> 4;
    double* const S = A;                    // ldz x ldz
    for (int tl = wave; tl < nt * nt; tl += SVD_THREADS / 64) {
        const int ta = tl / nt, tb = tl - ta * nt;
        v4d acc = (v4d){0.0, 0.0, 0.0, 0.0};
        for (int k = 0; k < LP; k += 4)
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(Z1[(k + kq) * ldz + 16 * ta + li], Z1[(k + kq) * ldz + 16 * tb + li],
                                                       acc, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int i = 16 * ta + 4 * v + kq, j = 16 * tb + li;
            const double want = (i == j && i < rank) ? 1.0 : 0.0, d = fabs(acc[v] - want);
            if (!(d <= 1e-4)) flags[0] = 1;
            if (d > 1e-11) flags[1] = 1;
            S[i * ldz + j] = (i == j ? 1.5 : 0.0) - 0.5 * acc[v];
        }
    }
    __syncthreads();
    const bool fail = flags[0] != 0, correct = flags[1] != 0;
    __syncthreads();        // (the flags may be reused by the caller)
    if (fail) return false;
    double* U = Z1;
    if (correct) {
        const int rt = LP >> 4;
        for (int tl = wave; tl < rt * nt; tl += SVD_THREADS / 64) {
            const int ta = tl / nt, tb = tl - ta * nt;
            v4d acc = (v4d){0.0, 0.0, 0.0, 0.0};
            for (int k = 0; k < ldz; k += 4)
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(Z1[(16 * ta + li) * ldz + k + kq], S[(k + kq) * ldz + 16 * tb + li],
                                                           acc, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 4; ++v) Z2[(16 * ta + 4 * v + kq) * ldz + 16 * tb + li] = acc[v];
        }
        U = Z2;
        __syncthreads();
    }
    const double top = sqrt(fmax(ev[0] * radius, 0.0));
    if (tid < rank) job.Sigma[tid] = (float)sqrt(fmax(ev[tid] * radius, 0.0));
    for (int idx = tid; idx < LP * rank; idx += SVD_THREADS) {
        const int a = idx / rank, t = idx % rank;
        double u = 0.0, mv = 0.0;
        if (a < ell) {
            u = U[a * ldz + t];
            const double sg = sqrt(fmax(ev[t] * radius, 0.0));
            mv = (sg > 1e-14 * top && sg > 0.0) ? u / sg : 0.0;
        }
        job.Ur[idx] = u;
        job.Mv[idx] = mv;
    }
    return true;
}

template <int NB, int LW>
__global__ __launch_bounds__(SVD_THREADS) void small_svd_kernel(SvdJob j0, SvdJob j1, int ell, int LP, int rank) {
    const SvdJob job = blockIdx.x == 0 ? j0 : j1;
    const double* __restrict__ const gram = job.gram;
    float* __restrict__ const Sigma = job.Sigma;
    double* __restrict__ const Ur = job.Ur;
    double* __restrict__ const Mv = job.Mv;
    __shared__ __align__(16) double pool[svd_pool(LW)];
    raise_wave_priority();
    __shared__ __align__(16) double2 rot[2][MAXL / 2];      // (c, s) per slot, two generations
    __shared__ int order[MAXL];
    __shared__ int finished;
    __shared__ int flags[2];
    const int tid = threadIdx.x;
    if (ell >= LRQ_TRI_MIN) {
        if (tridiagonal_svd<LW>(job, ell, LP, rank, pool, flags, order)) return;
        __syncthreads();
    }
    const int m = (ell + 1) & ~1;   // even number of players; a zero dummy row/column when ell is odd
    const int half = m / 2;
    int ldg = m + ((half - m) & 31);                      // >= m, = half (mod 32)
    if (2 * m * ldg + m * m > svd_pool(LW)) ldg = m + 1;       // largest sketches: accept bank conflicts
    const int ldv = m;
    double* const G0 = pool;
    double* const G1 = pool + m * ldg;
    double* const Vt = pool + 2 * m * ldg;
    // slot index of a player when the arrangement is the identity (start of a sweep)
    auto home = [&](int e) { return e < half ? e : half + (m - 1 - e); };
    // slot index after one step of the tournament
    auto moved = [&](int x) {
        if (m == 2) return x;
        if (x < half) return x == 0 ? half + 1 : x - 1;
        const int y = x - half;
        return y == 0 ? half : (y == half - 1 ? half - 1 : x + 1);
    };
    for (int idx = tid; idx < m * ldg; idx += SVD_THREADS) G0[idx] = 0.0;
    for (int idx = tid; idx < m * m; idx += SVD_THREADS) Vt[idx] = (idx / m == idx % m) ? 1.0 : 0.0;
    if (tid == 0) finished = 0;
    __syncthreads();
    for (int base = 0; base < ell * ell; base += 4 * SVD_THREADS) {     // stored by slot; four loads in flight
        double v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int idx = min(base + u * SVD_THREADS + tid, ell * ell - 1);
            v[u] = gram[(idx / ell) * LP + idx % ell];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int idx = base + u * SVD_THREADS + tid;
            if (idx < ell * ell) G0[home(idx / ell) * ldg + home(idx % ell)] = v[u];
        }
    }
    __syncthreads();

    // rotation wave: addresses of the ten entries behind the lane's next pair (loop invariant)
    double gsc = 0.0;
    bool seen_large = false;
    int iaa = 0, iab = 0, ibb = 0, jaa = 0, jab = 0, jbb = 0, x11i = 0, x12i = 0, x21i = 0, x22i = 0, sa = 0, sb = 0;
    bool xfirst = true, yfirst = true;
    SvdTask task[NB];
    if (tid < half) {
        double gmax = 0.0;
        for (int a = 0; a < m; ++a) gmax = fmax(gmax, fabs(G0[a * ldg + a]));
        gsc = gmax > 0.0 ? 1.0 / gmax : 0.0;
        const int p = tid, q = half + tid;
        double c, s;
        seen_large = jacobi_rotation(G0[p * ldg + p], G0[q * ldg + q], G0[p * ldg + q], gsc, c, s);
        rot[0][tid] = make_double2(c, s);
        int cx = p, cy = q;                                // where the next pair sits now
        for (int x = 0; x < m; ++x) {
            const int y = moved(x);
            if (y == p) cx = x;
            if (y == q) cy = x;
        }
        xfirst = cx < half;
        yfirst = cy < half;
        sa = xfirst ? cx : cx - half;
        sb = yfirst ? cy : cy - half;
        const int pa = sa, qa = half + sa, pb = sb, qb = half + sb;
        iaa = pa * ldg + pa; iab = pa * ldg + qa; ibb = qa * ldg + qa;
        jaa = pb * ldg + pb; jab = pb * ldg + qb; jbb = qb * ldg + qb;
        x11i = pa * ldg + pb; x12i = pa * ldg + qb; x21i = qa * ldg + pb; x22i = qa * ldg + qb;
    }
#pragma unroll
    for (int t = 0; t < NB; ++t) {
        SvdTask& k = task[t];
        const int blk = tid - 64 + t * SVD_UPDATE_THREADS;
        k.active = tid >= 64 && blk < half * half;
        const int P = k.active ? blk / half : 0, Q = k.active ? blk - P * half : 0;
        k.P = P; k.Q = Q;
        k.o11 = P * ldg + Q; k.o12 = k.o11 + half; k.o21 = (half + P) * ldg + Q; k.o22 = k.o21 + half;
        const int n1 = moved(P) * ldg, n2 = moved(half + P) * ldg, k1 = moved(Q), k2 = moved(half + Q);
        k.w11 = n1 + k1; k.w12 = n1 + k2; k.w21 = n2 + k1; k.w22 = n2 + k2;
        // eigenvector columns of slot P at step 0: players P and (m - 1 - P) (slot 0: m - 1, fixed)
        k.v1 = P * ldv + 2 * Q;
        k.v2 = (m - 1 - P) * ldv + 2 * Q;
        k.dv2 = (P == 0) ? 0 : ldv;
        k.v1_wrap = (m - 1) * ldv + 2 * Q;     // first offset past player m - 2
        k.v2_wrap = (P == 0) ? 0x7fffffff : k.v1_wrap;   // player m - 1 never moves
    }
    __syncthreads();
    // one tournament step: reads G/rr, writes Gn/rn
    auto do_step = [&](const double* __restrict__ G, double* __restrict__ Gn, const double2* __restrict__ rr,
                       double2* __restrict__ rn, bool last_of_sweep) {
        if (tid < 64) {
            if (tid < half) {
                const double2 ra = rr[sa], rb = rr[sb];
                const double ca = ra.x, sna = ra.y, cb = rb.x, snb = rb.y;
                const double a11 = G[iaa], a12 = G[iab], a22 = G[ibb];
                const double b11 = G[jaa], b12 = G[jab], b22 = G[jbb];
                const double x11 = G[x11i], x12 = G[x12i], x21 = G[x21i], x22 = G[x22i];
                // diagonal entry of J^T D J for a symmetric 2x2 block D:
                //   first : c^2 d11 - 2 c s d12 + s^2 d22     second: s^2 d11 + 2 c s d12 + c^2 d22
                const double wa = 2.0 * ca * sna * a12, wb = 2.0 * cb * snb * b12;
                const double ca2 = ca * ca, sa2 = sna * sna, cb2 = cb * cb, sb2 = snb * snb;
                const double gxx = xfirst ? fma(ca2, a11, fma(sa2, a22, -wa)) : fma(sa2, a11, fma(ca2, a22, wa));
                const double gyy = yfirst ? fma(cb2, b11, fma(sb2, b22, -wb)) : fma(sb2, b11, fma(cb2, b22, wb));
                // entry (x, y) of J_a^T X J_b: column of J_a for x, column of J_b for y
                const double al0 = xfirst ? ca : sna, al1 = xfirst ? -sna : ca;
                const double be0 = yfirst ? cb : snb, be1 = yfirst ? -snb : cb;
                const double gxy = fma(al0, fma(x11, be0, x12 * be1), al1 * fma(x21, be0, x22 * be1));
                double c, s;
                const bool large = jacobi_rotation(gxx, gyy, gxy, gsc, c, s);
                rn[tid] = make_double2(c, s);
                // the flags of a sweep cover the rotations applied in it; the one just
                // formed at the last step opens the next sweep
                if (last_of_sweep) {
                    const bool any = __any(seen_large);
                    if (tid == 0) finished = any ? 0 : 1;
                    seen_large = large;
                } else {
                    seen_large = seen_large || large;
                }
            }
        } else {
#pragma unroll
            for (int t = 0; t < NB; ++t) {
                SvdTask& k = task[t];
                if (k.active) {
                    const double2 r1 = rr[k.P], r2 = rr[k.Q];
                    const double c1 = r1.x, s1 = r1.y, c2 = r2.x, s2 = r2.y;
                    const double a11 = G[k.o11], a12 = G[k.o12], a21 = G[k.o21], a22 = G[k.o22];
                    double2* e1p = reinterpret_cast<double2*>(Vt + k.v1);
                    double2* e2p = reinterpret_cast<double2*>(Vt + k.v2);
                    const double2 e1 = *e1p, e2 = *e2p;
                    // rows: J^T G, then columns: (.) J
                    const double t11 = fma(c1, a11, -(s1 * a21)), t12 = fma(c1, a12, -(s1 * a22));
                    const double t21 = fma(s1, a11, c1 * a21), t22 = fma(s1, a12, c1 * a22);
                    Gn[k.w11] = fma(c2, t11, -(s2 * t12));
                    Gn[k.w12] = fma(s2, t11, c2 * t12);
                    Gn[k.w21] = fma(c2, t21, -(s2 * t22));
                    Gn[k.w22] = fma(s2, t21, c2 * t22);
                    *e1p = make_double2(fma(c1, e1.x, -(s1 * e2.x)), fma(c1, e1.y, -(s1 * e2.y)));
                    *e2p = make_double2(fma(s1, e1.x, c1 * e2.x), fma(s1, e1.y, c1 * e2.y));
                    // next step: both columns of the slot are one player further
                    k.v1 += ldv;
                    if (k.v1 >= k.v1_wrap) k.v1 -= (m - 1) * ldv;
                    k.v2 += k.dv2;
                    if (k.v2 >= k.v2_wrap) k.v2 -= (m - 1) * ldv;
                }
            }
        }
        __syncthreads();
    };
    int cur = 0, step = 0, sweeps = 0;
    for (;;) {
        const bool last = (step + 1 == m - 1);
        if (cur == 0) do_step(G0, G1, rot[0], rot[1], last);
        else          do_step(G1, G0, rot[1], rot[0], last);
        cur ^= 1;
        if (last) {
            step = 0;
            if (++sweeps == 16 || finished) break;
        } else {
            ++step;
        }
    }
    const double* G = cur ? G1 : G0;
    // rank eigenvalues: order[pos] = index of the pos-th largest (ties by index)
    if (tid < ell) {
        const double mine = G[home(tid) * ldg + home(tid)];
        int pos = 0;
#pragma unroll 8
        for (int o = 0; o < ell; ++o) {
            const double other = G[home(o) * ldg + home(o)];
            if (other > mine || (other == mine && o < tid)) ++pos;
        }
        order[pos] = tid;
    }
    __syncthreads();
    if (tid < rank) Sigma[tid] = (float)sqrt(fmax(G[home(order[tid]) * ldg + home(order[tid])], 0.0));
    const double top = sqrt(fmax(G[home(order[0]) * ldg + home(order[0])], 0.0));
    for (int idx = tid; idx < LP * rank; idx += SVD_THREADS) {
        const int a = idx / rank, t = idx % rank;
        double u = 0.0, mv = 0.0;
        if (a < ell) {
            const int e = order[t];
            u = Vt[e * ldv + a];
            const double sg = sqrt(fmax(G[home(e) * ldg + home(e)], 0.0));
            mv = (sg > 1e-14 * top && sg > 0.0) ? u / sg : 0.0;
        }
        Ur[idx] = u;
        Mv[idx] = mv;
    }
}

// U = Q's leading columns, Sigma = 1, Vt = (sum of the T pass's partials)^T for the jobs (see BasisJob; 16 padded
// columns).  Workgroups [0, nbV) of a job: 16 columns of R each, four waves with a run of the splits each, eight 16-byte
// loads in flight, the runs added in order (as reduce_gram_kernel does it) and stored transposed through LDS.  The rest
// copy Q, four entries of U per thread.  Bound by load latency: one launch in place of the Gram matrix, its sum, the
// small SVD and the product with its vectors.  Calls, with the SVD / without: 256^3, 8 columns 81 / 57 us; 2000^3, 10
// columns 204 / 177; 100352 x 64 x 576, 8 columns 242 / 218.
struct BasisGrid { int nbV, nb; };
__global__ __launch_bounds__(256) void take_basis_kernel(BasisJob a, BasisJob b, BasisGrid ga, BasisGrid gb, int rank) {
    __shared__ float4 runs[4][64];
    __shared__ float tile[16][17];
    const bool first = (int)blockIdx.x < ga.nb;
    const BasisJob job = first ? a : b;
    const int nbV = first ? ga.nbV : gb.nbV, blk = first ? blockIdx.x : blockIdx.x - ga.nb;
    const int tid = threadIdx.x;
    if (blk < nbV) {
        const int k0 = blk * 16, sg = tid >> 6, e = tid & 63;       // group e: row k0 + e / 4, columns 4 (e % 4) ..
        const int sb = sg * job.splits / 4, se = (sg + 1) * job.splits / 4;
        const size_t plane = (size_t)job.cols * 16;
        const float* src = job.partial + (size_t)min(k0 + e / 4, job.cols - 1) * 16 + (e % 4) * 4;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int s0 = sb; s0 < se; s0 += 8) {
            float4 p[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) p[u] = *reinterpret_cast<const float4*>(src + (size_t)min(s0 + u, se - 1) * plane);
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (s0 + u < se) { v.x += p[u].x; v.y += p[u].y; v.z += p[u].z; v.w += p[u].w; }
        }
        runs[sg][e] = v;
        __syncthreads();
        if (sg == 0) {
#pragma unroll
            for (int g = 1; g < 4; ++g) {
                const float4 t = runs[g][e];
                v.x += t.x; v.y += t.y; v.z += t.z; v.w += t.w;
            }
            float* t = &tile[e / 4][(e % 4) * 4];
            t[0] = v.x; t[1] = v.y; t[2] = v.z; t[3] = v.w;
        }
        __syncthreads();
        const int t = tid >> 4, k = tid & 15;
        if (t < rank && k0 + k < job.cols) job.Vt[(size_t)t * job.cols + k0 + k] = tile[k][t];
        if (blk == 0 && tid < rank) job.Sigma[tid] = 1.0f;
        return;
    }
    const size_t total = (size_t)job.rows * rank;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const size_t idx = (size_t)(blk - nbV) * 1024 + u * 256 + tid;
        if (idx < total) job.U[idx] = job.Q[(idx / rank) * 16 + idx % rank];
    }
}

// take_basis and panel_prep in one launch, where both operands' factors are 16 columns wide and K is short: workgroups [0, slices) take
// `per` k blocks of 64 each: the partials' sums (V) and B's Q (W) as matrix-core operands and their product's slice of X, straight
// from the 64 x 16 tiles in LDS; the rest take 64 columns of B each, for Zt.  1024 threads: four runs of the splits per group of
// values, added in order, as in take_basis_kernel.  Calls, two launches / this: 256^3 40.7 / 38.8
// us, 200^3 74.6 / 71.9, 2000^3 (two blocks a workgroup) 135.8 / 135.9, 100352 x 64 x 576 208 / 203.
#define BASIS_PER 2         // k blocks of a workgroup, at most: they follow each other
int basis_slices(int K) {
    const int nkb = pk_kblocks(K), per = ceil_div(nkb, LRQ_VTW_MAX_SLICES);
    return per <= BASIS_PER ? ceil_div(nkb, per) : 0;
}
__global__ __launch_bounds__(1024) void basis_panels_kernel(BasisPanels a) {
    __shared__ float4 runs[4][256];
    __shared__ float vt[64][17], wt[64][17];
    const bool isA = (int)blockIdx.x < a.slices;
    const int tid = threadIdx.x, r = a.r, sg = tid >> 8, e = tid & 255;
    const int first = isA ? blockIdx.x * a.per : blockIdx.x - a.slices, last = isA ? min(first + a.per, a.nkb) : first + 1;
    const bool second = isA && a.again && *a.again != 0;
    const float* const partial = isA ? (second ? a.partialA2 : a.partialA) : a.partialB;
    const int cols = isA ? a.K : a.N, splits = isA ? (second ? a.splitsA2 : a.splitsA) : a.splitsB;
    const int sb = sg * splits / 4, se = (sg + 1) * splits / 4;
    const size_t plane = (size_t)cols * 16;
    double x = 0.0;             // X[t][u] of thread 16 t + u
    for (int blk = first; blk < last; ++blk) {
        const int k0 = blk * 64;
        const float* src = partial + (size_t)min(k0 + e / 4, cols - 1) * 16 + (e % 4) * 4;
        const float w = isA ? a.QB[(size_t)min(k0 + tid / 16, a.K - 1) * 16 + tid % 16] : 0.f;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int s0 = sb; s0 < se; s0 += 8) {
            float4 p[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) p[u] = *reinterpret_cast<const float4*>(src + (size_t)min(s0 + u, se - 1) * plane);
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (s0 + u < se) { v.x += p[u].x; v.y += p[u].y; v.z += p[u].z; v.w += p[u].w; }
        }
        runs[sg][e] = v;
        wt[tid / 16][tid % 16] = k0 + tid / 16 < a.K && tid % 16 < r ? w : 0.f;
        __syncthreads();
        if (sg == 0) {
#pragma unroll
            for (int g = 1; g < 4; ++g) {
                const float4 t = runs[g][e];
                v.x += t.x; v.y += t.y; v.z += t.z; v.w += t.w;
            }
            const bool in = k0 + e / 4 < cols;
            const int c = (e % 4) * 4;
            vt[e / 4][c + 0] = in && c + 0 < r ? v.x : 0.f;
            vt[e / 4][c + 1] = in && c + 1 < r ? v.y : 0.f;
            vt[e / 4][c + 2] = in && c + 2 < r ? v.z : 0.f;
            vt[e / 4][c + 3] = in && c + 3 < r ? v.w : 0.f;
        }
        __syncthreads();
        if (isA) {
            if (tid < 256) {
#pragma unroll
                for (int k = 0; k < 64; ++k) x = fma((double)vt[k][tid >> 4], (double)wt[k][tid & 15], x);
            } else if (tid < 512) {         // a lane's eight k of an operand: V, then W
                const int lane = tid & 63, h = (tid >> 6) & 1;
                const bool isV = tid < 384;
                float q[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int k = 16 * (lane >> 4) + 8 * h + i;
                    q[i] = isV ? vt[k][lane & 15] : wt[k][lane & 15];
                }
                const Planes3 pl = split_planes<3>(q);
                uint16_t* const dst = (isV ? a.Vf : a.Wf) + (size_t)(blk * 6 + h) * FACTOR_PIECE + lane * 8;
                *reinterpret_cast<v8bf16*>(dst) = pl.p1;
                *reinterpret_cast<v8bf16*>(dst + 2 * FACTOR_PIECE) = pl.p2;
                *reinterpret_cast<v8bf16*>(dst + 4 * FACTOR_PIECE) = pl.p3;
            }
            __syncthreads();
        } else if (tid / 64 < r && k0 + tid % 64 < a.N) {
            a.Zt[(size_t)(tid / 64) * a.N + k0 + tid % 64] = vt[tid % 64][tid / 64];
        }
    }
    if (isA && tid < 256 && (tid >> 4) < r && (tid & 15) < r)
        a.Xp[((size_t)blockIdx.x * r + (tid >> 4)) * r + (tid & 15)] = (float)x;
    if (blockIdx.x == 0 && tid < r) a.Sig[tid] = a.Gam[tid] = 1.0f;
}

#define NT_SWITCH(NTV, CALL)            \
    switch (NTV) {                      \
        case 1: { constexpr int NT_ = 1; CALL; } break; \
        case 2: { constexpr int NT_ = 2; CALL; } break; \
        case 3: { constexpr int NT_ = 3; CALL; } break; \
        case 4: { constexpr int NT_ = 4; CALL; } break; \
        case 5: { constexpr int NT_ = 5; CALL; } break; \
        default: return LRQMM_ERR_UNSUPPORTED;          \
    }

int launch_reduce_gram(const GramJob* job, int njob, int LP, hipStream_t st) {
    GramJob j[2] = {job[0], njob > 1 ? job[1] : job[0]};
    bool small = true;      // one tile height per launch: 16 rows where both fit it
    for (int i = 0; i < njob; ++i) small = small && gram_rows_per_block(j[i].n, LP) == 16;
    for (int i = 0; i < njob; ++i) {
        j[i].rows_per_block = gram_rows_per_block(j[i].n, LP);
        j[i].blocks = gram_blocks(j[i].n, LP);
    }
    const int nb0 = j[0].blocks, nb1 = njob > 1 ? j[1].blocks : 0;
    if (small) {
        NT_SWITCH(LP / 16, hipLaunchKernelGGL((reduce_gram_kernel<NT_, 16>), dim3(nb0 + nb1), dim3(256), 0, st, j[0], j[1], nb0));
    } else {
        NT_SWITCH(LP / 16, hipLaunchKernelGGL((reduce_gram_kernel<NT_, 64>), dim3(nb0 + nb1), dim3(256), 0, st, j[0], j[1], nb0));
    }
    LRQ_CHECK_LAUNCH();
    return LRQMM_OK;
}

int launch_gram_sum(const GramJob* job, int njob, int LP, hipStream_t st) {
    GramJob j[2] = {job[0], njob > 1 ? job[1] : job[0]};
    int most = 0;
    for (int i = 0; i < njob; ++i) {
        if (j[i].blocks == 0) j[i].blocks = gram_blocks(j[i].n, LP);
        most = max(most, j[i].blocks);
    }
    dim3 grid(ceil_div(LP * LP, 8), njob);
#define LRQ_GSUM(B) hipLaunchKernelGGL(gram_sum_parts_kernel<B>, grid, dim3(64), 0, st, j[0], j[1], LP * LP)
    if (most <= 64)       LRQ_GSUM(8);
    else if (most <= 128) LRQ_GSUM(16);
    else if (most <= 256) LRQ_GSUM(32);
    else                  LRQ_GSUM(64);
#undef LRQ_GSUM
    LRQ_CHECK_LAUNCH();
    return LRQMM_OK;
}

int launch_project_sum(const double* gpart, const float* mpart, int blocks, int cols, double* gsum, double* msum, hipStream_t st) {
    const dim3 grid(1 + ceil_div(cols * 16, 512), PROJECT_GROUPS);
    hipLaunchKernelGGL(project_sum_kernel, grid, dim3(256), 0, st, gpart, mpart, blocks, cols * 16, gsum, msum);
    LRQ_CHECK_LAUNCH();
    return LRQMM_OK;
}

int launch_apply(const ApplyJob* job, int njob, int LP, hipStream_t st) {
    ApplyJobs a = {};
    int total = 0;
    for (int i = 0; i < njob; ++i) {
        a.j[i] = job[i];
        a.nb[i] = ceil_div(job[i].n, 16);
        total += a.nb[i];
    }
    if (total == 0) return LRQMM_OK;
    NT_SWITCH(LP / 16, hipLaunchKernelGGL((apply_kernel<NT_>), dim3(total), dim3(64), 0, st, a));
    LRQ_CHECK_LAUNCH();
    return LRQMM_OK;
}

// Few partials (16 columns, up to 256 rows) are added where they are used, one launch less.  Gram sum as a launch of its own /
// here: 200^3 l = 10 92.4 / 88.1 us per call, l = 24 139.6 / 140.6; with up to 64 partials 400^3 l = 10 105.3 / 108.3, 1000^3
// 113.5 / 119.1.
bool orth_apply_sums(int blocks, int LP) { return blocks <= 8 * ORTH_PER && LP == 16; }

int launch_orth_apply(const GramJob* job, int njob, int ell, int LP, bool sum, hipStream_t st) {
    OrthGrid g[2] = {};
    for (int i = 0; i < njob; ++i) {
        const int blocks = job[i].blocks > 0 ? job[i].blocks : gram_blocks(job[i].n, LP);
        if (sum && !orth_apply_sums(blocks, LP)) return LRQMM_ERR_UNSUPPORTED;
        const int units = ceil_div(job[i].n, 64);
        g[i].rows = 64 * ceil_div(units, ORTH_BLOCKS);
        g[i].nbY = ceil_div(job[i].n, g[i].rows);
        g[i].nb = g[i].nbY + (LP == 16 && job[i].M ? ceil_div(job[i].m, 64) : 0);
        g[i].parts = sum ? blocks : 0;
    }
    const dim3 grid(g[0].nb + g[1].nb);
    NT_SWITCH(LP / 16, hipLaunchKernelGGL((orth_apply_kernel<NT_>), grid, dim3(256), 0, st, job[0], job[njob - 1], g[0], g[1], ell));
    LRQ_CHECK_LAUNCH();
    return LRQMM_OK;
}

int launch_small_svd(const SvdJob* job, int njob, int ell, int LP, int rank, hipStream_t st) {
    const SvdJob j0 = job[0], j1 = job[njob - 1];
    // (NB: 2 x 2 blocks per update thread of the Jacobi solver; LW: register columns of the tridiagonalization)
#define LRQ_SVD(NB, LW) hipLaunchKernelGGL((small_svd_kernel<NB, LW>), dim3(njob), dim3(SVD_THREADS), 0, st, j0, j1, ell, LP, rank)
    if (ell <= 16)      LRQ_SVD(1, 16);
    else if (ell <= 24) LRQ_SVD(1, 24);
    else if (ell <= 32) LRQ_SVD(1, 32);
    else if (ell <= 40) LRQ_SVD(1, 40);
    else if (ell <= 48) LRQ_SVD(2, 48);
    else if (ell <= 64) LRQ_SVD(3, 64);
    else                LRQ_SVD(4, 80);
#undef LRQ_SVD
    LRQ_CHECK_LAUNCH();
    return LRQMM_OK;
}

int launch_take_basis(const BasisJob* job, int njob, int LP, int rank, hipStream_t st) {
    if (LP != 16 || rank < 1 || rank > 16) return LRQMM_ERR_UNSUPPORTED;
    BasisGrid g[2] = {};
    for (int i = 0; i < njob; ++i) {
        g[i].nbV = ceil_div(job[i].cols, 16);
        g[i].nb = g[i].nbV + (int)(((size_t)job[i].rows * rank + 1023) / 1024);
    }
    hipLaunchKernelGGL(take_basis_kernel, dim3(g[0].nb + g[1].nb), dim3(256), 0, st, job[0], job[njob - 1], g[0], g[1], rank);
    LRQ_CHECK_LAUNCH();
    return LRQMM_OK;
}

int launch_basis_panels(const BasisPanels& in, hipStream_t st) {
    BasisPanels a = in;
    a.slices = basis_slices(a.K);
    if (a.slices == 0 || a.r < 1 || a.r > 16) return LRQMM_ERR_UNSUPPORTED;
    a.nkb = pk_kblocks(a.K);
    a.per = ceil_div(a.nkb, a.slices);
    hipLaunchKernelGGL(basis_panels_kernel, dim3(a.slices + ceil_div(a.N, 64)), dim3(1024), 0, st, a);
    LRQ_CHECK_LAUNCH();
    return LRQMM_OK;
}
