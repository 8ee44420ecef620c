// Streaming products with the quantization residual R = X - Dequant(Quant(X))
// (paper: Algorithm 2, dequantization and residual steps, for R; Background 2.1 / Algorithm 1 for the
// products R.Omega, R^T Q, R Z, Q^T R of the randomized range finder), and the
// code-matrix products in the compensation terms of Algorithm 2 (A~ W and V^T B~).
//
// R is never stored: each pass re-reads the float32 operand once from HBM and
// regenerates the residual in registers from the per-group scales.  The
// tall-skinny contraction runs on the fp32 matrix cores (v_mfma_f32_16x16x4_f32);
// since the reduction index may be visited in any order, each lane loads 16
// contiguous bytes and the MFMA k-index is permuted to match.
//
// MFMA 16x16x4 f32 operand layout (lane l): A[i = l%16][k = l/16],
// B[k = l/16][j = l%16], D[i = 4*(l/16)+v][j = l%16] for v = 0..3.
#include <type_traits>
#include "kernels.h"

#define KCHUNK 128   // reduction elements staged per LDS step in the N-type kernels

__device__ __forceinline__ v4f mfma16(float a, float b, v4f c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Register image of one thread's share of W[k0 .. k0+KCHUNK)[0..16) (row-major, ld = 16).
struct WStage {
    static constexpr int LP = 16;
    static constexpr int N4 = KCHUNK * LP / 4 / 256;   // float4 per thread
    float4 v[N4];
    __device__ __forceinline__ void load_full(const float* __restrict__ W, int k0) {
#pragma unroll
        for (int u = 0; u < N4; ++u)
            v[u] = *reinterpret_cast<const float4*>(W + (size_t)k0 * LP + (threadIdx.x + 256 * u) * 4);
    }
    __device__ __forceinline__ void load(const float* __restrict__ W, int k0, int kend) {
#pragma unroll
        for (int u = 0; u < N4; ++u) {
            const int e = (threadIdx.x + 256 * u) * 4;
            const int kk = e / LP, n = e % LP;
            const int kr = min(k0 + kk, kend - 1);          // branch free: clamp, then select
            const float4 t = *reinterpret_cast<const float4*>(W + (size_t)kr * LP + n);
            const bool ok = k0 + kk < kend;
            v[u] = make_float4(ok ? t.x : 0.f, ok ? t.y : 0.f, ok ? t.z : 0.f, ok ? t.w : 0.f);
        }
    }
    __device__ __forceinline__ void store(float* __restrict__ wl) const {   // LDS row stride LP+4
#pragma unroll
        for (int u = 0; u < N4; ++u) {
            const int e = (threadIdx.x + 256 * u) * 4;
            const int kk = e / LP, n = e % LP;
            *reinterpret_cast<float4*>(wl + kk * (LP + 4) + n) = v[u];
        }
    }
};

// Quantization fused into the first residual product (the sketch pass): with the group maxima known, one
// read of the operand yields both its codes and Y = R.Omega.  amax: the group maxima (rows of X for AXIS 0,
// columns for AXIS 1); lam_out / s_out: the step vectors lambda = qmax/amax, s = amax/qmax that the later
// passes read; codes: rows x cols row-major (AXIS 0) or transposed, cols x rows (AXIS 1), or the same matrix packed (PK6, PK8).
enum { QOUT_NONE = 0, QOUT_BYTES = 1 };         // or PK6, PK8
struct QOut {
    const float* amax;
    float* lam_out;
    float* s_out;
    int8_t* codes;
};

// One residual pass over one operand.  Kernels take two jobs, A's and B's, in one launch: the two factorizations of a
// product advance together, one launch per step for both.
struct PassJob {
    const float *X, *lam, *sc, *W;
    float* partial;
    int ldx, rows, cols, chunk, nbx;        // nbx: workgroups of one range of the reduction
    QOut qo;
    const int* run;             // (see PassOperand)
};
#define LRQ_PASS_JOB(J)                                                                                      \
    const float* __restrict__ const X = (J).X;                                                               \
    const float* __restrict__ const lam = (J).lam;                                                           \
    const float* __restrict__ const sc = (J).sc;                                                             \
    const float* __restrict__ const W = (J).W;                                                               \
    float* __restrict__ const partial = (J).partial;                                                         \
    const int ldx = (J).ldx, rows = (J).rows, cols = (J).cols, chunk = (J).chunk

// ---------------------------------------------------------------------------
// N-type: partial[split][rows][LP] = R[:, k-range] . W[k-range, :]
// One workgroup per 64 rows and range of the reduction (rows fastest, job a before job b); 4 waves x 16 rows.  Per KCHUNK columns: the W chunk goes
// through double-buffered LDS, and both the next chunk of X and of W are already in
// flight (in registers) while the matrix cores work on the current one.
// ---------------------------------------------------------------------------
struct NSmem32 {
    float wl[2][KCHUNK * 20];
    float sl[2][2 * KCHUNK];        // per-column lambda | step of the chunk (AXIS 1)
};
template <int AXIS>
__device__ __forceinline__ void resid_mul_n_body(const PassJob& job, QuantParams q, int bx, int by, NSmem32& sm) {
    LRQ_PASS_JOB(job);
    constexpr int LP = 16;
    constexpr int KC = KCHUNK;
    constexpr int KS = KC / 16;          // float4 loads per lane per chunk
    auto& wl = sm.wl;
    auto& sl = sm.sl;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int r = lane & 15, g = lane >> 4;
    const int row = min(bx * 64 + wave * 16 + r, rows - 1);      // past the end: the last row, not stored
    const float* xp = X + (size_t)row * ldx;
    const int kb = by * chunk;
    const int ke = min(cols, kb + chunk);
    float lam_r = 0.f, s_r = 0.f;
    if (AXIS == 0) {
        lam_r = lam[row];
        s_r = sc[row];
    }
    v4f acc = (v4f){0.f, 0.f, 0.f, 0.f};
    float scale_reg = 0.f;     // this thread's element of the chunk's lambda (t < 128) or step vector
    WStage ws;
    const int st = threadIdx.x & (KC - 1);
    const float* const scq = (threadIdx.x & KC) == 0 ? lam : sc;
    // whole chunks without a guard (any stride and 4-byte alignment), the short last one through clamped loads
    auto load_chunk = [&](float4 (&x)[KS], int k0) {
        if (k0 + KC <= ke) {
            ws.load_full(W, k0);
#pragma unroll
            for (int j = 0; j < KS; ++j) x[j] = load4u(xp + k0 + 16 * j + 4 * g);
            if (AXIS == 1) scale_reg = scq[k0 + st];
        } else {
            ws.load(W, k0, ke);
#pragma unroll
            for (int j = 0; j < KS; ++j) x[j] = load4_tail(xp, k0 + 16 * j + 4 * g, ke);
            if (AXIS == 1) {
                const float v = scq[min(k0 + st, ke - 1)];
                scale_reg = (k0 + st < ke) ? v : 0.f;
            }
        }
    };
    int buf = 0;
    auto step = [&](float4 (&x)[KS], float4 (&xn)[KS], int k0) {
        ws.store(wl[buf]);
        if (AXIS == 1) sl[buf][threadIdx.x] = scale_reg;
        if (k0 + KC < ke) load_chunk(xn, k0 + KC);      // in flight during this chunk's products
        __syncthreads();             // wl[buf], sl[buf] complete; the other buffers no longer read
        const float* wb = wl[buf];
#pragma unroll
        for (int j = 0; j < KS; ++j) {
            float4 l4, s4;
            if (AXIS == 0) {
                l4 = make_float4(lam_r, lam_r, lam_r, lam_r);
                s4 = make_float4(s_r, s_r, s_r, s_r);
            } else {
                l4 = *reinterpret_cast<const float4*>(&sl[buf][16 * j + 4 * g]);
                s4 = *reinterpret_cast<const float4*>(&sl[buf][KC + 16 * j + 4 * g]);
            }
            const float res[4] = {quant_residual(x[j].x, l4.x, s4.x, q), quant_residual(x[j].y, l4.y, s4.y, q),
                                  quant_residual(x[j].z, l4.z, s4.z, q), quant_residual(x[j].w, l4.w, s4.w, q)};
#pragma unroll
            for (int t = 0; t < 4; ++t) acc = mfma16(res[t], wb[(16 * j + 4 * g + t) * (LP + 4) + r], acc);
        }
        buf ^= 1;
    };
    float4 xa[KS], xb[KS];
    if (kb < ke) load_chunk(xa, kb);
    for (int k0 = kb; k0 < ke; k0 += 2 * KC) {      // two chunks per round: the register sets swap roles
        step(xa, xb, k0);
        if (k0 + KC < ke) step(xb, xa, k0 + KC);
    }
    float* out = partial + (size_t)by * rows * LP;
    const int orow0 = bx * 64 + wave * 16 + 4 * g;
#pragma unroll
    for (int v = 0; v < 4; ++v)
        if (orow0 + v < rows) out[(size_t)(orow0 + v) * LP + r] = acc[v];
}

// Workgroups [0, nb0) work on job a (scales by row), the rest on job b (scales by column); likewise in the kernels below.
__global__ __launch_bounds__(256) void resid_mul_n_kernel(PassJob a, PassJob b, int nb0, QuantParams q) {
    __shared__ __align__(16) NSmem32 sm;
    const int id = blockIdx.x;
    if (id < nb0) resid_mul_n_body<0>(a, q, id % a.nbx, id / a.nbx, sm);
    else          resid_mul_n_body<1>(b, q, (id - nb0) % b.nbx, (id - nb0) / b.nbx, sm);
}

template <int ROUND_MODE>
__device__ __forceinline__ float quant_code_residual(float x, float lam, float s, const QuantParams& q, float& code) {
    const float t = x * lam;
    const float c = ROUND_MODE == 0 ? floorf(t) : rintf(t);
    code = clamp_code(c, q);
    return fmaf(-code, s, x);
}

// ---------------------------------------------------------------------------
// Row quantization (Eq. (quantA), one scale per row of A) and the sketch product Y = R.Omega (Algorithm 1, the
// sample matrix) from ONE read of the operand, for short rows (cols <= 576, a multiple of 16) and sketches
// padded to 16 columns.  A tile is 16 rows; workgroups of 8 waves are persistent, take a contiguous run of
// tiles, and load tile i+1 into a second register set while tile i is worked on.
//   * Wave w reads rows 2w and 2w+1 of the tile, adjacent lanes adjacent 16-byte pieces (NV float4 per lane), so
//     global loads and the code stores are fully coalesced and a row's maximum is a reduction inside one wave.
//   * The residuals go to LDS as a 16-row tile (row stride = 4 mod 64 floats: the 64 lanes of a matrix-core operand
//     read 64 different banks).  For the product the waves split the reduction: wave w always takes the same
//     columns, so its sketch operands stay in registers (4 NV values) for the life of the workgroup.
//   * The eight partial products of a tile meet in LDS and are added in the order of the waves, so the result
//     does not depend on the launch.  Two barriers per tile.
//   * A finished 16 x 16 tile of Y stays in LDS until the next barrier, where threads 0-255 add its Y^T Y to the
//     workgroup's float64 Gram matrix (also in LDS); at the end each workgroup leaves gpart[block][16][16], which
//     is what the orthonormalization needs next: no separate pass over Y forms it.
// amax, lam_out, s_out and the codes carry the bits the separate quantization kernel writes.
// ---------------------------------------------------------------------------
template <int NS>     // matrix-core steps (of 4 columns) per wave: ceil(cols / 32)
__global__ __launch_bounds__(512, 4) void quant_sketch_rows_kernel(
    const float* __restrict__ X, int ldx, int rows, int cols, QuantParams q, const float* __restrict__ W,
    float* __restrict__ Y, double* __restrict__ gpart, float* __restrict__ amax, float* __restrict__ lam_out,
    float* __restrict__ s_out, int8_t* __restrict__ codes) {
    constexpr int NV = (NS + 3) / 4;                     // 16-byte pieces per lane: ceil(cols / 128)
    extern __shared__ __align__(16) float rt[];          // residual tile: 16 rows of ldr floats
    __shared__ float pacc[8][256];
    __shared__ float yt[16][17];                         // the last finished tile of Y (rows past the end: zeros)
    __shared__ double gl[256];                           // the workgroup's Y^T Y so far, entry (t / 16, t % 16) by thread t
    if (threadIdx.x < 256) gl[threadIdx.x] = 0.0;        // (kept in LDS: no register lives across the tile loop for it)
    auto gram_tile = [&] {
        if (threadIdx.x < 256) {
            const int ga = threadIdx.x >> 4, gb = threadIdx.x & 15;
            double gacc = gl[threadIdx.x];
#pragma unroll
            for (int rr = 0; rr < 16; ++rr) gacc = fma((double)yt[rr][ga], (double)yt[rr][gb], gacc);
            gl[threadIdx.x] = gacc;
        }
    };
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int r = lane & 15, g = lane >> 4;
    const int cpr = cols >> 2;                           // 16-byte pieces, and steps, per row
    const int ldr = cols + ((68 - (cols & 63)) & 63);
    const int spw = (cpr + 7) >> 3;                      // steps per wave (= NS)
    const int s0 = min(cpr, wave * spw), s1 = min(cpr, s0 + spw);
    const int ntiles = (rows + 15) >> 4;
    const int t0 = (int)((long long)blockIdx.x * ntiles / gridDim.x);
    const int t1 = (int)((long long)(blockIdx.x + 1) * ntiles / gridDim.x);
    if (t0 >= t1) return;                                // uniform
    float wreg[NS];      // B operands: Omega[4 s + g][r] for the wave's steps
#pragma unroll
    for (int i = 0; i < NS; ++i) {
        const float v = W[(size_t)(4 * min(s0 + i, cpr - 1) + g) * 16 + r];
        wreg[i] = s0 + i < s1 ? v : 0.f;
    }
    // piece u of a lane: number lane + 64 u of the wave's two rows
    auto piece = [&](int u, int& rl, int& cc) {
        const int c = lane + 64 * u;
        rl = c >= cpr ? 1 : 0;
        cc = c - (rl ? cpr : 0);
        return c < 2 * cpr;
    };
    // No guard on the values: rows past the end read row 0 and only reach their own maxima, codes and output
    // rows, none of which is stored; pieces past the two rows read piece 0 and are not used.
    auto load_tile = [&](float4 (&x)[NV], int tile) {
        const int row0 = tile * 16 + 2 * wave;
        const float* p0 = X + (size_t)(row0 < rows ? row0 : 0) * ldx;
        const float* p1 = X + (size_t)(row0 + 1 < rows ? row0 + 1 : 0) * ldx;
#pragma unroll
        for (int u = 0; u < NV; ++u) {
            int rl, cc;
            const bool valid = piece(u, rl, cc);
            x[u] = *reinterpret_cast<const float4*>((rl ? p1 : p0) + 4 * (valid ? cc : 0));
        }
    };
    auto process = [&](const float4 (&x)[NV], int tile) {
        const int row0 = tile * 16 + 2 * wave;
        float m0 = 0.f, m1 = 0.f;
#pragma unroll
        for (int u = 0; u < NV; ++u) {
            int rl, cc;
            const bool valid = piece(u, rl, cc);
            const float mm = fmaxf(fmaxf(fabsf(x[u].x), fabsf(x[u].y)), fmaxf(fabsf(x[u].z), fabsf(x[u].w)));
            if (valid && rl == 0) m0 = fmaxf(m0, mm);
            if (valid && rl == 1) m1 = fmaxf(m1, mm);
        }
        m0 = wave_max(m0);
        m1 = wave_max(m1);
        float lam0, sc0, lam1, sc1;
        make_scales(m0, q.qmaxf, lam0, sc0);
        make_scales(m1, q.qmaxf, lam1, sc1);
        if (lane < 2 && row0 + lane < rows) {
            amax[row0 + lane] = lane ? m1 : m0;
            lam_out[row0 + lane] = lane ? lam1 : lam0;
            s_out[row0 + lane] = lane ? sc1 : sc0;
        }
        auto quantize = [&](auto mode) {         // one uniform branch on the rounding mode per tile
            constexpr int RM = decltype(mode)::value;
#pragma unroll
            for (int u = 0; u < NV; ++u) {
                int rl, cc;
                if (!piece(u, rl, cc)) continue;
                const float lam_r = rl ? lam1 : lam0, s_r = rl ? sc1 : sc0;
                float c0, c1, c2, c3;
                float4 res;
                res.x = quant_code_residual<RM>(x[u].x, lam_r, s_r, q, c0);
                res.y = quant_code_residual<RM>(x[u].y, lam_r, s_r, q, c1);
                res.z = quant_code_residual<RM>(x[u].z, lam_r, s_r, q, c2);
                res.w = quant_code_residual<RM>(x[u].w, lam_r, s_r, q, c3);
                const int i0 = (int)c0, i1 = (int)c1, i2 = (int)c2, i3 = (int)c3;
                const uint32_t pk = (uint32_t)(i0 & 0xff) | ((uint32_t)(i1 & 0xff) << 8) |
                                    ((uint32_t)(i2 & 0xff) << 16) | ((uint32_t)(i3 & 0xff) << 24);
                if (row0 + rl < rows) *reinterpret_cast<uint32_t*>(codes + (size_t)(row0 + rl) * cols + 4 * cc) = pk;
                *reinterpret_cast<float4*>(rt + (2 * wave + rl) * ldr + 4 * cc) = res;
            }
        };
        if (q.round_mode == 0) quantize(std::integral_constant<int, 0>{});
        else quantize(std::integral_constant<int, 1>{});
        __syncthreads();        // the tile's residuals are in LDS; the last tile's partial products have been read
        if (tile > t0) gram_tile();     // the previous tile of Y is in LDS too
        v4f acc = (v4f){0.f, 0.f, 0.f, 0.f};
        const float* ap = rt + r * ldr + 4 * s0 + g;
#pragma unroll
        for (int i = 0; i < NS; ++i)
            if (s0 + i < s1) acc = mfma16(ap[4 * i], wreg[i], acc);      // the same for all lanes of a wave
#pragma unroll
        for (int v = 0; v < 4; ++v) pacc[wave][(4 * g + v) * 16 + r] = acc[v];
        __syncthreads();        // the eight partial products are in LDS; the residual tile has been read
        if (threadIdx.x < 256) {
            float sum = pacc[0][threadIdx.x];
#pragma unroll
            for (int w = 1; w < 8; ++w) sum += pacc[w][threadIdx.x];
            const int orow = tile * 16 + (threadIdx.x >> 4);
            if (orow < rows) Y[(size_t)orow * 16 + (threadIdx.x & 15)] = sum;
            yt[threadIdx.x >> 4][threadIdx.x & 15] = orow < rows ? sum : 0.f;
        }
    };
    float4 xa[NV], xb[NV];
    int tile = t0;
    load_tile(xa, tile);
    while (true) {          // two tiles per round: the register sets swap roles
        load_tile(xb, min(tile + 1, t1 - 1));
        process(xa, tile);
        if (++tile >= t1) break;
        load_tile(xa, min(tile + 1, t1 - 1));
        process(xb, tile);
        if (++tile >= t1) break;
    }
    __syncthreads();
    gram_tile();
    if (threadIdx.x < 256) gpart[(size_t)blockIdx.x * 256 + threadIdx.x] = gl[threadIdx.x];
}

// ---------------------------------------------------------------------------
// The same product on the bf16 matrix cores.  A float32 value is the exact sum of three
// bfloat16 planes (8 + 8 + 8 significant bits: round to nearest, subtract, repeat), and the
// product of two such sums is evaluated with the six plane products whose weight is at least
// 2^-16 of the leading one (r1 w1, r1 w2, r2 w1, r1 w3, r2 w2, r3 w1), each exact, accumulated
// in float32 by the matrix core: the dropped products are below 2^-24 of the leading one,
// the size of the float32 accumulation rounding itself.  Six v_mfma_f32_16x16x32_bf16 take
// 96 cycles per 32 k against 256 for eight v_mfma_f32_16x16x4_f32, and these kernels are
// bound by the matrix cores as soon as two of them share the chip.
// Operand layout (lane l): A[i = l%16][k = 8(l/16) .. +8], B[k = 8(l/16) .. +8][j = l%16],
// D[i = 4(l/16)+v][j = l%16].  The 8 k-slots of lane group g in a 32-deep step are the
// columns 4g .. 4g+3 and 16+4g .. 16+4g+3 of that step (two 16-byte loads of X); W is staged
// in LDS as three planes [plane][n][k] with k in that slot order, so a B operand is one
// 16-byte LDS read.
// ---------------------------------------------------------------------------
// acc[m][n] += a[m] . b[n] for NA x NB independent accumulators: the six plane products are
// the outer loop (smallest terms first), so consecutive matrix instructions never depend on
// each other.
// Reduced precision (the compensation terms "in half precision", Methodology, after Eq. (gemm_r_split)):
// with PL = 2 planes per operand the three products of weight >= 2^-8 are formed (relative error of a
// product 2^-16), with PL = 1 the leading product alone (2^-8, plain bfloat16 operands).
template <int NA, int NB, int PL = 3>
__device__ __forceinline__ void mfma_planes(const Planes3 (&a)[NA], const Planes3 (&b)[NB], v4f (&acc)[NA][NB]) {
#define LRQ_PP(PA, PB)                                                                               \
    _Pragma("unroll") for (int m = 0; m < NA; ++m) _Pragma("unroll") for (int n = 0; n < NB; ++n)     \
        acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[m].PA, b[n].PB, acc[m][n], 0, 0, 0);
    if constexpr (PL >= 3) {
        LRQ_PP(p3, p1)
        LRQ_PP(p2, p2)
        LRQ_PP(p1, p3)
    }
    if constexpr (PL >= 2) {
        LRQ_PP(p2, p1)
        LRQ_PP(p1, p2)
    }
    LRQ_PP(p1, p1)
#undef LRQ_PP
}

// One thread's share of the chunk W[k0 .. k0+KC)[0..LP): units (n, group), a unit being the 8
// rows of W that form one lane group's k-slots of one 32-deep step, for one column n.
template <int NT, int KC, int THREADS, int PL = 3>
struct WStageBf16 {
    static constexpr int LP = NT * 16;
    static constexpr int LDK = KC + 8;                      // plane row stride in bfloat16
    static constexpr int UNITS = LP * (KC / 8);
    static constexpr int NU = (UNITS + THREADS - 1) / THREADS;
    float v[NU][8];
    int off[NU];        // this thread's units: offset of their first element inside a chunk of W
    // row of the lane group's k-slot e relative to its slot 0 (row 4 g of the step)
    static __device__ __forceinline__ int slot(int e) { return (e & 3) + 16 * (e >> 2); }
    __device__ __forceinline__ void init() {
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int unit = min((int)threadIdx.x + THREADS * u, UNITS - 1);
            const int n = unit % LP, grp = unit / LP;
            off[u] = (32 * (grp >> 2) + 4 * (grp & 3)) * LP + n;
        }
    }
    // whole chunk inside the reduction range: no clamps, constant offsets from one base
    __device__ __forceinline__ void load_full(const float* __restrict__ W, int k0) {
        const float* p = W + (size_t)k0 * LP;
#pragma unroll
        for (int u = 0; u < NU; ++u)
#pragma unroll
            for (int e = 0; e < 8; ++e) v[u][e] = p[off[u] + slot(e) * LP];
    }
    __device__ __forceinline__ void load(const float* __restrict__ W, int k0, int kend) {
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int unit = min((int)threadIdx.x + THREADS * u, UNITS - 1);
            const int n = unit % LP, grp = unit / LP;        // grp = 4 (step in chunk) + lane group
            const int kbase = k0 + 32 * (grp >> 2) + 4 * (grp & 3);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int k = kbase + slot(e);
                const float t = W[(size_t)min(k, kend - 1) * LP + n];   // branch free: clamp, then select
                v[u][e] = k < kend ? t : 0.f;
            }
        }
    }
    __device__ __forceinline__ void store(uint16_t* __restrict__ wl) const {
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int unit = (int)threadIdx.x + THREADS * u;
            if (unit < UNITS) {
                const int n = unit % LP, grp = unit / LP;
                const Planes3 pl = split_planes<PL>(v[u]);
                uint16_t* dst = wl + n * LDK + 8 * grp;
                *reinterpret_cast<v8bf16*>(dst) = pl.p1;
                if (PL >= 2) *reinterpret_cast<v8bf16*>(dst + LP * LDK) = pl.p2;
                if (PL >= 3) *reinterpret_cast<v8bf16*>(dst + 2 * LP * LDK) = pl.p3;
            }
        }
    }
};

// A workgroup of NW waves takes 16 NW rows and one range of the reduction, in chunks of KC columns.  Any shape, stride and
// 4-byte alignment: whole chunks are loaded without a guard, 16 bytes per lane, and only the last chunk
// of the reduction, when it is not whole, through clamped loads (the branch is the same for all waves); rows past
// the end re-read the last row and are not stored.  FULL: every chunk is whole and, with the code output, so are the
// row blocks -- without the branches a 512 x 4096 operand (24 columns) factors 4 % faster, 4096^3 0.7 %.
template <int NT, int PL, int QOUT, int NW, int KC>
struct NSmem {
    static constexpr int RB = 16 * NW;      // rows per workgroup
    static constexpr int LDK = WStageBf16<NT, KC, 64 * NW, PL>::LDK;
    static constexpr int CT0 = RB * (KC + 16), CT1 = KC * (RB + 16);
    int8_t ct[QOUT ? 2 : 1][QOUT ? (CT0 > CT1 ? CT0 : CT1) : 16];       // staged code tiles
    uint16_t wl[2][PL * NT * 16 * LDK];
    float sl[2][2 * KC];                    // per-column lambda | step of the chunk (AXIS 1)
};
template <int NT, int AXIS, int PL, int QOUT, int NW, int KC, bool FULL>
__device__ __forceinline__ void resid_mul_n_bf16_body(const PassJob& job, QuantParams q, int bx, int by,
                                                      NSmem<NT, PL, QOUT, NW, KC>& sm) {
    LRQ_PASS_JOB(job);
    const QOut& qo = job.qo;
    constexpr int LP = NT * 16;
    constexpr int THREADS = 64 * NW, RB = 16 * NW;     // rows per workgroup
    constexpr int CTW = AXIS == 0 ? RB : KC;                // staged code tile: rows ...
    constexpr int CTL = AXIS == 0 ? KC : RB;                // ... of this many codes
    constexpr int CTS = CTL + 16;                           // row stride, bytes
    constexpr int KS = KC / 16;                             // float4 loads per lane and chunk
    using WS = WStageBf16<NT, KC, THREADS, PL>;
    constexpr int LDK = WS::LDK;
    auto& ct = sm.ct;
    auto& wl = sm.wl;
    auto& sl = sm.sl;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int r = lane & 15, g = lane >> 4;
    const int row0 = bx * RB + wave * 16;
    const int kb = by * chunk;
    const int ke = min(cols, kb + chunk);
    const int row = min(row0 + r, rows - 1);
    const float* const xp = X + (size_t)row * ldx;
    float lam_r = 0.f, s_r = 0.f;
    if (AXIS == 0) {
        if (QOUT) {
            make_scales(qo.amax[row], q.qmaxf, lam_r, s_r);
            if (by == 0 && g == 0) {
                qo.lam_out[row] = lam_r;
                qo.s_out[row] = s_r;
            }
        } else {
            lam_r = lam[row];
            s_r = sc[row];
        }
    }
    v4f acc[1][NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[0][nt] = (v4f){0.f, 0.f, 0.f, 0.f};

    float scale_reg = 0.f;     // this thread's element of the chunk's lambda (t < KC) or step vector
    WS ws;
    ws.init();
    const int st = threadIdx.x & (KC - 1);
    const float* const scq = QOUT ? qo.amax : ((threadIdx.x & KC) == 0 ? lam : sc);
    // chunk k0: W into ws, X into x; the last chunk may be short
    float4 x[KS];
    auto load_chunk = [&](int k0) {
        if (FULL || k0 + KC <= ke) {
            ws.load_full(W, k0);
#pragma unroll
            for (int j = 0; j < KS; ++j) x[j] = load4u(xp + 4 * g + k0 + 16 * j);
            if (AXIS == 1) scale_reg = scq[k0 + st];     // (QOUT: the column's maximum, turned into lambda or s below)
        } else {
            ws.load(W, k0, ke);
#pragma unroll
            for (int j = 0; j < KS; ++j) x[j] = load4_tail(xp, k0 + 16 * j + 4 * g, ke);
            if (AXIS == 1) {
                const float v = scq[min(k0 + st, ke - 1)];
                scale_reg = (k0 + st < ke) ? v : 0.f;
            }
        }
    };
    // QOUT: the RB x KC code tile of a chunk is staged in LDS (two tiles, so the chunk loop keeps its single
    // barrier) and leaves for global memory one chunk later, 16 bytes per thread.  Tile rows are X rows (AXIS 0,
    // codes row-major) or X columns (AXIS 1, codes transposed).  16-byte stores at any alignment; the last group of
    // a row of codes byte by byte when it is not whole.  Packed: one lane of a block (32 codes) per thread.
    auto flush_codes = [&](int tb, int kprev) {
        constexpr int PIECES = CTW * CTL / 16;
        const int r0 = AXIS == 0 ? bx * RB : kprev, nrow = AXIS == 0 ? rows : cols;
        const int c0 = AXIS == 0 ? kprev : bx * RB, ld = AXIS == 0 ? cols : rows;
        if constexpr (QOUT == PK6 || QOUT == PK8) {
            store_packed_tile<QOUT, CTW, CTL, CTS, AXIS == 1>(ct[tb], reinterpret_cast<uint8_t*>(qo.codes), r0, nrow, c0, ld, threadIdx.x, THREADS);
            return;
        }
        int8_t* const base = qo.codes + (size_t)r0 * ld + c0;
        const bool whole = FULL || (r0 + CTW <= nrow && c0 + CTL <= ld);      // uniform
        for (int e = threadIdx.x; e < PIECES; e += THREADS) {
            const int tr = e / (CTL / 16), seg = (e % (CTL / 16)) * 16;
            const int8_t* src = &ct[tb][tr * CTS + seg];
            int8_t* dst = base + (size_t)tr * ld + seg;
            if (whole || (r0 + tr < nrow && c0 + seg + 16 <= ld))
                __builtin_memcpy(dst, __builtin_assume_aligned(src, 16), 16);
            else if (r0 + tr < nrow) {
                const int n = ld - c0 - seg;
#pragma unroll 1
                for (int b = 0; b < n; ++b) dst[b] = src[b];
            }
        }
    };
    int buf = 0;
    if (kb < ke) load_chunk(kb);
    for (int k0 = kb; k0 < ke; k0 += KC, buf ^= 1) {
        ws.store(wl[buf]);
        if (AXIS == 1 && threadIdx.x < 2 * KC) {
            if (QOUT) {     // scale_reg holds the column maximum: lambda for the first KC threads, the step for the next
                float l, stp;
                make_scales(scale_reg, q.qmaxf, l, stp);
                scale_reg = (threadIdx.x & KC) == 0 ? l : stp;
                if (bx == 0 && k0 + st < cols) ((threadIdx.x & KC) == 0 ? qo.lam_out : qo.s_out)[k0 + st] = scale_reg;
            }
            sl[buf][threadIdx.x] = scale_reg;
        }
        __syncthreads();             // wl[buf], sl[buf] complete; the other buffers no longer read
        if (QOUT && k0 > kb) flush_codes(buf ^ 1, k0 - KC);
        Planes3 ap[KC / 32][1];
        auto residuals = [&](auto mode) {       // one uniform branch on the rounding mode per chunk
            constexpr int RM = decltype(mode)::value;
#pragma unroll
            for (int jj = 0; jj < KC / 32; ++jj) {
                float res[8];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int j = 2 * jj + h;
                    float4 l4, s4;
                    if (AXIS == 0) {
                        l4 = make_float4(lam_r, lam_r, lam_r, lam_r);
                        s4 = make_float4(s_r, s_r, s_r, s_r);
                    } else {
                        l4 = *reinterpret_cast<const float4*>(&sl[buf][16 * j + 4 * g]);
                        s4 = *reinterpret_cast<const float4*>(&sl[buf][KC + 16 * j + 4 * g]);
                    }
                    const float4 xv = x[j];
                    if (QOUT) {
                        float c0, c1, c2, c3;
                        res[4 * h + 0] = quant_code_residual<RM>(xv.x, l4.x, s4.x, q, c0);
                        res[4 * h + 1] = quant_code_residual<RM>(xv.y, l4.y, s4.y, q, c1);
                        res[4 * h + 2] = quant_code_residual<RM>(xv.z, l4.z, s4.z, q, c2);
                        res[4 * h + 3] = quant_code_residual<RM>(xv.w, l4.w, s4.w, q, c3);
                        constexpr bool SIX = QOUT == PK6;
                        const int i0 = SIX ? (int)six_bits(c0) : (int)c0, i1 = SIX ? (int)six_bits(c1) : (int)c1;
                        const int i2 = SIX ? (int)six_bits(c2) : (int)c2, i3 = SIX ? (int)six_bits(c3) : (int)c3;
                        const int lr = wave * 16 + r;     // row inside the workgroup
                        if (AXIS == 0) {    // four codes along the row: one word (packed: of 24 bits)
                            const uint32_t pk = SIX ? (uint32_t)(i0 | (i1 << 6) | (i2 << 12) | (i3 << 18))
                                                    : (uint32_t)(i0 & 0xff) | ((uint32_t)(i1 & 0xff) << 8) |
                                                          ((uint32_t)(i2 & 0xff) << 16) | ((uint32_t)(i3 & 0xff) << 24);
                            *reinterpret_cast<uint32_t*>(&ct[buf][lr * CTS + 16 * j + 4 * g]) = pk;
                        } else {            // four columns of the transposed tile
                            int8_t* cp = &ct[buf][(16 * j + 4 * g) * CTS + lr];
                            cp[0] = (int8_t)i0;
                            cp[CTS] = (int8_t)i1;
                            cp[2 * CTS] = (int8_t)i2;
                            cp[3 * CTS] = (int8_t)i3;
                        }
                    } else {
                        res[4 * h + 0] = quant_residual_m<RM>(xv.x, l4.x, s4.x, q);
                        res[4 * h + 1] = quant_residual_m<RM>(xv.y, l4.y, s4.y, q);
                        res[4 * h + 2] = quant_residual_m<RM>(xv.z, l4.z, s4.z, q);
                        res[4 * h + 3] = quant_residual_m<RM>(xv.w, l4.w, s4.w, q);
                    }
                }
                ap[jj][0] = split_planes<PL>(res);
            }
        };
        if (q.round_mode == 0) residuals(std::integral_constant<int, 0>{});
        else residuals(std::integral_constant<int, 1>{});
        if (k0 + KC < ke) load_chunk(k0 + KC);      // in flight during this chunk's products
        const uint16_t* wb = wl[buf];
#pragma unroll
        for (int jj = 0; jj < KC / 32; ++jj) {
            Planes3 bp[NT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const uint16_t* src = wb + (16 * nt + r) * LDK + 32 * jj + 8 * g;
                bp[nt].p1 = *reinterpret_cast<const v8bf16*>(src);
                if (PL >= 2) bp[nt].p2 = *reinterpret_cast<const v8bf16*>(src + LP * LDK);
                if (PL >= 3) bp[nt].p3 = *reinterpret_cast<const v8bf16*>(src + 2 * LP * LDK);
            }
            mfma_planes<1, NT, PL>(ap[jj], bp, acc);
        }
    }
    if (QOUT && kb < ke) {
        __syncthreads();
        flush_codes(buf ^ 1, kb + (ke - kb - 1) / KC * KC);
    }
    float* out = partial + (size_t)by * rows * LP;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int orow = row0 + 4 * g + v;
            if (orow < rows) out[(size_t)orow * LP + 16 * nt + r] = acc[0][nt][v];
        }
}

template <int NT, int PL, int QOUT, int NW, int KC, bool FULL>
__global__ __launch_bounds__(64 * NW, NT <= 2 ? 4 : (NT <= 3 ? 3 : 2)) void resid_mul_n_bf16_kernel(PassJob a, PassJob b, int nb0,
                                                                                              QuantParams q) {
    __shared__ __align__(16) NSmem<NT, PL, QOUT, NW, KC> sm;
    const int id = blockIdx.x;
    if (id < nb0) resid_mul_n_bf16_body<NT, 0, PL, QOUT, NW, KC, FULL>(a, q, id % a.nbx, id / a.nbx, sm);
    else          resid_mul_n_bf16_body<NT, 1, PL, QOUT, NW, KC, FULL>(b, q, (id - nb0) % b.nbx, (id - nb0) / b.nbx, sm);
}

// ---------------------------------------------------------------------------
// Panels of the rank-2r update: the code products A~ W and (V^T B~)^T and what is made of them (see gemm.hip)
//   Lp[i][c] = U[i][c] Sig[c] (c < r),  sA[i] (Aq W)[i][c - r] (r <= c < 2r),  0 beyond;
//   Rp[j][c] = sB[j] (BqT V)[j][c] + sum_u X[c][u] Gam[u] Zt[u][j] (c < r),  Gam[c - r] Zt[c - r][j] (r <= c < 2r),  0 beyond.
//
// The products run on the bf16 matrix cores: an int8 code is exact in bfloat16 (8 significant bits) and the float32 factor comes as
// three bfloat16 planes hi + mid + lo (exact to 2^-27, see split_planes), so
//   code . w = code . hi + code . mid + code . lo
// holds with every product exact and float32 accumulation in the matrix core.
// v_mfma_f32_16x16x32_bf16 operand layout (lane l): A[i = l%16][k = 8(l/16) .. +8], B[k = 8(l/16) .. +8][j = l%16], D[i =
// 4(l/16)+v][j = l%16].  The reduction index may be visited in any order: in a 64-deep block lane group kq = l/16 owns k = 16 kq
// .. 16 kq + 15, the first half in step 0, the second in step 1.  The planes lie in that order (FACTOR_PIECE), so that an operand
// of a wave is 1 KB in a row and goes from memory to its registers without LDS.
//
// A workgroup takes 32 RB rows of codes over the whole reduction: its eight waves take a contiguous eighth of the k blocks each, on
// their own, loads one or more blocks ahead of the matrix cores; at the end their sums meet in LDS, are added in order, and leave
// as panel rows, so the products themselves never reach memory.  Before (K cut over workgroups, planes staged in LDS, a launch of its own that
// added the partials and formed the panels), us for both launches / this:
//   200^3 rank 10 5.3 + 6.5 / 5.1, 2000^3 rank 10 9.4 + 7.5 / 7.8, 1537 x 1021 x 2311 rank 16 13.9 + 8.3 / 8.3, 4096^3 int8 rank 16 12.7 + 9.1 /
//   12.0, int4 rank 32 14.9 + 12.0 / 18.7, 16384^3 rank 64 433 + 49 / 267, rows kernel below: 100352 x 64 x 576 rank 8 20.2 + 9.1 / 26.3.
// The planes come through every CU's L1 once per workgroup, at 40 to 45 GB/s a CU, which bounds the larger ones (64 rows a
// workgroup from 256 of them on: half the reads); touching the planes in the L2 some blocks ahead made them 15 % slower.
// FMT: PK6, PK8 (see common.h), or PK_NONE: packed rows of K bytes, read 16 bytes at a time at any alignment; the group that reaches
// past K is loaded from K - 16 and moved into place (tail16) where it is used.  All give the same bits.
// ---------------------------------------------------------------------------
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef uint32_t v6u __attribute__((ext_vector_type(6)));
typedef __bf16 v32bf __attribute__((ext_vector_type(32)));

template <bool WIDE>
__device__ __forceinline__ uint4 load_codes16(const int8_t* __restrict__ rowp, int K, int k) {
    if (WIDE) {
        uint4 v;
        __builtin_memcpy(&v, rowp + min(k, K - 16), 16);
        return v;
    }
    uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int b = 0; b < 16; ++b)
        if (k + b < K) w[b >> 2] |= (uint32_t)(uint8_t)rowp[k + b] << (8 * (b & 3));
    return make_uint4(w[0], w[1], w[2], w[3]);
}

// 8 int8 codes (two dwords) -> 8 bfloat16: float(code) keeps only its upper 16 bits.
__device__ __forceinline__ v8bf codes_to_bf16(uint32_t lo, uint32_t hi) {
    union { uint32_t u[4]; v8bf v; } r;
    const uint32_t w[2] = {lo, hi};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const float f0 = (float)(int)(int8_t)(w[h] & 0xff), f1 = (float)(int)(int8_t)((w[h] >> 8) & 0xff);
        const float f2 = (float)(int)(int8_t)((w[h] >> 16) & 0xff), f3 = (float)(int)(int8_t)(w[h] >> 24);
        r.u[2 * h + 0] = (__float_as_uint(f0) >> 16) | (__float_as_uint(f1) & 0xffff0000u);
        r.u[2 * h + 1] = (__float_as_uint(f2) >> 16) | (__float_as_uint(f3) & 0xffff0000u);
    }
    return r.v;
}

// The sum of X's slices times Gamma, zero columns from r on: r x (RP + 1) in LDS, by `threads` threads.
__device__ __forceinline__ void stage_x_gamma(const PanelArgs& a, int RP, float* __restrict__ xg, int tid, int threads) {
    const int r = a.r;
    for (int e0 = tid; e0 < r * r; e0 += 2 * threads) {      // two entries' slice loads in flight
        float x[2][LRQ_VTW_MAX_SLICES];
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int t = 0; t < LRQ_VTW_MAX_SLICES; ++t)
                x[m][t] = a.Xp[min(e0 + threads * m, r * r - 1) + (size_t)min(t, a.nslices - 1) * (r * r)];
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const int e = e0 + threads * m;
            float sum = 0.f;
#pragma unroll
            for (int t = 0; t < LRQ_VTW_MAX_SLICES; ++t) sum += t < a.nslices ? x[m][t] : 0.f;
            if (e < r * r) xg[e / r * (RP + 1) + e % r] = sum * a.Gam[e % r];
        }
    }
    for (int e = tid; e < r * (RP - r); e += threads) xg[e / (RP - r) * (RP + 1) + r + e % (RP - r)] = 0.f;
}

// Codes of one k block as a wave's operands: 32 rows as two tiles of 16, lane (li, kq) with codes 16 kq .. +16 of its rows.
template <int FMT>
struct CodeBlock {
    uint4 w[2];
    uint2 x[FMT == PK6 ? 2 : 1];
    __device__ __forceinline__ void load(const int8_t* codes, int rb, int rows, int kb, int K, int nkb, int li, int kq) {
        if constexpr (FMT == PK_NONE) {
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int8_t* row = codes + (size_t)min(32 * rb + 16 * t + li, rows - 1) * K;
                w[t] = K >= 16 ? load_codes16<true>(row, K, 64 * kb + 16 * kq) : load_codes16<false>(row, K, 16 * kq);
            }
        } else {
            const uint8_t* blk = reinterpret_cast<const uint8_t*>(codes) + ((size_t)min(rb, (rows - 1) >> 5) * nkb + kb) * pk_block(FMT);
            const int unit = 32 * (kq >> 1) + li;
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                if constexpr (FMT == PK8) w[t] = *reinterpret_cast<const uint4*>(blk + 1024 * (kq & 1) + (unit + 16 * t) * 16);
                else {      // (a lane's 24 bytes whole; the half that is wanted is picked below)
                    w[t] = *reinterpret_cast<const uint4*>(blk + (unit + 16 * t) * 16);
                    x[t] = *reinterpret_cast<const uint2*>(blk + 1024 + (unit + 16 * t) * 8);
                }
            }
        }
    }
    // -> [step][tile]
    __device__ __forceinline__ void operands(v8bf (&af)[2][2], int kb, int K, int kq) {
        if constexpr (FMT == PK6) {
            uint32_t h[2][3];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                h[t][0] = (kq & 1) ? w[t].w : w[t].x;        // (stored order: words 0 1 2 3 | 4 5)
                h[t][1] = (kq & 1) ? x[t].x : w[t].y;
                h[t][2] = (kq & 1) ? x[t].y : w[t].z;
            }
            const v6u six = {h[0][0], h[0][1], h[0][2], h[1][0], h[1][1], h[1][2]};
            const v32bf val = __builtin_amdgcn_cvt_scalef32_pk32_bf16_fp6(six, 8.0f);
            af[0][0] = __builtin_shufflevector(val, val, 0, 1, 2, 3, 4, 5, 6, 7);
            af[1][0] = __builtin_shufflevector(val, val, 8, 9, 10, 11, 12, 13, 14, 15);
            af[0][1] = __builtin_shufflevector(val, val, 16, 17, 18, 19, 20, 21, 22, 23);
            af[1][1] = __builtin_shufflevector(val, val, 24, 25, 26, 27, 28, 29, 30, 31);
        } else {
            // (codes past K meet zero planes, but the group that crosses K has to be moved into place)
            if (FMT == PK_NONE && (K & 15) && K >= 16 && 64 * kb + 64 > K) {     // uniform
#pragma unroll
                for (int t = 0; t < 2; ++t) w[t] = tail16(w[t], max(0, 64 * kb + 16 * kq - (K - 16)));
            }
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                af[0][t] = codes_to_bf16(w[t].x, w[t].y);
                af[1][t] = codes_to_bf16(w[t].z, w[t].w);
            }
        }
    }
};

// The first half (H = 0) or second half of the planes' operands of one k block.
template <int NT, int PL>
struct FactorHalf {
    v8bf b[NT][PL];
    __device__ __forceinline__ void load(const uint16_t* Wf, int kb, int h, int lane) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int pl = 0; pl < PL; ++pl)
                b[nt][pl] = *reinterpret_cast<const v8bf*>(Wf + (size_t)(((kb * NT + nt) * 3 + pl) * 2 + h) * FACTOR_PIECE + lane * 8);
    }
};
template <int NT, int PL>
__device__ __forceinline__ void panel_products(const v8bf (&af)[2], const FactorHalf<NT, PL>& f, v4f (&acc)[2][NT]) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int pl = 0; pl < PL; ++pl)
#pragma unroll
            for (int t = 0; t < 2; ++t) acc[t][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[t], f.b[nt][pl], acc[t][nt], 0, 0, 0);
}

#define PANEL_WAVES 8
#define PANEL_ROWS_MIN 16384    // rows from which panels_rows_kernel takes them
#define PANEL_TWO_MIN 256       // workgroups of 64 rows from which they are taken in place of 32
// k blocks of a wave; its sums are added to the others' in the order of the waves, whichever kernel forms them.
__host__ __device__ static inline int panel_range(int nkb) { return (nkb + PANEL_WAVES - 1) / PANEL_WAVES; }

template <int FMT, int NT, int PL, int RB>
__global__ __launch_bounds__(512, 2) void panels_kernel(PanelArgs a) {
    constexpr int RP = NT * 16, AHEAD = NT == 1 ? 3 : 2;
    __shared__ float red[PANEL_WAVES * 32 * RP];        // [wave][32 rows][RP]
    __shared__ float xg[RP * (RP + 1)];                 // X Gamma
    constexpr int OWN = 36;                             // (aligned groups of four rows)
    __shared__ __align__(16) float own[RB][RP * OWN];   // right: 32 columns of Zt, [u][row]; left: 32 rows of U Sig
    __shared__ float step[32 * RB];
    const bool right = (int)blockIdx.x < a.nbR;         // (the right panel has more to do)
    const int blk = right ? blockIdx.x : blockIdx.x - a.nbR;
    const int rows = right ? a.N : a.M, K = a.K, r = a.r, R2P = a.R2P;
    const int8_t* const codes = right ? a.codesB : a.codesA;
    const uint16_t* const Wf = right ? a.Vf : a.Wf;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int li = lane & 15, kq = lane >> 4;
    const int nkb = pk_kblocks(K), kb0 = wave * panel_range(nkb), kb1 = min(nkb, kb0 + panel_range(nkb));
    v4f acc[RB][2][NT];
#pragma unroll
    for (int b = 0; b < RB; ++b)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) acc[b][t][nt] = (v4f){0.f, 0.f, 0.f, 0.f};
    // What the panel rows need besides the products: loaded beside the first blocks, so that behind the loop nothing waits for memory
    // (loaded there / so, at 4096^3 and with one panel entry a thread behind the sums: r = 32 18.6 / 17.8 us, r = 16 12.5 / 11.5; now 15.4, 10.5).
    auto stage = [&] {
        if (right) stage_x_gamma(a, RP, xg, tid, 512);
#pragma unroll
        for (int b = 0; b < RB; ++b) {
            const int r0 = (blk * RB + b) * 32;
#pragma unroll
            for (int e0 = 0; e0 < RP * 32; e0 += 512) {
                const int e = e0 + tid;
                if (right) {
                    const int u = e >> 5, j = r0 + (e & 31);
                    const float z = a.Zt[(size_t)min(u, r - 1) * a.N + min(j, a.N - 1)];
                    own[b][u * OWN + (e & 31)] = u < r && j < a.N ? z : 0.f;
                } else if (e < 32 * r) {
                    own[b][e] = a.U[(size_t)min(r0 + e / r, a.M - 1) * a.ldu + e % r] * a.Sig[e % r];
                }
            }
        }
        if (tid < 32 * RB) step[tid] = (right ? a.sB : a.sA)[min(blk * RB * 32 + tid, rows - 1)];
    };
    // blocks ahead: whole blocks of codes, and of the planes as whole blocks, or as halves where they are wide
    if constexpr (NT <= 2 || NT * RB <= 3) {
        struct Stage { CodeBlock<FMT> c[RB]; FactorHalf<NT, PL> f[2]; } st[AHEAD];
        auto load = [&](Stage& s, int kb) {
            const int k = min(kb, nkb - 1);     // (past the end: the last one again, not used)
#pragma unroll
            for (int b = 0; b < RB; ++b) s.c[b].load(codes, blk * RB + b, rows, k, K, nkb, li, kq);
#pragma unroll
            for (int h = 0; h < 2; ++h) s.f[h].load(Wf, k, h, lane);
        };
        if (kb0 < kb1) {
#pragma unroll
            for (int i = 0; i < AHEAD - 1; ++i) load(st[i], kb0 + i);
        }
        stage();
        for (int kb = kb0; kb < kb1; kb += AHEAD) {
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) {
                if (kb + i < kb1) {
                    load(st[(i + AHEAD - 1) % AHEAD], kb + i + AHEAD - 1);
                    __builtin_amdgcn_sched_barrier(0);      // (or the loads sink to where they are used, and nothing is ahead)
#pragma unroll
                    for (int b = 0; b < RB; ++b) {
                        v8bf af[2][2];
                        st[i].c[b].operands(af, kb + i, K, kq);
#pragma unroll
                        for (int h = 0; h < 2; ++h) panel_products<NT, PL>(af[h], st[i].f[h], acc[b]);
                    }
                }
            }
        }
    } else {
        CodeBlock<FMT> c[RB];
        FactorHalf<NT, PL> f[2];
        auto load_codes = [&](int kb) {
#pragma unroll
            for (int b = 0; b < RB; ++b) c[b].load(codes, blk * RB + b, rows, min(kb, nkb - 1), K, nkb, li, kq);
        };
        if (kb0 < kb1) { load_codes(kb0); f[0].load(Wf, kb0, 0, lane); }
        stage();
        for (int kb = kb0; kb < kb1; ++kb) {
            v8bf af[RB][2][2];
#pragma unroll
            for (int b = 0; b < RB; ++b) c[b].operands(af[b], kb, K, kq);
            load_codes(kb + 1);
            f[1].load(Wf, kb, 1, lane);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int b = 0; b < RB; ++b) panel_products<NT, PL>(af[b][0], f[0], acc[b]);
            __builtin_amdgcn_sched_barrier(0);
            f[0].load(Wf, min(kb + 1, nkb - 1), 0, lane);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int b = 0; b < RB; ++b) panel_products<NT, PL>(af[b][1], f[1], acc[b]);
        }
    }
#pragma unroll
    for (int b = 0; b < RB; ++b) {
        const int r0 = (blk * RB + b) * 32;
        if (r0 >= rows) break;              // (uniform)
        if (b > 0) __syncthreads();
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int v = 0; v < 4; ++v) red[(wave * 32 + 16 * t + 4 * kq + v) * RP + 16 * nt + li] = acc[b][t][nt][v];
        __syncthreads();
        const int nrows = min(32, rows - r0);
        float* const out = (right ? a.Rp : a.Lp) + (size_t)r0 * R2P;
        // A thread takes GROUP rows of a column, so that an entry of X Gamma read from LDS serves as many products, and both halves of
        // the panel rows.  A thread per entry of them, with two LDS reads a product (which bound wide panels) and a division for the row /
        // this, lrqmm_gemm, 8 bits, us: rank 32 2000^3 43.2 / 41.2, 16384 x 100 x 252 27.1 / 23.9, rank 64 300^3 30.8 / 24.4, 4096^3 139 / 132,
        // 100 x 100352 x 100 245 / 158, 100352 x 100 x 100 127 / 112, rank 80 600 x 41152 x 252 228 / 188.  Four rows at two tiles: no better.
        constexpr int GROUP = NT <= 2 ? NT : 4;
        for (int e = tid; e < 32 / GROUP * RP; e += 512) {
            const int c = e % RP, i0 = e / RP * GROUP;
            if (c >= r) continue;
            float v[GROUP], z[GROUP];
#pragma unroll
            for (int i = 0; i < GROUP; ++i) {
                v[i] = 0.f;
#pragma unroll
                for (int w = 0; w < PANEL_WAVES; ++w) v[i] += red[(w * 32 + i0 + i) * RP + c];
                v[i] *= step[32 * b + i0 + i];
            }
            if (right) {
                auto z_of = [&](int u) {
                    const float* const p = &own[b][u * OWN + i0];
                    if constexpr (GROUP == 1) z[0] = *p;
                    else if constexpr (GROUP == 2) { const float2 t = *reinterpret_cast<const float2*>(p); z[0] = t.x; z[1] = t.y; }
                    else { const float4 t = *reinterpret_cast<const float4*>(p); z[0] = t.x; z[1] = t.y; z[2] = t.z; z[3] = t.w; }
                };
#pragma unroll 1                        // unrolled, its loads of X Gamma leave the loop over e and spill
                for (int u0 = 0; u0 < RP; u0 += 8) {       // rows u >= r of Zt are zero
#pragma unroll
                    for (int t = 0; t < 8; ++t) {
                        const float x = xg[c * (RP + 1) + u0 + t];
                        z_of(u0 + t);
#pragma unroll
                        for (int i = 0; i < GROUP; ++i) v[i] = fmaf(x, z[i], v[i]);
                    }
                }
                z_of(c);
#pragma unroll
                for (int i = 0; i < GROUP; ++i) z[i] *= a.Gam[c];
            } else {
#pragma unroll
                for (int i = 0; i < GROUP; ++i) z[i] = own[b][(i0 + i) * r + c];
            }
            float* const o = out + i0 * R2P + c;
            const int product = right ? 0 : r, factor = r - product;
#pragma unroll
            for (int i = 0; i < GROUP; ++i)
                if (i0 + i < nrows) {
                    o[i * R2P + product] = v[i];
                    o[i * R2P + factor] = z[i];
                }
        }
        const int pad = R2P - 2 * r;
        for (int e = tid; e < nrows * pad; e += 512) out[e / pad * R2P + 2 * r + e % pad] = 0.f;
    }
}

// The same for tall operands with short rows (K <= 640) of bytes and factors of at most 16 columns: all planes fit in LDS (three
// planes x 16 columns x Kp bfloat16), so workgroups are persistent -- two of eight waves per CU, the planes copied once -- and after
// the one barrier behind that copy the waves are on their own: a wave takes the 16-row tiles w, w + W, w + 2W, ... (W waves in the
// grid) and loads a tile's codes at once (NC 16-byte loads per lane, the whole row); the sixteen waves of a CU are at
// different points of that cycle, which keeps loads in flight while others compute.  blockIdx.z: 0 left panel, 1 right.
template <int PL, int NC>
__global__ __launch_bounds__(512, 4) void panels_rows_kernel(PanelArgs a) {
    extern __shared__ __align__(16) uint16_t wf[];        // [k block][plane][step][lane][8]; right: X Gamma behind it
    __shared__ float xg[16 * 17];
    const bool right = blockIdx.z == 1;
    const int rows = right ? a.N : a.M, K = a.K, r = a.r, R2P = a.R2P, nkb = pk_kblocks(K);
    const int ntiles = (rows + 15) >> 4;
    if ((int)blockIdx.x * 8 >= ntiles) return;            // no tile for any wave of this workgroup
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int li = lane & 15, kq = lane >> 4;
    const uint4* const src = reinterpret_cast<const uint4*>(right ? a.Vf : a.Wf);
    for (int p = threadIdx.x; p < nkb * 6 * 64; p += 512) reinterpret_cast<uint4*>(wf)[p] = src[p];
    if (right) stage_x_gamma(a, 16, xg, threadIdx.x, 512);
    __syncthreads();
    const int8_t* const codes = right ? a.codesB : a.codesA;
    const int nwaves = gridDim.x * 8, range = panel_range(nkb);
    const float scale = (right ? a.Gam : a.Sig)[min(li, r - 1)];
    for (int tile = blockIdx.x * 8 + wave; tile < ntiles; tile += nwaves) {
        // codes past K meet zero planes and rows past the end re-read the last row (never stored): clamped addresses, no masks
        uint4 ca[NC];
        const int8_t* ap = codes + (size_t)min(tile * 16 + li, rows - 1) * K;
#pragma unroll
        for (int c = 0; c < NC; ++c) ca[c] = load_codes16<true>(ap, K, 64 * c + 16 * kq);
        float step[4], us[4];       // (the epilogue's operands come beside the codes)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = min(tile * 16 + 4 * kq + v, rows - 1), col = min(li, r - 1);
            step[v] = (right ? a.sB : a.sA)[row];
            us[v] = right ? a.Zt[(size_t)col * rows + row] : a.U[(size_t)row * a.ldu + col];
        }
        __builtin_amdgcn_sched_barrier(0);
        v4f total = (v4f){0.f, 0.f, 0.f, 0.f}, acc = total;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if (c >= nkb) continue;             // (uniform)
            if (c > 0 && c % range == 0) {      // the sums of a range of their own, as in panels_kernel
                total += acc;
                acc = (v4f){0.f, 0.f, 0.f, 0.f};
            }
            if ((K & 15) && 64 * c + 64 > K) ca[c] = tail16(ca[c], max(0, 64 * c + 16 * kq - (K - 16)));     // uniform
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const v8bf af = h == 0 ? codes_to_bf16(ca[c].x, ca[c].y) : codes_to_bf16(ca[c].z, ca[c].w);
#pragma unroll
                for (int pl = 0; pl < PL; ++pl)
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        af, *reinterpret_cast<const v8bf*>(wf + ((c * 3 + pl) * 2 + h) * FACTOR_PIECE + lane * 8), acc, 0, 0, 0);
            }
        }
        total += acc;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = tile * 16 + 4 * kq + v;
            if (row >= rows) continue;
            float* const out = (right ? a.Rp : a.Lp) + (size_t)row * R2P;
            if (li < r) {
                float p = total[v] * step[v];
                if (right) {
#pragma unroll 1
                    for (int u = 0; u < r; ++u) p = fmaf(xg[li * 17 + u], a.Zt[(size_t)u * rows + row], p);
                }
                out[right ? li : r + li] = p;
                out[right ? r + li : li] = us[v] * scale;
            }
            if (2 * r + li < R2P) out[2 * r + li] = 0.f;
        }
    }
}

// The same for other tall operands: a wave takes 32 rows over the whole reduction, so its sums never leave its registers and no
// barrier stands between its codes and its panel rows; a workgroup of eight such waves shares the planes in LDS, two workgroups a CU, all
// k blocks at once where they fit, and otherwise tall_chunk of them at a time.  The sums of each eighth of the k blocks are added in
// order, as in panels_kernel: the same bits.  That one holds the registers of a CU with one workgroup, whose loads, sums through
// LDS and stores stand behind one another for every 64 rows.
//
// lrqmm_gemm, 8 bits, panels_kernel / this, us: 100352 x 64 rank 8 K = 1152 82.5 / 63.3, rank 24 K = 64 58.6 / 35.0, 576 78.9 / 55.8, 2304 162 / 126,
// rank 48 K = 576 99.8 / 82.9; 64 x 100352 rank 24 K = 576 112 / 79.0, rank 48 152 / 119 (few reads of Zt per row).  tall_panels picks.
constexpr int tall_chunk(int nt, int pl) { return (nt == 3 ? 60 : 72) / (2 * nt * pl); }       // k blocks of planes in LDS
template <int FMT, int NT, int PL>
__global__ __launch_bounds__(512, 4) void panels_tall_kernel(PanelArgs a) {
    constexpr int RP = NT * 16, PIECES = NT * PL * 2, CH = tall_chunk(NT, PL), AHEAD = NT == 1 ? 2 : 1;
    __shared__ __align__(16) uint16_t wf[CH * PIECES * FACTOR_PIECE];       // [k block][column tile][plane][step][lane][8]
    __shared__ float xg[RP * (RP + 1)];
    const bool right = (int)blockIdx.x < a.nbR;
    const int rows = right ? a.N : a.M, K = a.K, r = a.r, R2P = a.R2P, nkb = pk_kblocks(K);
    const int8_t* const codes = right ? a.codesB : a.codesA;
    const uint4* const src = reinterpret_cast<const uint4*>(right ? a.Vf : a.Wf);
    const float* const steps = right ? a.sB : a.sA;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int li = lane & 15, kq = lane >> 4;
    const int ngroups = (rows + 255) >> 8, range = panel_range(nkb);
    const int first = right ? blockIdx.x : blockIdx.x - a.nbR, stride = right ? a.nbR : gridDim.x - a.nbR;
    const bool once = nkb <= CH;
    auto stage = [&](int k0) {
        const int n = min(CH, nkb - k0) * PIECES * 64;
        for (int p = tid; p < n; p += 512) {
            const int piece = p >> 6, h = piece & 1, pl = (piece >> 1) % PL, bn = (piece >> 1) / PL;
            reinterpret_cast<uint4*>(wf)[p] = src[(size_t)(((k0 * NT + bn) * 3 + pl) * 2 + h) * 64 + (p & 63)];
        }
    };
    CodeBlock<FMT> c[AHEAD + 1];
    float step[2][4], us[2][4];
    auto begin = [&](int rb) {          // what a block of rows starts from, and (where it fits) what its panel rows need besides the products
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) c[i].load(codes, rb, rows, min(i, nkb - 1), K, nkb, li, kq);
        if (NT > 1) return;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = min(32 * rb + 16 * t + 4 * kq + v, rows - 1);
                step[t][v] = steps[row];
                if (!right) us[t][v] = a.U[(size_t)row * a.ldu + min(li, r - 1)];
            }
    };
    if (first >= ngroups) return;       // (uniform)
    begin(first * 8 + wave);
    if (right) stage_x_gamma(a, RP, xg, tid, 512);
    if (once) stage(0);
    __syncthreads();
    for (int g = first; g < ngroups; g += stride) {
        const int rb = g * 8 + wave;
        if (g != first) begin(rb);
        v4f total[2][NT], acc[2][NT];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) total[t][nt] = acc[t][nt] = (v4f){0.f, 0.f, 0.f, 0.f};
        auto add_range = [&] {
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) { total[t][nt] += acc[t][nt]; acc[t][nt] = (v4f){0.f, 0.f, 0.f, 0.f}; }
        };
        int left = range;
        for (int k0 = 0; k0 < nkb; k0 += CH) {
            if (!once) {
                __syncthreads();        // nobody reads the k blocks before
                stage(k0);
                __syncthreads();
            }
            const int k1 = min(nkb, k0 + CH);
            for (int kb = k0; kb < k1; ++kb) {
                c[AHEAD].load(codes, rb, rows, min(kb + AHEAD, nkb - 1), K, nkb, li, kq);
                __builtin_amdgcn_sched_barrier(0);
                if (left == 0) { add_range(); left = range; }       // (uniform)
                --left;
                v8bf af[2][2];
                c[0].operands(af, kb, K, kq);
                const uint16_t* const w = wf + (kb - k0) * PIECES * FACTOR_PIECE + lane * 8;
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                        for (int pl = 0; pl < PL; ++pl) {
                            const v8bf b = *reinterpret_cast<const v8bf*>(w + ((nt * PL + pl) * 2 + h) * FACTOR_PIECE);
#pragma unroll
                            for (int t = 0; t < 2; ++t) acc[t][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[h][t], b, acc[t][nt], 0, 0, 0);
                        }
#pragma unroll
                for (int i = 0; i < AHEAD; ++i) c[i] = c[i + 1];
            }
        }
        add_range();
        if (32 * rb >= rows) continue;          // (the barriers of the next group follow)
        const bool whole = 32 * rb + 32 <= rows;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int row0 = 32 * rb + 16 * t + 4 * kq;
            float p[NT][4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                if (NT > 1) step[t][v] = steps[min(row0 + v, rows - 1)];
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) p[nt][v] = total[t][nt][v] * step[t][v];
            }
            auto z_rows = [&](int u) {
                const float* const zt = a.Zt + (size_t)u * rows;
                return whole ? load4u(zt + row0) : load4_tail(zt, row0, rows);
            };
            if (right) {
                constexpr int BATCH = NT == 3 ? 2 : 4;
                for (int u0 = 0; u0 < r; u0 += BATCH) {
                    float4 z[BATCH];
#pragma unroll
                    for (int j = 0; j < BATCH; ++j) z[j] = z_rows(min(u0 + j, r - 1));
#pragma unroll
                    for (int j = 0; j < BATCH; ++j)
                        if (u0 + j < r) {
#pragma unroll
                            for (int nt = 0; nt < NT; ++nt) {
                                const float x = xg[(16 * nt + li) * (RP + 1) + u0 + j];
                                p[nt][0] = fmaf(x, z[j].x, p[nt][0]);
                                p[nt][1] = fmaf(x, z[j].y, p[nt][1]);
                                p[nt][2] = fmaf(x, z[j].z, p[nt][2]);
                                p[nt][3] = fmaf(x, z[j].w, p[nt][3]);
                            }
                        }
                }
            }
            float* const out = right ? a.Rp : a.Lp;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const int col = 16 * nt + li, cc = min(col, r - 1);
                float own[4];           // the columns that are not a product's
                if (right) {
                    const float4 z = z_rows(cc);
                    const float gam = a.Gam[cc];
                    own[0] = gam * z.x; own[1] = gam * z.y; own[2] = gam * z.z; own[3] = gam * z.w;
                } else {
                    const float sig = a.Sig[cc];
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        own[v] = (NT == 1 ? us[t][v] : a.U[(size_t)min(row0 + v, rows - 1) * a.ldu + cc]) * sig;
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    if (row0 + v >= rows) continue;
                    float* const o = out + (size_t)(row0 + v) * R2P;
                    if (col < r) {
                        o[right ? col : r + col] = p[nt][v];
                        o[right ? r + col : col] = own[v];
                    }
                    if (nt == 0 && 2 * r + li < R2P) o[2 * r + li] = 0.f;
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// T-type: partial[split][cols][LP] = R[i-range, :]^T . W[i-range, :]
// One workgroup per 64-column strip and range of rows (strips fastest, job a before job b); its 4 waves share the strip,
// interleave rows, and merge their accumulators through LDS.
// A lane's float4 holds columns c0+4c .. c0+4c+3; component t feeds M-tile t, so
// M-tile t covers the columns {c0 + 4 c + t}.  Likewise N-tile nt covers the W columns
// {NT c + nt}, so a lane's B operands are NT consecutive floats (one wide load).
// Loads run TUNR row groups ahead of the matrix cores (register double buffering).
// ---------------------------------------------------------------------------
// Any shape, stride and 4-byte alignment.  Columns: the lane whose four columns would cross the end of the row takes
// the row's last four instead (t_column) and stores only what lies at or beyond its own first column; lanes wholly
// past the end store nothing.  Rows: whole groups are loaded without a guard, the group that reaches past the chunk
// re-reads its last row with zeros for W.  (TINY, cols < 4: clamped scalar loads.)
struct TColumn {
    int kc;         // first column the lane loads
    int skip;       // components below this one are another lane's columns; 4 and more: the lane stores nothing
};
__device__ __forceinline__ TColumn t_column(int k, int cols) {
    const int kc = max(0, min(k, cols - 4));
    return {kc, k - kc};
}
// Four values of a row at the lane's columns (TINY: cols < 4).
template <bool TINY>
__device__ __forceinline__ float4 load_cols(const float* __restrict__ rowp, int kc, int cols) {
    return TINY ? load4_tail(rowp, kc, cols) : load4u(rowp + kc);
}
#define TUNR 4
template <int AXIS, bool TINY>
__device__ __forceinline__ void resid_mul_t_body(const PassJob& job, QuantParams q, int bx, int by,
                                                 float* __restrict__ const red) {
    if (job.run && *job.run == 0) return;               // (uniform)
    LRQ_PASS_JOB(job);
    constexpr int LP = 16;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int c = lane & 15, g = lane >> 4;
    const int c0 = bx * 64;
    const int kc = t_column(c0 + 4 * c, cols).kc;
    const int ib = by * chunk;
    const int ie = min(rows, ib + chunk);
    float4 lc = make_float4(0.f, 0.f, 0.f, 0.f), scol = lc;
    if (AXIS == 1) {
        lc = load_cols<TINY>(lam, kc, cols);
        scol = load_cols<TINY>(sc, kc, cols);
    }
    v4f acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = (v4f){0.f, 0.f, 0.f, 0.f};

    struct Frag {
        float4 x;
        float lr, sr, w;
    };
    // rows i0 + 16 u + g of the group, u < TUNR
    auto load_group = [&](int i0, Frag (&f)[TUNR]) {
        if (i0 + 16 * (TUNR - 1) + 4 <= ie) {
#pragma unroll
            for (int u = 0; u < TUNR; ++u) {
                const int i = i0 + 16 * u;      // wave-uniform
                f[u].x = load_cols<TINY>(X + (size_t)i * ldx + (size_t)g * ldx, kc, cols);
                if (AXIS == 0) {
                    f[u].lr = (lam + i)[g];
                    f[u].sr = (sc + i)[g];
                }
                f[u].w = (W + (size_t)i * LP)[g * LP + c];
            }
        } else {
#pragma unroll
            for (int u = 0; u < TUNR; ++u) {
                const int i = i0 + 16 * u + g, ii = min(i, ie - 1);
                f[u].x = load_cols<TINY>(X + (size_t)ii * ldx, kc, cols);
                if (AXIS == 0) {
                    f[u].lr = lam[ii];
                    f[u].sr = sc[ii];
                }
                const float wv = W[(size_t)ii * LP + c];
                f[u].w = i < ie ? wv : 0.f;
            }
        }
    };
    Frag fa[TUNR], fb[TUNR];
    const int istart = ib + wave * 4;
    auto step = [&](const Frag (&cur)[TUNR], Frag (&nxt)[TUNR], int i0) {
        if (i0 + 16 * TUNR < ie) load_group(i0 + 16 * TUNR, nxt);
#pragma unroll
        for (int u = 0; u < TUNR; ++u) {
            float4 l4 = lc, s4 = scol;
            if (AXIS == 0) {
                l4 = make_float4(cur[u].lr, cur[u].lr, cur[u].lr, cur[u].lr);
                s4 = make_float4(cur[u].sr, cur[u].sr, cur[u].sr, cur[u].sr);
            }
            const float res[4] = {quant_residual(cur[u].x.x, l4.x, s4.x, q), quant_residual(cur[u].x.y, l4.y, s4.y, q),
                                  quant_residual(cur[u].x.z, l4.z, s4.z, q), quant_residual(cur[u].x.w, l4.w, s4.w, q)};
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[t] = mfma16(res[t], cur[u].w, acc[t]);
        }
    };
    if (istart < ie) load_group(istart, fa);
    for (int i0 = istart; i0 < ie; i0 += 32 * TUNR) {       // two groups per round: the register sets swap roles
        step(fa, fb, i0);
        if (i0 + 16 * TUNR < ie) step(fb, fa, i0 + 16 * TUNR);
    }
    // merge the four waves (fixed order: deterministic)
    for (int wv = 0; wv < 4; ++wv) {
        if (wave == wv) {
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int cl = 16 * g + 4 * v;                      // local first column of D row 4g+v
                    const int skip = t_column(c0 + cl, cols).skip;      // component t: local column cl + t - skip
                    float* p = red + (cl + t - skip) * LP + c;
                    if (t >= skip) *p = (wv == 0) ? acc[t][v] : (*p + acc[t][v]);
                }
        }
        __syncthreads();
    }
    float* out = partial + (size_t)by * cols * LP;
    for (int idx = threadIdx.x; idx < 64 * LP / 4; idx += 256) {
        const int e = idx * 4;
        const int cl = e / LP, n = e % LP;
        if (c0 + cl < cols)
            *reinterpret_cast<float4*>(out + (size_t)(c0 + cl) * LP + n) =
                *reinterpret_cast<const float4*>(red + cl * LP + n);
    }
}

template <bool TINY>
__global__ __launch_bounds__(256) void resid_mul_t_kernel(PassJob a, PassJob b, int nb0, QuantParams q) {
    __shared__ __align__(16) float red[64 * 16];
    const int id = blockIdx.x;
    if (id < nb0) resid_mul_t_body<0, TINY>(a, q, id % a.nbx, id / a.nbx, red);
    else          resid_mul_t_body<1, TINY>(b, q, (id - nb0) % b.nbx, (id - nb0) / b.nbx, red);
}

// The T-type product on the bf16 matrix cores (see resid_mul_n_bf16_kernel for the plane
// arithmetic).  A wave takes 32 rows per step: lane group g loads rows base + 4e + g (e < 8),
// which are its 8 k-slots; both operands come straight from global memory in that order (a
// float4 of X and NT floats of W per row), so no LDS is needed before the final merge.  The row part of every
// address of a whole step is wave-uniform (scalar registers), the lane part a constant offset; the one step of a
// wave that reaches past the rows follows the loop.  FULL: whole column strips, whole 128-row steps of the workgroup.
// Measured against four strips per workgroup sharing W's planes in LDS (one plane split per workgroup instead of
// one per wave): alone equal (4096^2, 48 columns: 20 us), but with the other operand's pass on the chip 13.8 us per
// pass against 17.8 -- the LDS keeps the two from sharing a CU.
template <int NT, int AXIS, int PL, bool FULL, bool TINY>
__device__ __forceinline__ void resid_mul_t_bf16_body(const PassJob& job, QuantParams q, int bx, int by,
                                                      float* __restrict__ const red) {
    LRQ_PASS_JOB(job);
    constexpr int LP = NT * 16;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int c = lane & 15, g = lane >> 4;
    const int c0 = bx * 64;
    const int kc = FULL ? c0 + 4 * c : t_column(c0 + 4 * c, cols).kc;
    const int ib = by * chunk;
    const int ie = min(rows, ib + chunk);
    float lcol[4] = {0.f, 0.f, 0.f, 0.f}, scol[4] = {0.f, 0.f, 0.f, 0.f};
    if (AXIS == 1) {
        const float4 l4 = load_cols<TINY>(lam, kc, cols), s4 = load_cols<TINY>(sc, kc, cols);
        lcol[0] = l4.x; lcol[1] = l4.y; lcol[2] = l4.z; lcol[3] = l4.w;
        scol[0] = s4.x; scol[1] = s4.y; scol[2] = s4.z; scol[3] = s4.w;
    }
    v4f acc[4][NT];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[t][nt] = (v4f){0.f, 0.f, 0.f, 0.f};

    struct Group {
        float x[8][4];
        float lr[8], sr[8];
        float w[8][NT];
    };
    const ptrdiff_t xoff = (ptrdiff_t)g * ldx + (TINY ? 0 : kc);      // lane part of the addresses
    const int woff = g * LP + NT * c;
    auto load_group = [&](int i0, Group& f) {              // i0 wave-uniform, i0 + 32 <= ie
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float* xrow = X + (size_t)(i0 + 4 * e) * ldx;
            const float4 xv = TINY ? load4_tail(xrow + xoff, kc, cols) : load4u(xrow + xoff);
            f.x[e][0] = xv.x; f.x[e][1] = xv.y; f.x[e][2] = xv.z; f.x[e][3] = xv.w;
            if (AXIS == 0) {
                f.lr[e] = (lam + i0 + 4 * e)[g];
                f.sr[e] = (sc + i0 + 4 * e)[g];
            }
            const float* wrow = W + (size_t)(i0 + 4 * e) * LP;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) f.w[e][nt] = wrow[woff + nt];
        }
    };
    auto load_group_tail = [&](int i0, Group& f) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int i = i0 + 4 * e + g, ii = min(i, ie - 1);
            const float4 xv = load_cols<TINY>(X + (size_t)ii * ldx, kc, cols);
            f.x[e][0] = xv.x; f.x[e][1] = xv.y; f.x[e][2] = xv.z; f.x[e][3] = xv.w;
            if (AXIS == 0) {
                f.lr[e] = lam[ii];
                f.sr[e] = sc[ii];
            }
            const float* wp = W + (size_t)ii * LP + NT * c;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const float wv = wp[nt];
                f.w[e][nt] = i < ie ? wv : 0.f;
            }
        }
    };
    auto products = [&](const Group& cur) {
        Planes3 bp[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            float wv[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) wv[e] = cur.w[e][nt];
            bp[nt] = split_planes<PL>(wv);
        }
#pragma unroll
        for (int th = 0; th < 2; ++th) {        // two column components at a time: 2 NT independent chains
            Planes3 ap[2];
#pragma unroll
            for (int tt = 0; tt < 2; ++tt) {
                const int t = 2 * th + tt;
                float res[8];
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    res[e] = quant_residual(cur.x[e][t], AXIS == 0 ? cur.lr[e] : lcol[t],
                                            AXIS == 0 ? cur.sr[e] : scol[t], q);
                ap[tt] = split_planes<PL>(res);
            }
            v4f (&a2)[2][NT] = *reinterpret_cast<v4f (*)[2][NT]>(&acc[2 * th]);
            mfma_planes<2, NT, PL>(ap, bp, a2);
        }
    };
    // whole steps of this wave: i0 = ib + 32 wave + 128 n with i0 + 32 <= ie
    int i0 = ib + 32 * wave;
    {
        Group cur, nxt;
        if (FULL || i0 + 32 <= ie) load_group(i0, cur);
        for (; FULL ? i0 < ie : i0 + 32 <= ie; i0 += 128) {
            load_group((FULL ? i0 + 128 < ie : i0 + 160 <= ie) ? i0 + 128 : i0, nxt);     // last whole step: re-reads its own rows
            products(cur);
            cur = nxt;
        }
    }
    if (!FULL && i0 < ie) {
        Group last;
        load_group_tail(i0, last);
        products(last);
    }
    // merge the four waves (fixed order: deterministic)
    for (int wv = 0; wv < 4; ++wv) {
        if (wave == wv) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int cl = 16 * g + 4 * v;                      // local first column of D row 4g+v
                const int skip = FULL ? 0 : t_column(c0 + cl, cols).skip;      // component t: local column cl + t - skip
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    if (t >= skip) {
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt) {
                            float* p = red + (cl + t - skip) * LP + NT * c + nt;
                            *p = (wv == 0) ? acc[t][nt][v] : (*p + acc[t][nt][v]);
                        }
                    }
            }
        }
        __syncthreads();
    }
    float* out = partial + (size_t)by * cols * LP;
    for (int idx = threadIdx.x; idx < 64 * LP / 4; idx += 256) {
        const int e = idx * 4;
        const int cl = e / LP, n = e % LP;
        if (FULL || c0 + cl < cols)
            *reinterpret_cast<float4*>(out + (size_t)(c0 + cl) * LP + n) =
                *reinterpret_cast<const float4*>(red + cl * LP + n);
    }
}

template <int NT, int PL, bool FULL, bool TINY = false>
__global__ __launch_bounds__(256, 2) void resid_mul_t_bf16_kernel(PassJob a, PassJob b, int nb0, QuantParams q) {
    __shared__ __align__(16) float red[64 * NT * 16];
    const int id = blockIdx.x;
    if (id < nb0) resid_mul_t_bf16_body<NT, 0, PL, FULL, TINY>(a, q, id % a.nbx, id / a.nbx, red);
    else          resid_mul_t_bf16_body<NT, 1, PL, FULL, TINY>(b, q, (id - nb0) % b.nbx, (id - nb0) / b.nbx, red);
}

// One operand alone (two-chain calls, lrqmm_rsvd) at 48 columns: holding both forms costs the kernel above 176 registers,
// two waves per SIMD; one form takes 154 to 164, three.  A launch is about 512 workgroups of one wave per SIMD, often
// more (ceil), and those beyond two per CU ran as a second round: 7168^3 (560 workgroups per pass, 40 columns) 1.172 ->
// 1.159 ms per call, 5120^3 0.637 -> 0.630, 10240^3 2.37 -> 2.35; 8192^3 (512 workgroups) 1.490 -> 1.499.  At 32
// columns at least three waves fit in either form, at 64 and 80 two.
template <int NT, int AXIS, int PL, bool FULL>
__global__ __launch_bounds__(256, 2) void resid_mul_t_bf16_one_kernel(PassJob a, QuantParams q) {
    __shared__ __align__(16) float red[64 * NT * 16];
    resid_mul_t_bf16_body<NT, AXIS, PL, FULL, false>(a, q, (int)blockIdx.x % a.nbx, (int)blockIdx.x / a.nbx, red);
}

// ---------------------------------------------------------------------------
// launch plans and dispatch
// ---------------------------------------------------------------------------
// Ranges of the reduction: about `target` workgroups, at least `depth` reduction elements each.
static int pick_splits(int blocks_one_split, int reduce_len, int depth, int target, int limit) {
    const int want = ceil_div(target, max(1, blocks_one_split));
    return max(1, min(want, min(max(1, reduce_len / depth), limit)));
}

// Sketches of 64 and 80 columns: 128-row workgroups of eight waves where they fill the chip (half the plane splits of W
// per row), in 32-deep chunks without the code output (24 KB of LDS per buffer: two operands' workgroups share a
// CU).  Measured per pass with two passes on the chip, 80 columns, eight waves / four: 4096^2 18.1 / 22.9 us; 8192^2 83
// / 104; 16384^2 320 / 390; with the code output (64-deep) 16384^2 400 / 438.  Up to 48 columns the four-wave kernel
// is as fast or faster (8192^2, 48 columns: 75 / 76; 4096^2: 15.0 / 15.2; 1537 x 2311, 32 columns: 7.3 / 5.3).
static bool pass_n_wide(int rows, int cols, int LP) {
    return LP >= 64 && (long long)ceil_div(rows, 128) * min(MAX_SPLITS, max(1, cols / 128)) >= 256;
}

// (an empty reduction has no ranges: splits = 0)
// Up to 1024 rows ranges of one chunk, down to 64 elements: such a pass is the load latency of its chunks, one after the
// other.  Two chunks and more / this, us per call: 200^3 l = 10 87.7 / 83.5, 256^3 l = 8 50.8 / 48.2, 512^3 l = 24 130.4 /
// 127.9, 1000^3 l = 10 113.1 / 108.2; beyond 2000^3 l = 10 157.0 / 163.4.  Up to MAX_SPLITS_FEW ranges there: with eight a 512 x 4096
// operand was 64 workgroups of eight chunks each (12.2 us a pass, 24 columns).  Layer calls, 8 bits, one power iteration, 8 / 16 / 32 ranges,
// us: 512 x 4096 x 4096 l = 24 167 / 158 / 158, 40 231 / 224 / 223, 80 431 / 422 / 423; 128 x 4096 x 4096 l = 80 416 / 406 / 403; 1024 x 4096 x 4096
// l = 24 186 / 177 / 179, 80 454 / 447 / 451; 256 x 512 x 16384 l = 24 291 / 254 / 238, 80 659 / 611 / 589; 1000^3 equal.
PassPlan plan_pass_n(int rows, int cols, int LP) {
    const int unit = LP == 16 ? KCHUNK : 64;        // chunk depth of the kernel
    PassPlan p;
    int s = pick_splits(ceil_div(rows, pass_n_wide(rows, cols, LP) ? 128 : 64), cols, rows <= 1024 ? 64 : 2 * unit, 512, rows <= 1024 ? MAX_SPLITS_FEW : MAX_SPLITS);
    p.chunk = max(1, ceil_div(ceil_div(cols, s), unit)) * unit;
    p.splits = ceil_div(cols, p.chunk);
    return p;
}

int codes_splits(int rows, int K) {
    const int s = pick_splits(ceil_div(rows, 64), K, 4 * KCHUNK, 512, MAX_SPLITS);
    return ceil_div(K, max(1, ceil_div(ceil_div(K, s), KCHUNK)) * KCHUNK);
}

// Few column strips: many row chunks, of 32 rows and more with one tile of sketch columns, of 128 with more.  128 / 32, us
// per call: l = 10 200^3 87.7 / 83.3, 1000^3 113.1 / 111.7, 2000^3 157.0 / 153.5; l = 24 512^3 130.4 / 136.8, 1537 x 1021 x
// 2311 203.6 / 213.2.
PassPlan plan_pass_t(int rows, int cols, int LP) {
    PassPlan p;
    const int s = pick_splits(ceil_div(cols, 64), rows, LP == 16 ? 32 : 128, 512, MAX_SPLITS_T);
    // (a multiple of the 128 rows a workgroup takes per step when there are enough rows)
    const int unit = rows >= 512 * s ? 128 : 32;
    p.chunk = max(1, ceil_div(ceil_div(rows, s), unit)) * unit;
    p.splits = ceil_div(rows, p.chunk);
    return p;
}

// At least the rows of partial results (rows times ranges) of a plan of pick_splits at up to n rows in blocks of `block`:
// ceil(target / blocks) ranges of at most block rows a block.  Does not fall when an argument grows (the plans themselves do:
// 512 blocks make one range, 511 two).
static size_t most_partial_rows(int n, int block, int reduce_len, int depth, int target, int limit) {
    return min((size_t)n * min(limit, max(1, reduce_len / depth)), (size_t)n + (size_t)block * target);
}

size_t pass_partial_floats(int rows, int cols, int LP) {
    const PassPlan pn = plan_pass_n(rows, cols, LP), pt = plan_pass_t(rows, cols, LP);
    const int unit = LP == 16 ? KCHUNK : 64, block = LP >= 64 ? 128 : 64;
    size_t part = LP * max(most_partial_rows(rows, block, cols, 2 * unit, 512, MAX_SPLITS),
                           most_partial_rows(min(rows, 1024), block, cols, 64, 512, MAX_SPLITS_FEW));
    part = max(part, LP * most_partial_rows(cols, 64, rows, 128, 512, MAX_SPLITS_T));
    part = max(part, 16 * most_partial_rows(cols, 64, rows, 32, 512, MAX_SPLITS_T));
    part = max(part, (size_t)LP * 4096);        // (pass_full_ranges: up to 256 workgroups of 16 results)
    return max(part, LP * max((size_t)pn.splits * rows, (size_t)pt.splits * cols));
}

// The jobs of one launch: at most one with scales by row and one with scales by column.  Workgroup shape and plan of an
// operand depend on its own sizes; a launch has one workgroup shape, so a pair takes the wide one only when both do.
namespace {
struct PassPair {
    PassJob job[2];
    int nb[2];
};
PassPair make_pair(const PassOperand* op, int nop, bool t_type, int rows_per_wg) {
    PassPair p = {};
    for (int i = 0; i < nop; ++i) {
        const PassOperand& o = op[i];
        const PassPlan& plan = t_type ? o.pt : o.pn;
        PassJob& j = p.job[o.axis];
        j.X = o.X; j.lam = o.lam; j.sc = o.s; j.W = t_type ? o.Y : o.W; j.partial = o.partial;
        j.ldx = o.ldx; j.rows = o.rows; j.cols = o.cols; j.chunk = plan.chunk;
        j.nbx = t_type ? ceil_div(o.cols, 64) : ceil_div(o.rows, rows_per_wg);
        j.qo = {o.amax, o.lam, o.s, o.codes};
        j.run = o.run;
        p.nb[o.axis] = j.nbx * plan.splits;
    }
    for (int i = 0; i < 2; ++i) if (p.job[i].nbx == 0) p.job[i].nbx = 1;        // (an absent job: never indexed)
    return p;
}
}  // namespace
#define LRQ_PAIR_ARGS(P, THREADS) dim3((P).nb[0] + (P).nb[1]), dim3(THREADS), 0, st, (P).job[0], (P).job[1], (P).nb[0], q

// Sketches of up to 16 columns keep the float32 matrix-core kernels in float32 precision (one tile of W columns: the
// matrix cores are nowhere near busy and splitting operands into planes only adds work; the
// conv-shaped workload with l = 8 measures 0.37 ms against 0.39 ms), except in the quantizing pass, which has no float32
// form; wider ones use the bf16 kernels.
template <int NT, int PL, int QOUT>
static int dispatch_n(const PassOperand* op, int nop, QuantParams q, hipStream_t st) {
    bool wide = NT >= 4, full = true;
    for (int i = 0; i < nop; ++i) wide = wide && pass_n_wide(op[i].rows, op[i].cols, 16 * NT);
    for (int i = 0; i < nop; ++i) full = full && op[i].cols % 64 == 0 && (!QOUT || op[i].rows % (wide ? 128 : 64) == 0);
    const PassPair p = make_pair(op, nop, false, wide ? 128 : 64);
    if constexpr (NT >= 4) {
        constexpr int KC = QOUT ? 64 : 32;
        if (wide && full) hipLaunchKernelGGL((resid_mul_n_bf16_kernel<NT, PL, QOUT, 8, KC, true>), LRQ_PAIR_ARGS(p, 512));
        else if (wide)    hipLaunchKernelGGL((resid_mul_n_bf16_kernel<NT, PL, QOUT, 8, KC, false>), LRQ_PAIR_ARGS(p, 512));
    }
    if (!wide && full) hipLaunchKernelGGL((resid_mul_n_bf16_kernel<NT, PL, QOUT, 4, 64, true>), LRQ_PAIR_ARGS(p, 256));
    else if (!wide)    hipLaunchKernelGGL((resid_mul_n_bf16_kernel<NT, PL, QOUT, 4, 64, false>), LRQ_PAIR_ARGS(p, 256));
    LRQ_CHECK_LAUNCH();
    return LRQMM_OK;
}
template <int NT, int PL>
static int dispatch_t(const PassOperand* op, int nop, QuantParams q, hipStream_t st) {
    const PassPair p = make_pair(op, nop, true, 0);
    bool full = true, tiny = false;
    for (int i = 0; i < nop; ++i) {
        full = full && op[i].cols % 64 == 0 && op[i].rows % 128 == 0 && op[i].pt.chunk % 128 == 0;
        tiny = tiny || op[i].cols < 4;
    }
    if constexpr (NT == 1) {        // (fewer than four columns leave room for no wider sketch)
        if (tiny) hipLaunchKernelGGL((resid_mul_t_bf16_kernel<NT, PL, false, true>), LRQ_PAIR_ARGS(p, 256));
    }
    if constexpr (NT == 3) {
        if (nop == 1) {
            const int axis = op[0].axis;
            const dim3 grid(p.nb[axis]);
#define LRQ_T1(AX, FL) hipLaunchKernelGGL((resid_mul_t_bf16_one_kernel<NT, AX, PL, FL>), grid, dim3(256), 0, st, p.job[AX], q)
            if (axis == 0) { if (full) LRQ_T1(0, true); else LRQ_T1(0, false); }
            else           { if (full) LRQ_T1(1, true); else LRQ_T1(1, false); }
#undef LRQ_T1
            LRQ_CHECK_LAUNCH();
            return LRQMM_OK;
        }
    }
    if (!tiny && full) hipLaunchKernelGGL((resid_mul_t_bf16_kernel<NT, PL, true>), LRQ_PAIR_ARGS(p, 256));
    else if (!tiny)    hipLaunchKernelGGL((resid_mul_t_bf16_kernel<NT, PL, false>), LRQ_PAIR_ARGS(p, 256));
    LRQ_CHECK_LAUNCH();
    return LRQMM_OK;
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

// One call of F<NT, PL> for the sketch width and the number of planes.
#define LRQ_NT_PL(F, ...)                                                              \
    do {                                                                               \
        if (planes == 2)      NT_SWITCH(LP / 16, return (F<NT_, 2 __VA_ARGS__))        \
        else if (planes == 1) NT_SWITCH(LP / 16, return (F<NT_, 1 __VA_ARGS__))        \
        else                  NT_SWITCH(LP / 16, return (F<NT_, 3 __VA_ARGS__))        \
    } while (0)

int launch_resid_mul_n(const PassOperand* op, int nop, QuantParams q, int LP, bool quantize, hipStream_t st, int planes, int packed) {
    if (quantize && packed == PK6) LRQ_NT_PL(dispatch_n, , PK6>(op, nop, q, st));
    if (quantize && packed == PK8) LRQ_NT_PL(dispatch_n, , PK8>(op, nop, q, st));
    if (quantize) {     // rows of bytes: beside the one-read kernel alone, whose sketches have 16 columns
        if (LP != 16) return LRQMM_ERR_UNSUPPORTED;
        if (planes == 1) return dispatch_n<1, 1, QOUT_BYTES>(op, nop, q, st);
        if (planes == 2) return dispatch_n<1, 2, QOUT_BYTES>(op, nop, q, st);
        return dispatch_n<1, 3, QOUT_BYTES>(op, nop, q, st);
    }
    if (LP == 16 && planes == 3) {
        const PassPair p = make_pair(op, nop, false, 64);
        hipLaunchKernelGGL(resid_mul_n_kernel, LRQ_PAIR_ARGS(p, 256));
        LRQ_CHECK_LAUNCH();
        return LRQMM_OK;
    }
    LRQ_NT_PL(dispatch_n, , QOUT_NONE>(op, nop, q, st));
    return LRQMM_ERR_UNSUPPORTED;
}

static inline bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

bool quant_sketch_rows_usable(const float* X, int ldx, int rows, int cols, int LP, const int8_t* codes) {
    // (rows of up to 576 columns: beyond that the two register sets of a tile no longer fit 128 registers)
    return rows > 0 && LP == 16 && cols >= 16 && cols % 16 == 0 && cols <= LRQ_QSR_MAX_COLS && ldx % 4 == 0 && aligned16(X) &&
           ((uintptr_t)codes & 3) == 0;
}

int quant_sketch_rows_blocks(int rows) { return min(ceil_div(rows, 16), LRQ_QSR_MAX_BLOCKS); }

int launch_quant_sketch_rows(const float* X, int ldx, int rows, int cols, QuantParams q, const float* W, int LP,
                             float* Y, double* gpart, float* amax, float* lam_out, float* s_out, int8_t* codes,
                             hipStream_t st) {
    if (!quant_sketch_rows_usable(X, ldx, rows, cols, LP, codes)) return LRQMM_ERR_UNSUPPORTED;
    // persistent workgroups, each with a run of 16-row tiles; their number does not depend on the device, so
    // neither does the order in which the Gram matrix is summed (two per compute unit on a 256-CU chip)
    dim3 grid(quant_sketch_rows_blocks(rows));
    const size_t lds = (size_t)16 * (cols + ((68 - (cols & 63)) & 63)) * sizeof(float);
#define LRQ_QSR(NSV) case NSV: hipLaunchKernelGGL((quant_sketch_rows_kernel<NSV>), grid, dim3(512), lds, st, X, ldx, rows, cols, q, W, Y, gpart, amax, lam_out, s_out, codes); break
    switch (ceil_div(cols, 32)) {
        LRQ_QSR(1); LRQ_QSR(2); LRQ_QSR(3); LRQ_QSR(4); LRQ_QSR(5); LRQ_QSR(6); LRQ_QSR(7); LRQ_QSR(8); LRQ_QSR(9); LRQ_QSR(10);
        LRQ_QSR(11); LRQ_QSR(12); LRQ_QSR(13); LRQ_QSR(14); LRQ_QSR(15); LRQ_QSR(16); LRQ_QSR(17); LRQ_QSR(18);
        default: return LRQMM_ERR_UNSUPPORTED;
    }
#undef LRQ_QSR
    LRQ_CHECK_LAUNCH();
    return LRQMM_OK;
}

int launch_resid_mul_t(const PassOperand* op, int nop, QuantParams q, int LP, hipStream_t st, int planes) {
    if (LP == 16 && planes == 3) {
        const PassPair p = make_pair(op, nop, true, 0);
        bool tiny = false;
        for (int i = 0; i < nop; ++i) tiny = tiny || op[i].cols < 4;
        if (tiny) hipLaunchKernelGGL((resid_mul_t_kernel<true>), LRQ_PAIR_ARGS(p, 256));
        else      hipLaunchKernelGGL((resid_mul_t_kernel<false>), LRQ_PAIR_ARGS(p, 256));
        LRQ_CHECK_LAUNCH();
        return LRQMM_OK;
    }
    LRQ_NT_PL(dispatch_t, >(op, nop, q, st));
    return LRQMM_ERR_UNSUPPORTED;
}

// Where a workgroup's 256 rows leave CUs idle or with one workgroup, the copies of the planes into LDS, which nothing covers then, make
// panels_tall_kernel the slower form, the more so the more chunks of planes there are.  Of tall left panels it is the slower one up to more
// rows when the right operand has enough of them for whole workgroups, whose waves then each form 32 right panel rows, the longest
// part of such a launch.  lrqmm_gemm, 8 bits, panels_kernel / panels_tall_kernel, us, M x N:
//   rank 8    41152 x 600 K = 1152 97.9 / 99.2, 49152 x 64 48.5 / 41.7, 50000 x 600 133 / 128
//   rank 24   32768 x 64 K = 252 29.8 / 28.5, 576 36.8 / 38.6, 49152 x 64 46.8 / 42.9, 1152 59.2 / 56.3; 50000 x 300 K = 100 89.3 / 85.4
//   rank 32   41152 x 600 K = 252 104 / 112, 50000 x 600 141 / 145, 576 160 / 165, 65536 x 600 172 / 172, 131072 x 600 357 / 333
//   rank 40   57344 x 128 K = 100 59.0 / 54.4; rank 48 57344 x 64 K = 252 54.5 / 56.7, 65536 x 600 137 / 150, 98304 x 200 126 / 123,
//             98304 x 600 222 / 229, 131072 x 600 296 / 288
//   right     64 x 32768 rank 24 K = 252 39.6 / 35.9, 1152 56.0 / 56.3, 2304 77.0 / 82.4, rank 48 K = 252 54.8 / 60.1; 64 x 49152 rank 48 K = 576
//             83.6 / 81.2, 2304 133 / 147, 64 x 65536 159 / 157
static bool tall_panels(int M, int N, int nkb, int nt, int planes) {
    if (nt > 3) return false;
    const int chunks = ceil_div(nkb, tall_chunk(nt, planes));
    if (N >= 49152) return nt < 3 || chunks <= 6 || N >= 65536;
    if (N >= 32768) return nt < 3 && chunks <= 3;
    if (nt == 1) return M >= 65536 || (M >= 49152 && chunks <= 12);
    if (nt == 2) return M >= 65536 || (M >= 49152 && (N <= 128 || nkb <= 2)) || (M >= 32768 && N <= 128 && chunks == 1);
    return M >= 98304 || (M >= 57344 && N <= 128 && chunks == 1);
}

int launch_panels(const PanelArgs& in, int RP, int planes, int packed, hipStream_t st) {
    PanelArgs a = in;
    const int most = max(a.M, a.N), nkb = pk_kblocks(a.K);
    if (packed == PK_NONE && RP == 16 && a.K >= 16 && a.K <= 640 && most >= PANEL_ROWS_MIN) {
        int dev = 0, cus = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
            return LRQMM_ERR_HIP;
        const dim3 grid(min(ceil_div(ceil_div(most, 16), 8), 2 * cus), 1, 2);
        const size_t lds = (size_t)nkb * 6 * FACTOR_PIECE * sizeof(uint16_t);
#define LRQ_PR(PLV, NCV) hipLaunchKernelGGL((panels_rows_kernel<PLV, NCV>), grid, dim3(512), lds, st, a)
#define LRQ_PR_NC(PLV) do { if (nkb <= 2) LRQ_PR(PLV, 2); else if (nkb <= 4) LRQ_PR(PLV, 4); else if (nkb <= 6) LRQ_PR(PLV, 6); \
        else if (nkb <= 8) LRQ_PR(PLV, 8); else LRQ_PR(PLV, 10); } while (0)
        if (planes == 2) LRQ_PR_NC(2); else if (planes == 1) LRQ_PR_NC(1); else LRQ_PR_NC(3);
#undef LRQ_PR_NC
#undef LRQ_PR
        LRQ_CHECK_LAUNCH();
        return LRQMM_OK;
    }
    if (tall_panels(a.M, a.N, nkb, RP / 16, planes)) {
        int dev = 0, cus = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
            return LRQMM_ERR_HIP;
        a.nbR = min(ceil_div(a.N, 256), 2 * cus);
        const dim3 grid(a.nbR + min(ceil_div(a.M, 256), 2 * cus));
#define LRQ_PT(FMT, PLV)                                                                                                    \
    do {                                                                                                                    \
        if (RP == 16)      hipLaunchKernelGGL((panels_tall_kernel<FMT, 1, PLV>), grid, dim3(512), 0, st, a);                \
        else if (RP == 32) hipLaunchKernelGGL((panels_tall_kernel<FMT, 2, PLV>), grid, dim3(512), 0, st, a);                \
        else               hipLaunchKernelGGL((panels_tall_kernel<FMT, 3, PLV>), grid, dim3(512), 0, st, a);                \
    } while (0)
#define LRQ_PT_PL(FMT) do { if (planes == 2) LRQ_PT(FMT, 2); else if (planes == 1) LRQ_PT(FMT, 1); else LRQ_PT(FMT, 3); } while (0)
        if (packed == PK6)      LRQ_PT_PL(PK6);
        else if (packed == PK8) LRQ_PT_PL(PK8);
        else                    LRQ_PT_PL(PK_NONE);
#undef LRQ_PT_PL
#undef LRQ_PT
        LRQ_CHECK_LAUNCH();
        return LRQMM_OK;
    }
    // 64 rows a workgroup: half the reads of the planes.  From 65 columns on the sums of 64 rows no longer fit in the registers beside
    // them (lrqmm_gemm, 8 bits, 64 / 32 rows, us: 8192^2 x 1024 rank 72 283.8 / 272.7, 80 288.1 / 277.2, 16384 x 4096 x 2048 rank 72 363.4 / 346.7).
    const bool two = RP <= 64 && ceil_div(a.M, 64) + ceil_div(a.N, 64) >= PANEL_TWO_MIN;
    const int block = two ? 64 : 32;
    a.nbR = ceil_div(a.N, block);
    const dim3 grid(a.nbR + ceil_div(a.M, block));
#define LRQ_PK(FMT, PLV)                                                                                                       \
    do {                                                                                                                       \
        if (two) { NT_SWITCH(RP / 16, hipLaunchKernelGGL((panels_kernel<FMT, NT_, PLV, NT_ < 5 ? 2 : 1>), grid, dim3(512), 0, st, a)); } \
        else { NT_SWITCH(RP / 16, hipLaunchKernelGGL((panels_kernel<FMT, NT_, PLV, 1>), grid, dim3(512), 0, st, a)); }     \
    } while (0)
#define LRQ_PK_PL(FMT) do { if (planes == 2) { LRQ_PK(FMT, 2); } else if (planes == 1) { LRQ_PK(FMT, 1); } else { LRQ_PK(FMT, 3); } } while (0)
    if (packed == PK6)      LRQ_PK_PL(PK6);
    else if (packed == PK8) LRQ_PK_PL(PK8);
    else                    LRQ_PK_PL(PK_NONE);
#undef LRQ_PK_PL
#undef LRQ_PK
    LRQ_CHECK_LAUNCH();
    return LRQMM_OK;
}
