// Symmetric absmax quantization (paper: Background 2.2 Eq. (quantA); floor variant
// Methodology Eq. (get_ra2); Algorithm 2, quantization step).  HBM-streaming kernels: each
// input element is read from HBM once (the second touch of a row/tile hits L2).
#include "sketch.h"

// One wavefront per row: absmax by wave reduction, then codes with 4-byte packed stores.
// Second quantization level (complete residual compensation, Eq. (gemm_r_split)): when amax0 is
// given, the value that is quantized is the residual fl32(x - code0 * s0) of the first level, whose
// scales come from amax0 (the first level's maxima of the same groups).
__device__ __forceinline__ float4 first_level_residual(float4 v, float lam0, float s0, const QuantParams& q) {
    return make_float4(quant_residual(v.x, lam0, s0, q), quant_residual(v.y, lam0, s0, q),
                       quant_residual(v.z, lam0, s0, q), quant_residual(v.w, lam0, s0, q));
}

// Row kernels, any stride and alignment: the lane whose four columns would cross the end of the row takes the row's last
// four instead -- a maximum does not mind seeing a value twice, and two lanes then write the same codes -- so loads
// are 16 bytes and stores 4 bytes wide throughout (TINY, fewer than four columns: single elements).
__device__ __forceinline__ uint32_t pack_codes(float4 v, float lam, const QuantParams& q) {
    const int c0 = (int)quant_code(v.x, lam, q), c1 = (int)quant_code(v.y, lam, q);
    const int c2 = (int)quant_code(v.z, lam, q), c3 = (int)quant_code(v.w, lam, q);
    return (uint32_t)(c0 & 0xff) | ((uint32_t)(c1 & 0xff) << 8) | ((uint32_t)(c2 & 0xff) << 16) | ((uint32_t)(c3 & 0xff) << 24);
}
template <bool TINY>
__device__ __forceinline__ float4 load_quad(const float* __restrict__ xp, int k, int cols) {
    return TINY ? load4_tail(xp, k, cols) : load4u(xp + min(k, cols - 4));
}
// Codes of columns k .. k+3 (k < cols).
template <bool TINY>
__device__ __forceinline__ void store_quad(int8_t* __restrict__ cp, int k, int cols, uint32_t p) {
    if (TINY) {
        for (int t = 0; t < 4 && k + t < cols; ++t) cp[k + t] = (int8_t)(p >> (8 * t));
    } else {
        __builtin_memcpy(cp + min(k, cols - 4), &p, 4);
    }
}

// mode (all row kernels): ROWS_FULL computes amax and codes; ROWS_AMAX_ONLY stops after amax;
// ROWS_GIVEN_AMAX reads amax[row] (written by an earlier launch) instead of the row's own maximum.
enum { ROWS_FULL = 0, ROWS_AMAX_ONLY = 1, ROWS_GIVEN_AMAX = 2 };
template <bool TINY>
__global__ __launch_bounds__(256) void quant_rows_kernel(const float* __restrict__ X, int ldx, int rows,
                                                         int cols, QuantParams q,
                                                         int8_t* __restrict__ codes,
                                                         float* __restrict__ amax, int mode,
                                                         const float* __restrict__ amax0) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + wave;
    if (row >= rows) return;
    const float* xp = X + (size_t)row * ldx;
    float lam0 = 0.f, s0 = 0.f;
    if (amax0) make_scales(amax0[row], q.qmaxf, lam0, s0);
    float m = 0.0f;
    if (mode == ROWS_GIVEN_AMAX) {
        m = amax[row];
    } else {
        for (int k = lane * 4; k < cols; k += 256) {
            float4 v = load_quad<TINY>(xp, k, cols);
            if (amax0) v = first_level_residual(v, lam0, s0, q);
            m = fmaxf(fmaxf(m, fabsf(v.x)), fmaxf(fabsf(v.y), fmaxf(fabsf(v.z), fabsf(v.w))));
        }
        m = wave_max(m);
        if (lane == 0) amax[row] = m;
        if (mode == ROWS_AMAX_ONLY) return;
    }
    float lam, s;
    make_scales(m, q.qmaxf, lam, s);
    int8_t* cp = codes + (size_t)row * cols;
    for (int k = lane * 4; k < cols; k += 256) {
        float4 v = load_quad<TINY>(xp, k, cols);
        if (amax0) v = first_level_residual(v, lam0, s0, q);
        store_quad<TINY>(cp, k, cols, pack_codes(v, lam, q));
    }
}

// Single-read variant: the row is kept in registers between the absmax reduction and the
// code computation (NV float4 per thread, NV <= 16), so A is fetched from HBM once.  TPR threads
// cooperate on a row: 64 (one wavefront, cols <= 4096) or 256 (a workgroup, cols <= 16384).
template <bool TINY, int TPR, int NV>
__global__ __launch_bounds__(256) void quant_rows_cached_kernel(const float* __restrict__ X, int ldx, int rows,
                                                                int cols, QuantParams q,
                                                                int8_t* __restrict__ codes,
                                                                float* __restrict__ amax, int mode,
                                                                const float* __restrict__ amax0) {
    __shared__ float wmax[4];
    const int t = threadIdx.x % TPR;
    const int row = blockIdx.x * (256 / TPR) + threadIdx.x / TPR;
    const bool row_ok = row < rows;
    const float* xp = X + (size_t)(row_ok ? row : 0) * ldx;
    float4 v[NV];
    float m = 0.0f;
    float lam0 = 0.f, s0 = 0.f;
    if (amax0) make_scales(amax0[row_ok ? row : 0], q.qmaxf, lam0, s0);
#pragma unroll
    for (int u = 0; u < NV; ++u) {
        const int k = (t + TPR * u) * 4;
        v[u] = load_quad<TINY>(xp, k, cols);
        if (amax0) v[u] = first_level_residual(v[u], lam0, s0, q);     // (zeros past the end of a tiny row stay zeros)
        m = fmaxf(fmaxf(m, fabsf(v[u].x)), fmaxf(fabsf(v[u].y), fmaxf(fabsf(v[u].z), fabsf(v[u].w))));
    }
    m = wave_max(m);
    if (TPR == 256) {
        if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = m;
        __syncthreads();
        m = fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]));
    }
    if (!row_ok) return;
    if (mode == ROWS_GIVEN_AMAX) m = amax[row];
    else if (t == 0) amax[row] = m;
    if (mode == ROWS_AMAX_ONLY) return;
    float lam, s;
    make_scales(m, q.qmaxf, lam, s);
    int8_t* cp = codes + (size_t)row * cols;
#pragma unroll
    for (int u = 0; u < NV; ++u) {
        const int k = (t + TPR * u) * 4;
        if (k >= cols) continue;
        store_quad<TINY>(cp, k, cols, pack_codes(v[u], lam, q));
    }
}

__global__ void fill_u32_kernel(uint32_t* p, int n, uint32_t v, uint32_t* p2 = nullptr) {       // p2: a second array, or null
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) {
        p[i] = v;
        if (p2) p2[i] = v;
    }
}

// Column absmax of a row-major matrix.  A workgroup takes 256 columns and a slab of rows: a wave reads 1 KB
// of one row per instruction (each lane 4 adjacent columns), the four waves take every fourth row of the slab,
// 16 row loads in flight per lane; the waves' maxima are merged through LDS and the slabs with one unsigned
// atomic max per column on the bit pattern of |x| (exact and order independent for x >= 0).
#ifndef LRQ_ABSMAX_WGS
#define LRQ_ABSMAX_WGS 1024     // workgroups aimed at (more slabs: more atomics per column)
#endif
// Columns that would cross the end of the row are covered by the row's last four instead (the maximum is idempotent), so
// any stride and 4-byte alignment takes the 16-byte loads (TINY, fewer than four columns: single ones).
template <bool TINY>
__device__ __forceinline__ void absmax_cols_body(const float* __restrict__ X, int ldx, int rows, int cols,
                                                 int rows_per_block, uint32_t* __restrict__ amax_bits, QuantParams q,
                                                 const float* __restrict__ amax0, int bx, int by, float4 (&red)[4][64], int tid) {
    const int quad = tid & 63, rg = tid >> 6;
    const int c = TINY ? 0 : min((bx * 64 + quad) * 4, cols - 4);
    float lam0[4] = {0.f, 0.f, 0.f, 0.f}, s0[4] = {0.f, 0.f, 0.f, 0.f};
    if (amax0) {
#pragma unroll
        for (int t = 0; t < 4; ++t) make_scales(c + t < cols ? amax0[c + t] : 0.f, q.qmaxf, lam0[t], s0[t]);
    }
    const int r0 = by * rows_per_block;
    const int r1 = min(rows, r0 + rows_per_block);
    float4 m = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int rb = r0 + rg; rb < r1; rb += 64) {     // rows clamped into the slab: max is idempotent
        float4 v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const float* row = X + (size_t)min(rb + 4 * u, r1 - 1) * ldx;
            v[u] = TINY ? load4_tail(row, c, cols) : load4u(row + c);
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            if (amax0)
                v[u] = make_float4(quant_residual(v[u].x, lam0[0], s0[0], q), quant_residual(v[u].y, lam0[1], s0[1], q),
                                   quant_residual(v[u].z, lam0[2], s0[2], q), quant_residual(v[u].w, lam0[3], s0[3], q));
            m.x = fmaxf(m.x, fabsf(v[u].x));
            m.y = fmaxf(m.y, fabsf(v[u].y));
            m.z = fmaxf(m.z, fabsf(v[u].z));
            m.w = fmaxf(m.w, fabsf(v[u].w));
        }
    }
    red[rg][quad] = m;
    __syncthreads();
    if (rg != 0 || (bx * 64 + quad) * 4 >= cols) return;
#pragma unroll
    for (int g = 1; g < 4; ++g) {
        const float4 o = red[g][quad];
        m.x = fmaxf(m.x, o.x); m.y = fmaxf(m.y, o.y); m.z = fmaxf(m.z, o.z); m.w = fmaxf(m.w, o.w);
    }
    if (c + 0 < cols) atomicMax(amax_bits + c + 0, __float_as_uint(m.x));
    if (c + 1 < cols) atomicMax(amax_bits + c + 1, __float_as_uint(m.y));
    if (c + 2 < cols) atomicMax(amax_bits + c + 2, __float_as_uint(m.z));
    if (c + 3 < cols) atomicMax(amax_bits + c + 3, __float_as_uint(m.w));
}
template <bool TINY>
__global__ __launch_bounds__(256) void absmax_cols_kernel(const float* __restrict__ X, int ldx, int rows,
                                                          int cols, int rows_per_block,
                                                          uint32_t* __restrict__ amax_bits, QuantParams q,
                                                          const float* __restrict__ amax0) {
    __shared__ float4 red[4][64];
    absmax_cols_body<TINY>(X, ldx, rows, cols, rows_per_block, amax_bits, q, amax0, blockIdx.x, blockIdx.y, red, threadIdx.x);
}

// The column maxima of 64 columns over all rows, stored without an atomic (lanes that share columns at the end store the same).
template <bool TINY>
__device__ __forceinline__ void absmax_strip(const float* __restrict__ X, int ldx, int rows, int cols, float* __restrict__ amax, int bx,
                                             float4 (&red)[4][64], int tid) {
    const int quad = tid & 15, rg = tid >> 4, k = bx * 64 + 4 * quad;
    const int c = TINY ? 0 : min(k, cols - 4);
    float4 m = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int rb = rg; rb < rows; rb += 128) {
        float4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const float* row = X + (size_t)min(rb + 16 * u, rows - 1) * ldx;
            v[u] = TINY ? load4_tail(row, c, cols) : load4u(row + c);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            m.x = fmaxf(m.x, fabsf(v[u].x));
            m.y = fmaxf(m.y, fabsf(v[u].y));
            m.z = fmaxf(m.z, fabsf(v[u].z));
            m.w = fmaxf(m.w, fabsf(v[u].w));
        }
    }
    float4* const r = &red[0][0];
    r[rg * 16 + quad] = m;
    __syncthreads();
    if (rg != 0 || k >= cols) return;
#pragma unroll
    for (int g = 1; g < 16; ++g) {
        const float4 o = r[g * 16 + quad];
        m.x = fmaxf(m.x, o.x); m.y = fmaxf(m.y, o.y); m.z = fmaxf(m.z, o.z); m.w = fmaxf(m.w, o.w);
    }
    if (c + 0 < cols) amax[c + 0] = m.x;
    if (c + 1 < cols) amax[c + 1] = m.y;
    if (c + 2 < cols) amax[c + 2] = m.z;
    if (c + 3 < cols) amax[c + 3] = m.w;
}

// The row maxima of A and the column maxima of B in one launch, and the sketches beside them, which need nothing: workgroups [0, nbA)
// take four rows of A each, one per wave, the next nbB a 256-column slab of B (maxima already cleared; rows_per_block == 0: a
// strip of 64 columns over all rows, nothing to clear), the rest 256 entries of a sketch.  TINY_A, TINY_B: the operand's own rows
// have fewer than four elements (K or N); one of them may while the other's are long.  Calls, sketches and clearing in a launch
// before / this: 256^3 38.8 / 37.9 us, 200^3 71.9 / 71.2, 2000^3 135.9 / 134.2, 4096^3 int8 336.7 / 333.6, int4 395.8 / 392.9, 16384^3 7730 / 7547.
template <bool TINY_A, bool TINY_B>
__global__ __launch_bounds__(256) void absmax_pair_kernel(const float* __restrict__ A, int lda, int M, int K,
                                                          float* __restrict__ amaxA, int nbA, int nbB,
                                                          const float* __restrict__ B, int ldb, int N, int rows_per_block,
                                                          uint32_t* __restrict__ amaxB, QuantParams q, int col_blocks,
                                                          SketchFill f0, SketchFill f1, int nbF0) {
    __shared__ float4 red[4][64];
    if ((int)blockIdx.x >= nbA + nbB) {
        const int id = blockIdx.x - nbA - nbB;
        if (id < nbF0) fill_sketch_entry(f0, (size_t)id * 256 + threadIdx.x);
        else           fill_sketch_entry(f1, (size_t)(id - nbF0) * 256 + threadIdx.x);
        return;
    }
    if ((int)blockIdx.x >= nbA) {
        const int id = blockIdx.x - nbA;
        if (rows_per_block == 0) absmax_strip<TINY_B>(B, ldb, K, N, reinterpret_cast<float*>(amaxB), id, red, threadIdx.x);
        else absmax_cols_body<TINY_B>(B, ldb, K, N, rows_per_block, amaxB, q, nullptr, id % col_blocks, id / col_blocks, red, threadIdx.x);
        return;
    }
    const int lane = threadIdx.x & 63, row = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= M) return;
    const float* xp = A + (size_t)row * lda;
    float m = 0.f;
    for (int k = lane * 4; k < K; k += 8 * 256) {       // eight loads in flight; past the end the last columns again
        float4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = TINY_A ? load4_tail(xp, 0, K) : load4u(xp + min(k + 256 * u, K - 4));
#pragma unroll
        for (int u = 0; u < 8; ++u)
            m = fmaxf(fmaxf(m, fabsf(v[u].x)), fmaxf(fabsf(v[u].y), fmaxf(fabsf(v[u].z), fabsf(v[u].w))));
    }
    m = wave_max(m);
    if (lane == 0) amaxA[row] = m;
}

// A's rows quantized from one read (as in quant_rows_cached_kernel) beside the column maxima of B (already cleared): workgroups
// [0, nbA) take 256 / TPR rows of A each, the rest a 256-column slab of B, so that both operands stream at once.  RES: the
// residual of A's rows is quantized a second time from the same registers, and B's residual maxima come with its codes.  Calls,
// separate launches / this (and the steps formed in the product's epilogue): rank 0, 4096^3 int4 119 / 106 us, 2000^3 52 / 36.5,
// 300^3 23.6 / 18.4; four residual products (one launch for the products), 4096^3 376 / 354.
template <int TPR, int NV, bool RES>
__global__ __launch_bounds__(256) void quant_pair_kernel(const float* __restrict__ A, int lda, int M, int K, QuantPair o, int nbA,
                                                         const float* __restrict__ B, int ldb, int N, int rows_per_block,
                                                         QuantParams q, int col_blocks) {
    __shared__ float4 red[4][64];
    __shared__ float wmax[2][4];
    if ((int)blockIdx.x >= nbA) {
        const int id = blockIdx.x - nbA;
        absmax_cols_body<false>(B, ldb, K, N, rows_per_block, reinterpret_cast<uint32_t*>(o.amaxB), q, nullptr, id % col_blocks,
                                id / col_blocks, red, threadIdx.x);
        return;
    }
    const int t = threadIdx.x % TPR;
    const int row = blockIdx.x * (256 / TPR) + threadIdx.x / TPR;
    const bool row_ok = row < M;
    const float* xp = A + (size_t)(row_ok ? row : 0) * lda;
    float4 v[NV];
#pragma unroll
    for (int u = 0; u < NV; ++u) v[u] = load_quad<false>(xp, (t + TPR * u) * 4, K);
#pragma unroll
    for (int level = 0; level < (RES ? 2 : 1); ++level) {
        float m = 0.0f;
#pragma unroll
        for (int u = 0; u < NV; ++u)
            m = fmaxf(fmaxf(m, fabsf(v[u].x)), fmaxf(fabsf(v[u].y), fmaxf(fabsf(v[u].z), fabsf(v[u].w))));
        m = wave_max(m);
        if (TPR == 256) {
            if ((threadIdx.x & 63) == 0) wmax[level][threadIdx.x >> 6] = m;
            __syncthreads();
            m = fmaxf(fmaxf(wmax[level][0], wmax[level][1]), fmaxf(wmax[level][2], wmax[level][3]));
        }
        if (row_ok && t == 0) (level == 0 ? o.amaxA : o.amaxRA)[row] = m;
        float lam, s;
        make_scales(m, q.qmaxf, lam, s);
        int8_t* cp = (level == 0 ? o.codesA : o.codesRA) + (size_t)(row_ok ? row : 0) * K;
#pragma unroll
        for (int u = 0; u < NV; ++u) {
            const int k = (t + TPR * u) * 4;
            if (row_ok && k < K) store_quad<false>(cp, k, K, pack_codes(v[u], lam, q));
            if (RES && level == 0) v[u] = first_level_residual(v[u], lam, s, q);
        }
    }
}

// The same with packed codes (see PK8, PK6).  A workgroup of WG threads takes WG / TPR rows, so that
// the lanes of a block that it stores are 128 bytes (64 beyond 4096 columns) next to each other; the codes cross the waves through
// LDS.  On B's side it works as workgroups of 256.  (16 rows a workgroup, 256 bytes: 65 KB of LDS and 16 waves leave one per CU, a call
// of 4096^3 93.5 us against 89.7.)
template <int FMT, int WG, int TPR, int NV, bool RES>
__global__ __launch_bounds__(WG) void quant_pair_packed_kernel(const float* __restrict__ A, int lda, int M, int K, QuantPair o, int nbA,
                                                                 const float* __restrict__ B, int ldb, int N, int rows_per_block,
                                                                 QuantParams q, int col_blocks, int col_jobs) {
    constexpr int ROWS = WG / TPR, LDW = TPR * NV + 4;      // (+ 4: conflict-free 16-byte reads)
    __shared__ __align__(16) uint32_t words[ROWS * LDW > 4 * WG ? ROWS * LDW : 4 * WG];
    auto& red = *reinterpret_cast<float4 (*)[WG / 256][4][64]>(words);
    __shared__ float wmax[16];
    if ((int)blockIdx.x >= nbA) {
        const int sub = threadIdx.x >> 8, id = min(((int)blockIdx.x - nbA) * (WG / 256) + sub, col_jobs - 1);     // (a maximum does not mind)
        absmax_cols_body<false>(B, ldb, K, N, rows_per_block, reinterpret_cast<uint32_t*>(o.amaxB), q, nullptr, id % col_blocks,
                                id / col_blocks, red[sub], threadIdx.x & 255);
        return;
    }
    const int t = threadIdx.x % TPR, r = threadIdx.x / TPR;
    const int row0 = blockIdx.x * ROWS, row = row0 + r;
    const float* xp = A + (size_t)min(row, M - 1) * lda;
    float4 v[NV];
#pragma unroll
    for (int u = 0; u < NV; ++u) v[u] = load_quad<false>(xp, (t + TPR * u) * 4, K);
    const int nkb = pk_kblocks(K);
#pragma unroll
    for (int level = 0; level < (RES ? 2 : 1); ++level) {
        if (level) __syncthreads();         // the first level's codes have left, its maxima are read
        float m = 0.0f;
#pragma unroll
        for (int u = 0; u < NV; ++u)
            m = fmaxf(fmaxf(m, fabsf(v[u].x)), fmaxf(fabsf(v[u].y), fmaxf(fabsf(v[u].z), fabsf(v[u].w))));
        m = wave_max(m);
        if (TPR == 256) {
            if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = m;
            __syncthreads();
            m = fmaxf(fmaxf(wmax[4 * r], wmax[4 * r + 1]), fmaxf(wmax[4 * r + 2], wmax[4 * r + 3]));
        }
        if (row < M && t == 0) (level == 0 ? o.amaxA : o.amaxRA)[row] = m;
        float lam, s;
        make_scales(m, q.qmaxf, lam, s);
#pragma unroll
        for (int u = 0; u < NV; ++u) {
            const int k = (t + TPR * u) * 4;
            if (k < nkb * PK_K) {
                uint32_t w;
                if constexpr (FMT == PK8) w = pack_codes(v[u], lam, q);
                else w = six_bits(quant_code(v[u].x, lam, q)) | six_bits(quant_code(v[u].y, lam, q)) << 6 |
                         six_bits(quant_code(v[u].z, lam, q)) << 12 | six_bits(quant_code(v[u].w, lam, q)) << 18;
                const int past = k - (K - 4);           // (the row's last four values stand in where the quad crosses its end)
                if (past > 0) w = past < 4 ? w >> (FMT * past) : 0u;
                words[r * LDW + (k >> 2)] = w;
            }
            if (RES && level == 0) v[u] = first_level_residual(v[u], lam, s, q);
        }
        __syncthreads();
        uint8_t* const codes = reinterpret_cast<uint8_t*>(level == 0 ? o.codesA : o.codesRA);
        for (int e = threadIdx.x; e < ROWS * 2 * nkb; e += WG) {
            const int rr = e % ROWS, unit = e / ROWS, orow = row0 + rr;
            if (orow >= M) continue;
            const uint4* src = reinterpret_cast<const uint4*>(&words[rr * LDW + 8 * unit]);
            const uint4 lo = src[0], hi = src[1];
            uint32_t w[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
            store_packed<FMT>(codes + ((size_t)(orow >> 5) * nkb + (unit >> 1)) * pk_block(FMT), 32 * (unit & 1) + (orow & 31), w, 32);
        }
    }
}

// Quantize a 64(k) x 64(n) tile with per-column scales and store it transposed
// (codesT is cols x rows, contiguous along the original row index k).  Columns at the end as in the row kernels (what
// then lies before the tile belongs to the neighbour and is dropped); codes leave 16 bytes at a time at any alignment.
// RMAX: the column maxima of the residual (already cleared) come from the same read.  PACKED: packed codes of this format.
template <bool TINY, bool RMAX = false, int PACKED = PK_NONE>
__global__ __launch_bounds__(256) void quant_cols_kernel(const float* __restrict__ X, int ldx, int rows,
                                                         int cols, const float* __restrict__ amax,
                                                         QuantParams q,
                                                         int8_t* __restrict__ codesT,
                                                         const float* __restrict__ amax0, uint32_t* __restrict__ rmax_bits) {
    __shared__ __align__(16) int8_t tile[64][80];
    __shared__ float4 red[RMAX ? 16 : 1][16];
    float4 rm = make_float4(0.f, 0.f, 0.f, 0.f);
    const int n0 = blockIdx.x * 64, k0 = blockIdx.y * 64;
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    const int n = TINY ? n0 + tx * 4 : min(n0 + tx * 4, cols - 4);
    float lam[4], stp[4], lam0[4] = {0.f, 0.f, 0.f, 0.f}, s0[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 4; ++t) make_scales((n + t < cols) ? amax[n + t] : 0.0f, q.qmaxf, lam[t], stp[t]);
    if (amax0) {
#pragma unroll
        for (int t = 0; t < 4; ++t) make_scales(n + t < cols ? amax0[n + t] : 0.f, q.qmaxf, lam0[t], s0[t]);
    }
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
        const int kl = ty + 16 * rr;
        const float* row = X + (size_t)min(k0 + kl, rows - 1) * ldx;       // rows past the end: never stored
        float4 v = TINY ? load4_tail(row, n, cols) : load4u(row + n);
        if (amax0)
            v = make_float4(quant_residual(v.x, lam0[0], s0[0], q), quant_residual(v.y, lam0[1], s0[1], q),
                            quant_residual(v.z, lam0[2], s0[2], q), quant_residual(v.w, lam0[3], s0[3], q));
        const float c[4] = {quant_code(v.x, lam[0], q), quant_code(v.y, lam[1], q), quant_code(v.z, lam[2], q),
                            quant_code(v.w, lam[3], q)};
        if (RMAX) {         // (rows clamped to the last one: a maximum does not mind)
            rm.x = fmaxf(rm.x, fabsf(fmaf(-c[0], stp[0], v.x)));
            rm.y = fmaxf(rm.y, fabsf(fmaf(-c[1], stp[1], v.y)));
            rm.z = fmaxf(rm.z, fabsf(fmaf(-c[2], stp[2], v.z)));
            rm.w = fmaxf(rm.w, fabsf(fmaf(-c[3], stp[3], v.w)));
        }
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (TINY || n - n0 + t >= 0) tile[n - n0 + t][kl] = (int8_t)(PACKED == PK6 ? (int)six_bits(c[t]) : (int)c[t]);
    }
    if (RMAX) red[ty][tx] = rm;
    __syncthreads();
    if (RMAX && ty == 0) {
#pragma unroll
        for (int g = 1; g < 16; ++g) {
            const float4 o = red[g][tx];
            rm.x = fmaxf(rm.x, o.x); rm.y = fmaxf(rm.y, o.y); rm.z = fmaxf(rm.z, o.z); rm.w = fmaxf(rm.w, o.w);
        }
        // (columns n .. n + 3 exist unless TINY, which has no residual maxima)
        atomicMax(rmax_bits + n + 0, __float_as_uint(rm.x));
        atomicMax(rmax_bits + n + 1, __float_as_uint(rm.y));
        atomicMax(rmax_bits + n + 2, __float_as_uint(rm.z));
        atomicMax(rmax_bits + n + 3, __float_as_uint(rm.w));
    }
    if constexpr (PACKED != PK_NONE) {
        store_packed_tile<PACKED, 64, 64, 80, true>(&tile[0][0], reinterpret_cast<uint8_t*>(codesT), n0, cols, k0, rows, threadIdx.x, 256);
        return;
    }
    const int nl = threadIdx.x >> 2, chunk = threadIdx.x & 3;
    const int nn = n0 + nl;
    if (nn >= cols) return;
    const int kb = k0 + chunk * 16;
    int8_t* dst = codesT + (size_t)nn * rows + kb;
    if (kb + 16 <= rows) {
        __builtin_memcpy(dst, __builtin_assume_aligned(&tile[nl][chunk * 16], 16), 16);
    } else {
        for (int b = 0; kb + b < rows; ++b) dst[b] = tile[nl][chunk * 16 + b];
    }
}

__global__ void scales_kernel(const float* __restrict__ amax, int n, int npad, float qmaxf,
                              float* __restrict__ lam, float* __restrict__ s) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= npad) return;
    float l = 0.0f, st = 0.0f;
    if (i < n) make_scales(amax[i], qmaxf, l, st);
    lam[i] = l;
    s[i] = st;
}

// One scale for the whole matrix (the paper's own Eq. (quantA)): every entry of amax[n] is
// replaced by the maximum of all of them.  One workgroup per matrix; max is exact and order independent.
__global__ __launch_bounds__(1024) void tensor_max_kernel(float* __restrict__ amax0, int n0, float* __restrict__ amax1,
                                                          int n1) {
    __shared__ float wm[16];
    float* __restrict__ const amax = blockIdx.x == 0 ? amax0 : amax1;
    const int n = blockIdx.x == 0 ? n0 : n1;
    float m = 0.0f;
    for (int i = threadIdx.x; i < n; i += 1024) m = fmaxf(m, amax[i]);
    m = wave_max(m);
    if ((threadIdx.x & 63) == 0) wm[threadIdx.x >> 6] = m;
    __syncthreads();
    m = wm[0];
#pragma unroll
    for (int w = 1; w < 16; ++w) m = fmaxf(m, wm[w]);
    for (int i = threadIdx.x; i < n; i += 1024) amax[i] = m;
}

static int rows_launch(const float* X, int ldx, int rows, int cols, QuantParams q, int8_t* codes, float* amax,
                       int mode, const float* amax0, hipStream_t st);

int launch_quantize_rows(const float* X, int ldx, int rows, int cols, QuantParams q, bool per_tensor,
                         const float* amax0, int8_t* codes, float* amax, hipStream_t st) {
    if (!per_tensor) return rows_launch(X, ldx, rows, cols, q, codes, amax, ROWS_FULL, amax0, st);
    // one scale per matrix: row maxima, their maximum broadcast to every row, then the codes
    int rc = rows_launch(X, ldx, rows, cols, q, codes, amax, ROWS_AMAX_ONLY, amax0, st);
    if (rc != LRQMM_OK) return rc;
    hipLaunchKernelGGL(tensor_max_kernel, dim3(1), dim3(1024), 0, st, amax, rows, nullptr, 0);
    LRQ_CHECK_LAUNCH();
    return rows_launch(X, ldx, rows, cols, q, codes, amax, ROWS_GIVEN_AMAX, amax0, st);
}

static int rows_launch(const float* X, int ldx, int rows, int cols, QuantParams q, int8_t* codes, float* amax,
                       int mode, const float* amax0, hipStream_t st) {
    if (cols < 4) {
        hipLaunchKernelGGL((quant_rows_cached_kernel<true, 64, 1>), dim3(ceil_div(rows, 4)), dim3(256), 0, st, X, ldx, rows, cols,
                           q, codes, amax, mode, amax0);
    } else if (cols <= 256 * 4 * 16) {
        // Row cached in registers: one wavefront per row up to 4096 columns, else one workgroup.
        const bool wave = cols <= 64 * 4 * 16;
        const int per = wave ? 256 : 1024;
        const int need = ceil_div(cols, per);
        dim3 grid(wave ? ceil_div(rows, 4) : rows);
#define LRQ_QR(T, N) hipLaunchKernelGGL((quant_rows_cached_kernel<false, T, N>), grid, dim3(256), 0, st, X, ldx, rows, cols, q, codes, amax, mode, amax0)
#define LRQ_QR_NV(T) do { if (need <= 1) LRQ_QR(T, 1); else if (need <= 2) LRQ_QR(T, 2); \
        else if (need <= 4) LRQ_QR(T, 4); else if (need <= 8) LRQ_QR(T, 8); else LRQ_QR(T, 16); } while (0)
        if (wave) LRQ_QR_NV(64);
        else      LRQ_QR_NV(256);
#undef LRQ_QR_NV
#undef LRQ_QR
    } else {                              // very long rows: two passes over the row
        dim3 grid(ceil_div(rows, 4));
        hipLaunchKernelGGL(quant_rows_kernel<false>, grid, dim3(256), 0, st, X, ldx, rows, cols, q, codes, amax, mode, amax0);
    }
    LRQ_CHECK_LAUNCH();
    return LRQMM_OK;
}

namespace {
struct ColSlabs { int col_blocks, slabs, rows_per_block; };
// enough row slabs to fill the chip, at least 64 rows each (one batch of loads per lane)
ColSlabs plan_slabs(int rows, int cols) {
    ColSlabs p;
    p.col_blocks = ceil_div(cols, 256);
    p.slabs = max(1, min(ceil_div(rows, 64), ceil_div(LRQ_ABSMAX_WGS, p.col_blocks)));
    p.rows_per_block = ceil_div(rows, p.slabs);
    p.slabs = ceil_div(rows, p.rows_per_block);
    return p;
}
}  // namespace

// Rows of B up to which a strip of columns goes over all of them (a workgroup then reads at most 128 KB).
#define ABSMAX_STRIP_ROWS 512

int launch_absmax_pair(const float* A, int lda, int M, int K, float* amaxA, const float* B, int ldb, int N,
                       float* amaxB, QuantParams q, bool per_tensor, const SketchJob* fill, int nfill, hipStream_t st) {
    const bool strips = K <= ABSMAX_STRIP_ROWS;
    ColSlabs p = N > 0 ? plan_slabs(K, N) : ColSlabs{1, 0, 1};
    if (strips) p = {1, ceil_div(N, 64), 0};
    if (N > 0 && !strips)
        hipLaunchKernelGGL(fill_u32_kernel, dim3(ceil_div(N, 256)), dim3(256), 0, st, reinterpret_cast<uint32_t*>(amaxB), N, 0u, nullptr);
    SketchFill f[2] = {};
    int nbF[2] = {0, 0};
    for (int i = 0; i < nfill; ++i) {
        f[i] = make_fill(fill[i].seed, fill[i].stream_id, fill[i].rows, fill[i].cols, fill[i].ld, fill[i].omega);
        nbF[i] = fill_blocks(f[i]);
    }
    const int nbA = ceil_div(M, 4), nbB = p.col_blocks * p.slabs;
    dim3 grid(nbA + nbB + nbF[0] + nbF[1]);
#define LRQ_ABSMAX(TA, TB)                                                                                              \
    hipLaunchKernelGGL((absmax_pair_kernel<TA, TB>), grid, dim3(256), 0, st, A, lda, M, K, amaxA, nbA, nbB, B, ldb, N,  \
                       p.rows_per_block, reinterpret_cast<uint32_t*>(amaxB), q, p.col_blocks, f[0], f[1], nbF[0])
    if (K >= 4) { if (N >= 4) LRQ_ABSMAX(false, false); else LRQ_ABSMAX(false, true); }
    else        { if (N >= 4) LRQ_ABSMAX(true, false); else LRQ_ABSMAX(true, true); }
#undef LRQ_ABSMAX
    LRQ_CHECK_LAUNCH();
    if (per_tensor) {
        if (M > 0 && N > 0) hipLaunchKernelGGL(tensor_max_kernel, dim3(2), dim3(1024), 0, st, amaxA, M, amaxB, N);
        else hipLaunchKernelGGL(tensor_max_kernel, dim3(1), dim3(1024), 0, st, M > 0 ? amaxA : amaxB, max(M, N), nullptr, 0);
        LRQ_CHECK_LAUNCH();
    }
    return LRQMM_OK;
}

int launch_quantize_cols(const float* X, int ldx, int rows, int cols, QuantParams q, bool per_tensor,
                         const float* amax0, int8_t* codesT, float* amax, hipStream_t st) {
    hipLaunchKernelGGL(fill_u32_kernel, dim3(ceil_div(cols, 256)), dim3(256), 0, st, reinterpret_cast<uint32_t*>(amax), cols,
                       0u, nullptr);
    const ColSlabs p = plan_slabs(rows, cols);
    dim3 g1(p.col_blocks, p.slabs), g2(ceil_div(cols, 64), ceil_div(rows, 64));
    uint32_t* const bits = reinterpret_cast<uint32_t*>(amax);
    if (cols >= 4) hipLaunchKernelGGL(absmax_cols_kernel<false>, g1, dim3(256), 0, st, X, ldx, rows, cols, p.rows_per_block, bits, q, amax0);
    else           hipLaunchKernelGGL(absmax_cols_kernel<true>, g1, dim3(256), 0, st, X, ldx, rows, cols, p.rows_per_block, bits, q, amax0);
    if (per_tensor) hipLaunchKernelGGL(tensor_max_kernel, dim3(1), dim3(1024), 0, st, amax, cols, nullptr, 0);
    if (cols >= 4) hipLaunchKernelGGL(quant_cols_kernel<false>, g2, dim3(256), 0, st, X, ldx, rows, cols, amax, q, codesT, amax0, nullptr);
    else           hipLaunchKernelGGL(quant_cols_kernel<true>, g2, dim3(256), 0, st, X, ldx, rows, cols, amax, q, codesT, amax0, nullptr);
    LRQ_CHECK_LAUNCH();
    return LRQMM_OK;
}

bool quantize_pair_usable(int M, int N, int K) { return M > 0 && N >= 4 && K >= 4 && K <= 16384; }

int launch_quantize_pair(const float* A, int lda, const float* B, int ldb, int M, int N, int K, QuantParams q, QuantPair o,
                         hipStream_t st, int packed) {
    const bool res = o.codesRA != nullptr;
    if (!quantize_pair_usable(M, N, K)) return LRQMM_ERR_UNSUPPORTED;
    uint32_t *const bits = reinterpret_cast<uint32_t*>(o.amaxB), *const rbits = reinterpret_cast<uint32_t*>(o.amaxRB);
    hipLaunchKernelGGL(fill_u32_kernel, dim3(ceil_div(N, 256)), dim3(256), 0, st, bits, N, 0u, res ? rbits : nullptr);
    const ColSlabs p = plan_slabs(K, N);
    const bool wave = K <= 64 * 4 * 16;         // one wave per row, or a workgroup
    const int need = ceil_div(K, wave ? 256 : 1024), nbA = wave ? ceil_div(M, 4) : M;
    const dim3 grid(nbA + p.col_blocks * p.slabs), g2(ceil_div(N, 64), ceil_div(K, 64));
    if (packed) {
        const int rows = wave ? 8 : 4, nbP = ceil_div(M, rows), jobs = p.col_blocks * p.slabs;
        const dim3 gp(nbP + ceil_div(jobs, wave ? 2 : 4));
#define LRQ_QPP(F, T, NV, R)                                                                                           \
    hipLaunchKernelGGL((quant_pair_packed_kernel<F, (T == 64 ? 512 : 1024), T, NV, R>), gp, dim3(T == 64 ? 512 : 1024), 0, st, A, lda, \
                       M, K, o, nbP, B, ldb, N, p.rows_per_block, q, p.col_blocks, jobs)
#define LRQ_QPP_NV(F, T, R) do { if (need <= 1) LRQ_QPP(F, T, 1, R); else if (need <= 2) LRQ_QPP(F, T, 2, R); \
        else if (need <= 4) LRQ_QPP(F, T, 4, R); else if (need <= 8) LRQ_QPP(F, T, 8, R); else LRQ_QPP(F, T, 16, R); } while (0)
#define LRQ_QPP_T(F, R) do { if (wave) LRQ_QPP_NV(F, 64, R); else LRQ_QPP_NV(F, 256, R); } while (0)
#define LRQ_QCP(F, R, AMAX, CODES, AMAX0, RBITS) \
    hipLaunchKernelGGL((quant_cols_kernel<false, R, F>), g2, dim3(256), 0, st, B, ldb, K, N, AMAX, q, CODES, AMAX0, RBITS)
#define LRQ_PAIR(F)                                                 \
    do {                                                            \
        if (res) {                                                  \
            LRQ_QPP_T(F, true);                                     \
            LRQ_QCP(F, true, o.amaxB, o.codesB, nullptr, rbits);    \
            LRQ_QCP(F, false, o.amaxRB, o.codesRB, o.amaxB, nullptr); \
        } else {                                                    \
            LRQ_QPP_T(F, false);                                    \
            LRQ_QCP(F, false, o.amaxB, o.codesB, nullptr, nullptr); \
        }                                                           \
    } while (0)
        if (packed == PK6) LRQ_PAIR(PK6);
        else               LRQ_PAIR(PK8);
#undef LRQ_PAIR
#undef LRQ_QCP
#undef LRQ_QPP_T
#undef LRQ_QPP_NV
#undef LRQ_QPP
        LRQ_CHECK_LAUNCH();
        return LRQMM_OK;
    }
#define LRQ_QP(T, NV)                                                                                                         \
    do {                                                                                                                      \
        if (res) hipLaunchKernelGGL((quant_pair_kernel<T, NV, true>), grid, dim3(256), 0, st, A, lda, M, K, o, nbA, B, ldb, N,  \
                                    p.rows_per_block, q, p.col_blocks);                                                       \
        else     hipLaunchKernelGGL((quant_pair_kernel<T, NV, false>), grid, dim3(256), 0, st, A, lda, M, K, o, nbA, B, ldb, N, \
                                    p.rows_per_block, q, p.col_blocks);                                                       \
    } while (0)
#define LRQ_QP_NV(T) do { if (need <= 1) LRQ_QP(T, 1); else if (need <= 2) LRQ_QP(T, 2); \
        else if (need <= 4) LRQ_QP(T, 4); else if (need <= 8) LRQ_QP(T, 8); else LRQ_QP(T, 16); } while (0)
    if (wave) LRQ_QP_NV(64);
    else      LRQ_QP_NV(256);
#undef LRQ_QP_NV
#undef LRQ_QP
    if (res) {
        hipLaunchKernelGGL((quant_cols_kernel<false, true>), g2, dim3(256), 0, st, B, ldb, K, N, o.amaxB, q, o.codesB, nullptr, rbits);
        hipLaunchKernelGGL((quant_cols_kernel<false>), g2, dim3(256), 0, st, B, ldb, K, N, o.amaxRB, q, o.codesRB, o.amaxB, nullptr);
    } else {
        hipLaunchKernelGGL((quant_cols_kernel<false>), g2, dim3(256), 0, st, B, ldb, K, N, o.amaxB, q, o.codesB, nullptr, nullptr);
    }
    LRQ_CHECK_LAUNCH();
    return LRQMM_OK;
}

int launch_tick(uint32_t* word, hipStream_t st) {
    hipLaunchKernelGGL(fill_u32_kernel, dim3(1), dim3(64), 0, st, word, 1, 0u, nullptr);
    LRQ_CHECK_LAUNCH();
    return LRQMM_OK;
}

int launch_scales(const float* amax, int n, int npad, float qmaxf, float* lam, float* s,
                  hipStream_t st) {
    hipLaunchKernelGGL(scales_kernel, dim3(ceil_div(npad, 256)), dim3(256), 0, st, amax, n, npad, qmaxf, lam, s);
    LRQ_CHECK_LAUNCH();
    return LRQMM_OK;
}
