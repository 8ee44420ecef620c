// Quantization of a tall operand with short rows and both of its residual products from one read (paper: Algorithm 2, quantization and
// residual steps; Algorithm 1 without power iterations: the sample matrix Y = R Omega, and R^T Q as (R^T Y) T with Q = Y T).
#include <type_traits>
#include "kernels.h"

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

__device__ __forceinline__ v4f mfma_f32(float a, float b, v4f c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// The largest value of a wave, the same in every lane.
__device__ __forceinline__ float wave_max_uniform(float v) {
    auto take = [&](auto ctrl) {
        v = fmaxf(v, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), decltype(ctrl)::value, 0xf, 0xf, true)));
    };
    take(std::integral_constant<int, 0xb1>{});      // neighbours, pairs, halves and the whole of a row of 16 lanes
    take(std::integral_constant<int, 0x4e>{});
    take(std::integral_constant<int, 0x141>{});
    take(std::integral_constant<int, 0x140>{});
    float m = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 0));
#pragma unroll
    for (int i = 16; i < 64; i += 16) m = fmaxf(m, __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), i)));
    return m;
}

// A lane's offset from a wave-uniform base, opaque to the compiler, which else moves 64-bit forms of all of them out of the loop and spills
// them: every reload then waits for the next tile's loads (142 us in place of 93).
__device__ __forceinline__ uint32_t lane_offset(uint32_t o) {
    asm("" : "+v"(o));
    return o;
}

template <int RM>
__device__ __forceinline__ float code_residual(float x, float lam, float s, const QuantParams& q, float& code) {
    const float t = x * lam;
    code = clamp_code(RM == 0 ? floorf(t) : rintf(t), q);
    return fmaf(-code, s, x);
}

// A tile is 16 rows, a row to each of sixteen waves; workgroups are persistent and take a contiguous run of tiles.
//   * Adjacent lanes read adjacent 16-byte pieces of the row, so loads and the code stores are coalesced and a row's maximum stays inside
//     one wave.  The next tile is loaded into the same registers as soon as the residuals are in LDS.
//   * The residuals are a tile in LDS (row stride = 4 mod 64 floats: the 64 lanes of an operand read 64 different banks, along the rows and
//     across them).  For Y the waves split the columns, the wave's part of the sketch in registers; the sixteen partial products are
//     added in pairs.  For R^T Y a wave has up to three tiles of 16 columns, whose sums stay in its registers for the whole run.
//   * Y^T Y is added to a float64 matrix in LDS.
// The sketch is multiplied by a reflection that leaves only its first column with a sum.  Residuals of floor rounding have a mean, so every
// column of R Omega would be nearly the same vector, and T would have to take that out of R^T Y again; Q Q^T R is the same for both.  Where
// Y is ill-conditioned all the same, or far from unit scale, a pass for R^T Q follows (PROJECT_AMPLIFICATION).
// What bounds it: the phases between the barriers, one after the other, of two workgroups a CU that cover each other (what the 64 registers are
// for).  100352 x 576: 93 us for 289 MB; without the product R^T Y 72, without Y 75, without the loads 86.  quant_sketch_rows_kernel and a pass
// for R^T Q, which read X twice, 73 + 48 us; the call of 64 columns 203 -> 170 us.  (Eight waves of two rows with 128 registers spilled: 110 us.)
template <int NB>       // blocks of 64 columns
__global__ __launch_bounds__(1024, 8) void quant_project_rows_kernel(
    const float* __restrict__ X, int ldx, int rows, int cols, QuantParams q, const float* __restrict__ W,
    float* __restrict__ Y, double* __restrict__ gpart, float* __restrict__ mpart, float* __restrict__ amax, float* __restrict__ lam_out,
    float* __restrict__ s_out, int8_t* __restrict__ codes) {
    constexpr int NV = (NB + 3) / 4, NS = NB, ND = (4 * NB + 15) / 16;      // 16-byte pieces a lane, steps and tiles of R^T Y a wave
    extern __shared__ __align__(16) float rt[];
    __shared__ __align__(16) float pacc[16][256];
    __shared__ float yt[16][17];
    __shared__ double gl[256];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int r = lane & 15, g = lane >> 4;
    const int cpr = cols >> 2;
    constexpr int ldr = 64 * NB + 4;                     // (a constant: addresses are one register and immediate offsets)
    const int s0 = wave * NS;                            // the wave's steps of four columns; columns past the end are zeros
    const int ntiles = (rows + 15) >> 4;
    const int t0 = (int)((long long)blockIdx.x * ntiles / gridDim.x);
    const int t1 = (int)((long long)(blockIdx.x + 1) * ntiles / gridDim.x);
    if (t0 >= t1) return;                                // uniform
    if (tid < 256) gl[tid] = 0.0;
    for (int c = cols + lane; c < 64 * NB; c += 64) rt[wave * ldr + c] = 0.f;
    float4 x[NV];
    auto load_row = [&](int tile) {     // (rows past the end: the last one, not stored; pieces past the row: its last, not used)
        const char* p = reinterpret_cast<const char*>(X + (size_t)min(tile * 16 + wave, rows - 1) * ldx);
        asm("" : "+s"(p));
#pragma unroll
        for (int u = 0; u < NV; ++u) x[u] = *reinterpret_cast<const float4*>(p + lane_offset(16u * min((uint32_t)(lane + 64 * u), (uint32_t)(cpr - 1))));
    };
    // The reflection, from the column sums of the sketch
    float wreg[NS];             // B operands: (Omega H)[4 s + g][r] for the wave's steps
    {
        float* const part = &pacc[0][0];                // [64][16]
        float w[NS], sum = 0.f;
#pragma unroll
        for (int i = 0; i < NS; ++i) w[i] = W[(size_t)min((tid >> 4) + 64 * i, cols - 1) * 16 + (tid & 15)];
#pragma unroll
        for (int i = 0; i < NS; ++i) wreg[i] = W[(size_t)min(4 * (s0 + i) + g, cols - 1) * 16 + r];
#pragma unroll
        for (int i = 0; i < NS; ++i) sum += (tid >> 4) + 64 * i < cols ? w[i] : 0.f;
        part[tid] = sum;
        __syncthreads();
        float v = 0.f;
        for (int k = 0; k < 64; ++k) v += part[16 * k + r];         // column r's, in every wave
        float norm2 = v * v;
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) norm2 += __shfl_xor(norm2, o, 64);
        const float v0 = __shfl(v, 0, 64), head = v0 + copysignf(__fsqrt_rn(norm2), v0);
        if (r == 0) v = head;
        const float vv = norm2 - v0 * v0 + head * head, beta = vv > 0.f ? 2.f / vv : 0.f;
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            float dot = wreg[i] * v;                    // over the 16 lanes of the row
#pragma unroll
            for (int o = 1; o < 16; o <<= 1) dot += __shfl_xor(dot, o, 64);
            wreg[i] = 4 * (s0 + i) + g < cols ? fmaf(-(beta * dot), v, wreg[i]) : 0.f;
        }
        __syncthreads();
    }
    load_row(t0);
    v4f macc[ND];               // R^T Y so far: columns col_of(i) + 16 g + v, sketch column r
#pragma unroll
    for (int i = 0; i < ND; ++i) macc[i] = (v4f){0.f, 0.f, 0.f, 0.f};
    auto col_of = [&](int i) { const int d = wave + 16 * i; return 64 * (d >> 2) + 4 * (d & 3); };
    for (int tile = t0; tile < t1; ++tile) {
        const int row = tile * 16 + wave;
        float m = 0.f;
#pragma unroll
        for (int u = 0; u < NV; ++u) {
            const float mm = fmaxf(fmaxf(fabsf(x[u].x), fabsf(x[u].y)), fmaxf(fabsf(x[u].z), fabsf(x[u].w)));
            m = fmaxf(m, lane + 64 * u < cpr ? mm : 0.f);
        }
        m = wave_max_uniform(m);
        float lam, sc;
        make_scales(m, q.qmaxf, lam, sc);
        if (lane == 0 && row < rows) {
            amax[row] = m;
            lam_out[row] = lam;
            s_out[row] = sc;
        }
        if (tile > t0) __syncthreads();                 // the last tile's residuals have been read
        int8_t* crow = codes + (size_t)min(row, rows - 1) * cols;
        asm("" : "+s"(crow));
        auto quantize = [&](auto mode) {
            constexpr int RM = decltype(mode)::value;
#pragma unroll
            for (int u = 0; u < NV; ++u) {
                const int c = lane + 64 * u;
                if (c >= cpr) continue;
                float c0, c1, c2, c3;
                float4 res;
                res.x = code_residual<RM>(x[u].x, lam, sc, q, c0);
                res.y = code_residual<RM>(x[u].y, lam, sc, q, c1);
                res.z = code_residual<RM>(x[u].z, lam, sc, q, c2);
                res.w = code_residual<RM>(x[u].w, lam, sc, q, c3);
                // (the low byte of code + 1.5 2^23 is the code)
                const uint32_t b0 = __float_as_uint(c0 + 12582912.f), b1 = __float_as_uint(c1 + 12582912.f);
                const uint32_t b2 = __float_as_uint(c2 + 12582912.f), b3 = __float_as_uint(c3 + 12582912.f);
                const uint32_t pk = __builtin_amdgcn_perm(__builtin_amdgcn_perm(b3, b2, 0x0c0c0400), __builtin_amdgcn_perm(b1, b0, 0x0c0c0400), 0x05040100);
                if (row < rows) *reinterpret_cast<uint32_t*>(crow + lane_offset(4u * (uint32_t)c)) = pk;
                *reinterpret_cast<float4*>(rt + wave * ldr + 4 * c) = res;
            }
        };
        if (q.round_mode == 0) quantize(std::integral_constant<int, 0>{});
        else quantize(std::integral_constant<int, 1>{});
        if (tile + 1 < t1) load_row(tile + 1);          // in flight during the products
        __syncthreads();        // the tile's residuals are in LDS
        const int ln = (int)lane_offset(lane), r = ln & 15, g = ln >> 4;        // (addresses formed here, not held over the tile)
        v4f acc = (v4f){0.f, 0.f, 0.f, 0.f};
        const float* ap = rt + r * ldr + 4 * s0 + g;
#pragma unroll
        for (int i = 0; i < NS; ++i)
            acc = mfma_f32(ap[4 * i], wreg[i], acc);
#pragma unroll
        for (int v = 0; v < 4; ++v) pacc[wave][(4 * g + v) * 16 + r] = acc[v];
        __syncthreads();        // the partial products are in LDS
        if (tid < 256) {
            float part[4];
#pragma unroll
            for (int w = 0; w < 4; ++w) part[w] = (pacc[4 * w][tid] + pacc[4 * w + 1][tid]) + (pacc[4 * w + 2][tid] + pacc[4 * w + 3][tid]);
            const float sum = (part[0] + part[1]) + (part[2] + part[3]);
            const int orow = tile * 16 + (tid >> 4);
            if (orow < rows) (Y + (size_t)tile * 256)[lane_offset(tid)] = sum;
            yt[tid >> 4][tid & 15] = orow < rows ? sum : 0.f;
        }
        __syncthreads();        // the tile of Y is in LDS beside its residuals
        float y4[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) y4[k] = yt[4 * k + g][r];
        const float* tp = rt + g * ldr + 16 * (r >> 2) + (r & 3) + col_of(0);
        // (columns past the end reach their own results only)
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int i = 0; i < ND; ++i) macc[i] = mfma_f32(tp[4 * k * ldr + 256 * i], y4[k], macc[i]);
        if (wave == 15) {                   // (of the waves with the fewest tiles) entry (4 v + g, r) of the Gram matrix
            v4d ga;
#pragma unroll
            for (int v = 0; v < 4; ++v) ga[v] = gl[(4 * v + g) * 16 + r];
#pragma unroll
            for (int k = 0; k < 4; ++k) ga = __builtin_amdgcn_mfma_f64_16x16x4f64((double)y4[k], (double)y4[k], ga, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 4; ++v) gl[(4 * v + g) * 16 + r] = ga[v];
        }
    }
    __syncthreads();
    if (tid < 256) gpart[(size_t)blockIdx.x * 256 + tid] = gl[tid];
    float* const mp = mpart + (size_t)blockIdx.x * cols * 16;
#pragma unroll
    for (int i = 0; i < ND; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int c = col_of(i) + 16 * g + v;
            if (c < cols) mp[(size_t)c * 16 + r] = macc[i][v];
        }
}

}  // namespace

int quant_project_blocks(int rows) { return min(ceil_div(rows, 16), LRQ_QPR_MAX_BLOCKS); }

int launch_quant_project_rows(const float* X, int ldx, int rows, int cols, QuantParams q, const float* W, int LP, float* Y, double* gpart,
                              float* mpart, float* amax, float* lam_out, float* s_out, int8_t* codes, hipStream_t st) {
    if (!quant_sketch_rows_usable(X, ldx, rows, cols, LP, codes)) return LRQMM_ERR_UNSUPPORTED;
    const dim3 grid(quant_project_blocks(rows));
    const int nb = ceil_div(cols, 64);
    const size_t lds = (size_t)(16 * (64 * nb + 4) + 768) * sizeof(float);       // (and what the tiles past the last column read)
#define LRQ_QPR(NBV) case NBV: hipLaunchKernelGGL((quant_project_rows_kernel<NBV>), grid, dim3(1024), lds, st, X, ldx, rows, cols, q, W, Y, gpart, mpart, amax, lam_out, s_out, codes); break
    switch (nb) {
        LRQ_QPR(1); LRQ_QPR(2); LRQ_QPR(3); LRQ_QPR(4); LRQ_QPR(5); LRQ_QPR(6); LRQ_QPR(7); LRQ_QPR(8); LRQ_QPR(9);
        default: return LRQMM_ERR_UNSUPPORTED;
    }
#undef LRQ_QPR
    LRQ_CHECK_LAUNCH();
    return LRQMM_OK;
}
