// Internal helpers shared by the LRQMM HIP kernels (gfx950 only).
// Compiled with -ffp-contract=off: a*b+c is never fused implicitly; every FMA
// in this library is written as fmaf()/fma() on purpose.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));

#define LRQ_WAVE 64

static inline int ceil_div(int a, int b) { return (a + b - 1) / b; }
static inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Quantizer parameters of one call (Eq. (quantA)): qmax as float, clamp range, rounding mode.
struct QuantParams {
    float qmaxf;   // 2^(bits-1) - 1
    float lo;      // -qmax - 1
    float hi;      // qmax
    int round_mode;
};

static inline QuantParams make_quant_params(int bits, int round_mode) {
    QuantParams q;
    int qm = (1 << (bits - 1)) - 1;
    q.qmaxf = (float)qm;
    q.lo = (float)(-qm - 1);
    q.hi = (float)qm;
    q.round_mode = round_mode;
    return q;
}

// lambda = fl32(qmax / amax), s = fl32(amax / qmax); zero group when amax < 1e-30.
__device__ __forceinline__ void make_scales(float amax, float qmaxf, float& lam, float& s) {
    if (amax >= 1e-30f) {
        lam = qmaxf / amax;
        s = amax / qmaxf;
    } else {
        lam = 0.0f;
        s = 0.0f;
    }
}

// One instruction; lo for a NaN, as fminf(fmaxf(c, lo), hi) gives.
__device__ __forceinline__ float clamp_code(float c, const QuantParams& q) { return __builtin_amdgcn_fmed3f(c, q.lo, q.hi); }

// code = clamp(round(fl32(lambda * x))) as a float holding an integer value.
__device__ __forceinline__ float quant_code(float x, float lam, const QuantParams& q) {
    float t = x * lam;
    float c = (q.round_mode == 0) ? floorf(t) : rintf(t);
    return clamp_code(c, q);
}

// The same residual with the rounding mode fixed at compile time (callers branch once on
// q.round_mode around a block of these instead of selecting per element).
template <int ROUND_MODE>
__device__ __forceinline__ float quant_residual_m(float x, float lam, float s, const QuantParams& q) {
    const float t = x * lam;
    const float c = ROUND_MODE == 0 ? floorf(t) : rintf(t);
    return fmaf(-clamp_code(c, q), s, x);
}

// residual x - code * s with a single rounding.
__device__ __forceinline__ float quant_residual(float x, float lam, float s, const QuantParams& q) {
    float c = quant_code(x, lam, q);
    return fmaf(-c, s, x);
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}

// Four consecutive floats at any 4-byte boundary (rows of an odd stride leave no better alignment).
typedef float v4fu __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ float4 load4u(const float* __restrict__ p) {
    const v4fu t = *reinterpret_cast<const v4fu*>(p);
    return make_float4(t.x, t.y, t.z, t.w);
}
// Columns k .. k+3 of a row, zeros from `end` on (end > 0): four clamped loads, for the last chunk of a reduction.
__device__ __forceinline__ float4 load4_tail(const float* __restrict__ rowp, int k, int end) {
    float4 v;
    v.x = rowp[min(k + 0, end - 1)];
    v.y = rowp[min(k + 1, end - 1)];
    v.z = rowp[min(k + 2, end - 1)];
    v.w = rowp[min(k + 3, end - 1)];
    return make_float4(k + 0 < end ? v.x : 0.f, k + 1 < end ? v.y : 0.f, k + 2 < end ? v.z : 0.f, k + 3 < end ? v.w : 0.f);
}

// ---- float32 values as sums of bfloat16 planes (for the bf16 matrix cores) ----
// A float32 value is the exact sum of three bfloat16 planes (8 + 8 + 8 significant bits: round to nearest,
// subtract, repeat); products of such sums are evaluated plane by plane, each product exact, accumulated in
// float32 by the matrix core.
typedef __bf16 v8bf16 __attribute__((ext_vector_type(8)));
struct Planes3 {
    v8bf16 p1, p2, p3;
};
typedef __bf16 v2bf16 __attribute__((ext_vector_type(2)));
typedef float v2f32 __attribute__((ext_vector_type(2)));
// Two values per conversion instruction; a bfloat16 is the upper half of its float32, so the
// converted pair is widened again with a shift and a mask.
__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((v2f32){a, b}, v2bf16));
}
// PL planes are formed (1, 2 or 3); the members beyond PL stay unset and must not be used.
template <int PL = 3>
__device__ __forceinline__ Planes3 split_planes(const float (&r)[8]) {
    uint32_t w1[4], w2[4], w3[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float a = r[2 * e], b = r[2 * e + 1];
        const uint32_t h = pack_bf16x2(a, b);
        w1[e] = h;
        if (PL >= 2) {
            const float ra = a - __uint_as_float(h << 16);              // exact
            const float rb = b - __uint_as_float(h & 0xffff0000u);
            const uint32_t m = pack_bf16x2(ra, rb);
            w2[e] = m;
            if (PL >= 3) {
                const float ra2 = ra - __uint_as_float(m << 16);            // exact
                const float rb2 = rb - __uint_as_float(m & 0xffff0000u);
                w3[e] = pack_bf16x2(ra2, rb2);
            }
        }
    }
    typedef uint32_t v4u32 __attribute__((ext_vector_type(4)));
    Planes3 o;
    o.p1 = __builtin_bit_cast(v8bf16, (v4u32){w1[0], w1[1], w1[2], w1[3]});
    if (PL >= 2) o.p2 = __builtin_bit_cast(v8bf16, (v4u32){w2[0], w2[1], w2[2], w2[3]});
    if (PL >= 3) o.p3 = __builtin_bit_cast(v8bf16, (v4u32){w3[0], w3[1], w3[2], w3[3]});
    return o;
}

// The 16 code bytes k .. k+15 of a row of K from the 16 bytes at kc = min(k, K - 16), sh = k - kc: moved down by sh
// bytes, zeros above (all zeros from sh = 16 on).
__device__ __forceinline__ uint4 tail16(uint4 v, int sh) {
    uint64_t lo = (uint64_t)v.y << 32 | v.x, hi = (uint64_t)v.w << 32 | v.z;
    if (sh >= 8) { lo = hi; hi = 0; }
    const int b = 8 * (sh & 7);
    lo = (lo >> b) | ((hi << 1) << (63 - b));
    hi >>= b;
    if (sh >= 16) lo = hi = 0;
    return make_uint4((uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32));
}

// ---- packed codes: the order of the matrix cores' operands ----
// Inside a call codes travel as blocks that a wave loads whole, or copies to LDS as they are: [row block of 32][k block of 64]
// [pk_block bytes], a block being an operand of 32 rows and 64 k: lane l holds row l % 32, codes 32 (l / 32) .. +32 of the block.
// Codes past K are zero; rows past the end of a block hold anything.  Two formats:
//   PK8: bytes, 32 per lane: first the lanes' codes 0 .. 15, then 16 .. 31, two operands of v_mfma_i32_32x32x32_i8 (which takes the
//   k of a block in another order than the memory's, A and B alike).
//   PK6: codes of at most five bits.  The magnitudes 0 .. 16 are the first seventeen values of the six-bit e2m3 format in units of
//   1/8 (its subnormals and the first binades continue each other), so a code is exact in it, sign and magnitude, and so is a
//   product of two.  v_mfma_f32_32x32x64_f8f6f4 takes such operands at twice the rate of the int8 instructions, from 3/4 of the
//   bytes, and adds in float32, where integers are exact up to 2^24: the sums are the int8 matrix cores' sums (times 1/64).
//   Measured on random 4-bit codes, int8 from rows of codes / this: 4096^3 59 / 46 us, 16384^3 3.99 / 2.56 ms; operands in
//   registers, one probe of both, 2.4 / 5.0 POP/s (int8 with four waves a SIMD: 2.9).  24 bytes per lane (code e in bits 6 e ..): first the lanes' bytes 0 .. 15, then 16 .. 23.
// Both LDS reads of a wave are contiguous.
enum { PK_NONE = 0, PK6 = 6, PK8 = 8 };
#define PK_K 64
__host__ __device__ static constexpr int pk_block(int fmt) { return fmt == PK6 ? 1536 : 2048; }
__host__ __device__ static inline int pk_kblocks(int K) { return (K + PK_K - 1) / PK_K; }
static inline size_t pk_bytes(int rows, int K, int fmt) { return (size_t)((rows + 31) / 32) * pk_kblocks(K) * pk_block(fmt); }

// Sign and magnitude of a code that is given as a float.
__device__ __forceinline__ uint32_t six_bits(float c) { return (uint32_t)fabsf(c) | ((__float_as_uint(c) >> 26) & 32u); }
// Four codes in the low six bits of each byte -> 24 bits.
__device__ __forceinline__ uint32_t squeeze_six(uint32_t w) {
    const uint32_t t = (w & 0x003f003fu) | ((w >> 2) & 0x0fc00fc0u);
    return (t & 0xfffu) | ((t >> 4) & 0xfff000u);
}
// 32 codes as eight words of four (PK6: 24 bits each) -> a lane's part of block `blk`; valid: codes from this one on are zeroed.
template <int FMT>
__device__ __forceinline__ void store_packed(uint8_t* __restrict__ blk, int lane, uint32_t (&t)[8], int valid) {
    if (valid < 32) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int v = max(0, min(4, valid - 4 * j));
            t[j] &= v == 4 ? 0xffffffffu : (1u << (FMT * v)) - 1u;
        }
    }
    if (FMT == PK8) {
        *reinterpret_cast<uint4*>(blk + lane * 16) = make_uint4(t[0], t[1], t[2], t[3]);
        *reinterpret_cast<uint4*>(blk + 1024 + lane * 16) = make_uint4(t[4], t[5], t[6], t[7]);
        return;
    }
    *reinterpret_cast<uint4*>(blk + lane * 16) = make_uint4(t[0] | (t[1] << 24), (t[1] >> 8) | (t[2] << 16),
                                                            (t[2] >> 16) | (t[3] << 8), t[4] | (t[5] << 24));
    *reinterpret_cast<uint2*>(blk + 1024 + lane * 8) = make_uint2((t[5] >> 8) | (t[6] << 16), (t[6] >> 16) | (t[7] << 8));
}
// A tile of codes in LDS (TW rows of TL codes, stride TS bytes; PK6: a word of 24 bits per four codes, or BYTES of six) -> its
// blocks: row block r0 / 32, k block c0 / 64 on; a wave stores one block at a time.
template <int FMT, int TW, int TL, int TS, bool BYTES>
__device__ __forceinline__ void store_packed_tile(const int8_t* tile, uint8_t* __restrict__ codes, int r0, int rows, int c0, int K,
                                                  int tid, int threads) {
    const int nrb = (rows + 31) >> 5, nkb = pk_kblocks(K);
    for (int e = tid; e < TW * TL / 32; e += threads) {
        const int l = e & 63, b = e >> 6, rb = b % (TW / 32), cb = b / (TW / 32);
        if ((r0 >> 5) + rb >= nrb || (c0 >> 6) + cb >= nkb) continue;
        const int seg = 64 * cb + 32 * (l >> 5);
        const uint4* src = reinterpret_cast<const uint4*>(&tile[(32 * rb + (l & 31)) * TS + seg]);
        const uint4 lo = src[0], hi = src[1];
        uint32_t t[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
        if (FMT == PK6 && BYTES) {
#pragma unroll
            for (int j = 0; j < 8; ++j) t[j] = squeeze_six(t[j]);
        }
        store_packed<FMT>(codes + ((size_t)((r0 >> 5) + rb) * nkb + (c0 >> 6) + cb) * pk_block(FMT), l, t, K - c0 - seg);
    }
}

#define LRQ_CHECK_LAUNCH()                                   \
    do {                                                     \
        if (hipGetLastError() != hipSuccess) return LRQMM_ERR_HIP; \
    } while (0)
