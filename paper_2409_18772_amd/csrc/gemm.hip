// Integer GEMM on the int8 matrix cores with a fused dequantize + low-rank
// compensation epilogue (paper: Eq. (INTGEMM), Eq. (QUANTGEMM); Algorithm 2, integer product,
// dequantization and compensation steps).
//
// The three compensation terms of Algorithm 2 are never formed as M x N matrices:
//   RC1 + RC2 + RC3 = (U Sig)(Vt B~) + (A~ W)(Gam Zt) + (U Sig)(Vt W)(Gam Zt)
//                   = [U Sig | A~ W] . [Vt B~ + (Vt W) Gam Zt ; Gam Zt]
// i.e. a rank-2r update Lp . Rp^T applied to each output tile while its int32
// accumulators are still in registers.
//
// Main loop: up to 128x128 workgroup tile, 4 waves in 2x2, each wave up to 64x64 as 2x2
// v_mfma_i32_32x32x32_i8 tiles; both operands are K-major (A codes M x K, B codes
// stored transposed N x K), staged through double-buffered LDS with a padded row
// stride (144 B) that makes the 16-byte operand reads bank-conflict free.
// 32x32 accumulator layout (lane l, register v): row 8*(v/4) + 4*(l/32) + v%4,
// column l%32 -- identical for the i32 and f32 32x32 MFMAs, which lets the
// epilogue continue on the same registers with v_mfma_f32_32x32x2_f32.
#include <type_traits>
#include "kernels.h"

static inline bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

#define BBK 128                 // K depth of one staged tile
#define BSTRIDE (BBK + 16)      // padded LDS row stride, conflict-free 16-byte reads
#define GEMM_MIN_TILES 256      // of the smaller tiles: fewer, and the next smaller size is taken
#define GEMM_CUS 256            // compute units that one round of workgroups fills
#define PANEL_KC 32         // panel columns staged at a time as bfloat16 planes
#define PANEL_LD 40         // row stride of such a chunk of a plane (80 bytes: conflict-free 16-byte reads)

// 16 code bytes of one operand row, k .. k+15, zeros past K.  WIDE (K >= 16): one 16-byte load at any byte
// alignment (codes are packed rows of K bytes, so an odd K leaves none), branch free with a clamped address; the
// bytes are put in place by tail16 when the tile is written to LDS, and only in tiles that reach past K: nothing
// touches the loaded register before, so a ring of loads stays in flight.  Rows past the end re-read the last one:
// they only enter output rows (columns) that are never stored.
// Measured at 1537 x 1021 x 2311, 128 x 128 tiles: byte loads 347 us, 16-byte loads 36 us.
template <bool WIDE>
__device__ __forceinline__ uint4 load16b(const int8_t* __restrict__ rowp, int K, int k) {
    if (WIDE) {
        uint4 v;
        __builtin_memcpy(&v, rowp + min(k, K - 16), 16);
        return v;
    }
    uint32_t w[4] = {0u, 0u, 0u, 0u};       // K < 16: the whole row is one group
#pragma unroll
    for (int b = 0; b < 16; ++b)
        if (k + b < K) w[b >> 2] |= (uint32_t)(uint8_t)rowp[k + b] << (8 * (b & 3));
    return make_uint4(w[0], w[1], w[2], w[3]);
}
__device__ __forceinline__ const int8_t* code_row(const int8_t* __restrict__ base, int row, int nrows, int K) {
    return base + (size_t)min(row, nrows - 1) * K;
}

// A sum of code products as a float (sums on the fp6 matrix cores are in units of 1/64).
__device__ __forceinline__ float code_sum(int a) { return (float)a; }
__device__ __forceinline__ float code_sum(float a) { return a * 64.0f; }

// ---- main loop on packed codes (see PK8, PK6) ----
// A wave's 64 lanes copy 16 bytes each from global memory to 1 KB of LDS, without registers in between.
__device__ __forceinline__ void load_to_lds(uint32_t lds, const uint8_t* base, uint32_t off) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %1" ::"s"(lds), "s"(base), "v"(off) : "memory", "m0");
}
typedef int v8i __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) uint8_t lds_u8;
// Sums of a 32 x 32 tile: int32, or float32 in units of 1/64 (exact either way).
template <int FMT> using PackedSum = std::conditional_t<FMT == PK6, v16f, v16i>;

template <int H>
__device__ __forceinline__ v4i half(const v8i& v) { return __builtin_shufflevector(v, v, 4 * H, 4 * H + 1, 4 * H + 2, 4 * H + 3); }

// acc += the tile's products over nk k blocks from kb0 on.  The tile is BA row blocks of A (from ra0) by BB of B (from rb0), a wave
// MT x NT of them (from wa, wb inside the tile); ST stages of LDS hold one k block of the tile each.  The copies of ST - 3 k
// blocks are in flight while the matrix cores work on one and the next one's operands are read from LDS to registers, so a step
// is one barrier and no wait for LDS or memory; an even share of 1 KB pieces per wave, the last ones twice where they do not
// divide.  Row and k blocks past the end: the last one again.  At 16384^3 it reaches 3.4 POP/s of the 5.0 of operands in
// registers (one k block ahead instead of its operands, 128-deep stages: 3.35); with operand bits that do not change 4.1, so
// it is the power that bounds it.
template <int FMT, int MT, int NT, int BA, int BB, int NW, int ST, bool STACK = false>
__device__ __forceinline__ void packed_products(const uint8_t* __restrict__ A, const uint8_t* __restrict__ B, int ra0, int nra, int rb0,
                                                int nrb, int nkb, int kb0, int nk, uint8_t* sm, int wave, int lane, int wa, int wb,
                                                PackedSum<FMT> (&acc)[MT][NT], const uint8_t* __restrict__ A1 = nullptr,
                                                const uint8_t* __restrict__ B1 = nullptr) {
    constexpr int PK_BLOCK = pk_block(FMT);
    constexpr int STAGE = (BA + BB) * PK_BLOCK, PIECES = STAGE / 1024, PER = (PIECES + NW - 1) / NW;
    static_assert(STAGE % 1024 == 0 && BA * PK_BLOCK % 1024 == 0, "pieces belong to one operand");
    const size_t rowb = (size_t)nkb * PK_BLOCK;
    const uint8_t* src[PER];
    uint32_t off[PER], dst[PER];
    const uint32_t base = (uint32_t)(uintptr_t)(lds_u8*)sm;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int piece = min(wave * PER + u, PIECES - 1);
        const bool isb = piece >= BA * PK_BLOCK / 1024;
        int pi = piece - (isb ? BA * PK_BLOCK / 1024 : 0);
        const uint8_t* operand = isb ? B : A;
        if constexpr (STACK) {
            const int h = (isb ? BB : BA) / 2 * PK_BLOCK / 1024;
            if (pi >= h) { pi -= h; operand = isb ? B1 : A1; }
        }
        const int at = pi * 1024 + lane * 16, r = at / PK_BLOCK;
        src[u] = operand + (size_t)(isb ? rb0 : ra0) * rowb + (size_t)kb0 * PK_BLOCK;
        off[u] = (uint32_t)(min(r, (isb ? nrb - rb0 : nra - ra0) - 1) * rowb) + at % PK_BLOCK;
        dst[u] = base + piece * 1024;
    }
    auto issue = [&](int t, int s) {
        const size_t o = (size_t)min(t, nk - 1) * PK_BLOCK;
#pragma unroll
        for (int u = 0; u < PER; ++u) load_to_lds(dst[u] + s * STAGE, src[u] + o, off[u]);
    };
    struct Frag { v8i a[MT], b[NT]; };
    auto operand = [&](const uint8_t* p) {
        const v4i lo = *reinterpret_cast<const v4i*>(p + lane * 16);
        if constexpr (FMT == PK8) {
            const v4i h4 = *reinterpret_cast<const v4i*>(p + 1024 + lane * 16);
            return (v8i){lo.x, lo.y, lo.z, lo.w, h4.x, h4.y, h4.z, h4.w};
        }
        const int2 hi = *reinterpret_cast<const int2*>(p + 1024 + lane * 8);
        return (v8i){lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, 0, 0};
    };
    auto fetch = [&](Frag& f, int s) {
        const uint8_t* const p = sm + s * STAGE;
#pragma unroll
        for (int m = 0; m < MT; ++m) f.a[m] = operand(p + (wa + m) * PK_BLOCK);
#pragma unroll
        for (int n = 0; n < NT; ++n) f.b[n] = operand(p + (BA + wb + n) * PK_BLOCK);
    };
#pragma unroll
    for (int t = 0; t < ST - 1; ++t) issue(t, t);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PER * (ST - 2)) : "memory");       // this wave's pieces of block 0
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    Frag f0, f1;
    fetch(f0, 0);
    int s = 0;
    // block i is in `cur`; i + 1 has landed, and nobody reads stage i - 1 any more, behind the barrier
    auto step = [&](Frag& cur, Frag& nxt, int i) {
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PER * (ST - 3)) : "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        const int prev = s == 0 ? ST - 1 : s - 1, next = s + 1 == ST ? 0 : s + 1;
        issue(i + ST - 1, prev);
        fetch(nxt, next);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                if constexpr (FMT == PK6)       // (2: e2m3 operands; scales of 1)
                    acc[m][n] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(cur.a[m], cur.b[n], acc[m][n], 2, 2, 0, 0, 0, 0);
                else
                    acc[m][n] = __builtin_amdgcn_mfma_i32_32x32x32_i8(half<0>(cur.a[m]), half<0>(cur.b[n]), acc[m][n], 0, 0, 0);
            }
        if constexpr (FMT == PK8) {
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int n = 0; n < NT; ++n)
                    acc[m][n] = __builtin_amdgcn_mfma_i32_32x32x32_i8(half<1>(cur.a[m]), half<1>(cur.b[n]), acc[m][n], 0, 0, 0);
        }
        __builtin_amdgcn_s_setprio(0);
        __builtin_amdgcn_sched_barrier(0);
        s = next;
    };
    for (int i = 0; i < nk; i += 2) {
        step(f0, f1, i);
        if (i + 1 < nk) step(f1, f0, i + 1);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // (copies past the end, too)
    __syncthreads();
}

// Step of a group from its maximum (the quantizer's).
__device__ __forceinline__ float step_of(float amax, float qmaxf) {
    float l, s;
    make_scales(amax, qmaxf, l, s);
    return s;
}

// Columns c .. c + 7 of a panel row, zeros from R2P on, as three bfloat16 planes to dst, dst + plane and dst + 2 plane.
__device__ __forceinline__ void stage_planes(const float* __restrict__ row, int c, int R2P, uint16_t* dst, int plane) {
    float v[8];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int col = c + 4 * h;
        const bool in = col < R2P;
        const float4 x = *reinterpret_cast<const float4*>(row + min(col, R2P - 4));
        v[4 * h + 0] = in ? x.x : 0.f; v[4 * h + 1] = in ? x.y : 0.f;
        v[4 * h + 2] = in ? x.z : 0.f; v[4 * h + 3] = in ? x.w : 0.f;
    }
    const Planes3 pl = split_planes<3>(v);
    *reinterpret_cast<v8bf16*>(dst) = pl.p1;
    *reinterpret_cast<v8bf16*>(dst + plane) = pl.p2;
    *reinterpret_cast<v8bf16*>(dst + 2 * plane) = pl.p3;
}

// Last step of Algorithm 2 on one element: D <- alpha * value + beta * D (D is not read when
// beta == 0, so it may then hold anything).
__device__ __forceinline__ void store_out(const GemmOut& out, int row, int col, float value) {
    float* p = out.C + (size_t)row * out.ldc + col;
    float o = out.alpha * value;
    if (out.beta != 0.f) o = o + out.beta * *p;
    *p = o;
}

// Workgroup ids are dealt round-robin to the 8 XCDs, each with an L2 of its own.  The tile grid
// is cut into gm x gn = 8 rectangles, one per XCD, as square as the tile counts allow, so that an
// XCD fetches tiles_m/gm row panels of A and tiles_n/gn of B instead of whole bands (at 16 x 16
// tiles: 8 + 4 panels per XCD instead of 2 + 16).  Tile counts that are no multiple of 8 keep
// the launch order.
__device__ __forceinline__ int xcd_tile(int id, int tiles_n, int ntiles) {
    if (ntiles & 7) return id;
    const int tiles_m = ntiles / tiles_n;
    int gm = 0, best = 0x7fffffff;
#pragma unroll
    for (int g = 1; g <= 8; g *= 2) {
        const int h = 8 / g;
        if (tiles_m % g == 0 && tiles_n % h == 0) {
            const int cost = tiles_m / g + tiles_n / h;
            if (cost < best) { best = cost; gm = g; }
        }
    }
    // ntiles % 8 == 0 guarantees that one of the four cuts divides both tile counts
    const int gn = 8 / gm, bn = tiles_n / gn, bm = tiles_m / gm;
    const int x = id & 7, j = id >> 3;
    // Inside its rectangle an XCD works through sub-blocks of 32 tiles (one per CU, the tiles that run at the
    // same time), 4 x 8 or 8 x 4 where the rectangle allows: the panels that one round of tiles streams through
    // the L2 are then 12 instead of bn + 32 / bn.
    int r = j / bn, c = j % bn;
    if (bm * bn > 32) {
        const int sm = (bm % 4 == 0 && bn % 8 == 0) ? 4 : ((bm % 8 == 0 && bn % 4 == 0) ? 8 : 0);
        if (sm) {
            const int sn = 32 / sm, sub = j >> 5, in = j & 31, per_row = bn / sn;
            r = (sub / per_row) * sm + in / sn;
            c = (sub % per_row) * sn + in % sn;
        }
    }
    return ((x / gn) * bm + r) * tiles_n + (x % gn) * bn + c;
}

// MTW, NTW: 32 x 32 MFMA tiles per wave along M and N; the four waves form a 2 x 2 grid, so the workgroup tile is
// 64 MTW x 64 NTW: 128 x 128; 64 x 64 for outputs of at most 64 columns, e.g. a convolution with 64 output channels as a
// product -- on a 128-wide tile half the matrix-core work and half of B's LDS tile would be zeros; 64 x 128 and 64 x 64 where
// the larger tiles are too few to fill the chip (see launch_int8_gemm).
//
// K tiles are 128 deep, global loads two of them ahead of the matrix cores in a ring of two sets of named registers (as arrays
// they would go to scratch memory).  The epilogue's operands travel beside the K loop: the steps are in LDS before it starts,
// the first 32 panel columns of the tile's rows in registers; each further 32 are loaded while the matrix cores take the ones
// before, in two buffers of the LDS that the operand tiles have left.  lrqmm_gemm, us, 64-deep tiles with panels straight from
// global memory / 128-deep with 64 columns at a time loaded behind the K loop / this: 2048^3 rank 48 74.6 / 72.8 / 65.0; 512 x
// 4096 x 4096 rank 16 50.1 / 45.9 / 43.8; 4096 x 2048 x 2048 rank 80 186 / 134 / 123; short reductions, where the load latency
// of the epilogue shows most, 128 x 8192 x 576 rank 80 85.3 / 88.8 / 82.1, 1024 x 1024 x 576 rank 48 45.8 / 47.5 / 43.7,
// 100352 x 64 x 64 rank 8 33.7 / 34.1 / 31.7, 100352 x 16 x 16 31.5 / 32.7 / 30.4.
// PACKED: the format of packed codes, or PK_NONE for rows of bytes; the same tiles and epilogue.
template <bool WIDE, bool COMP, bool WCINT, int MTW, int NTW, int PACKED>
__global__ __launch_bounds__(256, 2) void int8_gemm_kernel(int M, int N, int K,
                                                           const int8_t* __restrict__ Aq,
                                                           const int8_t* __restrict__ BqT,
                                                           const float* __restrict__ sA,
                                                           const float* __restrict__ sB,
                                                           const float* __restrict__ Lp,
                                                           const float* __restrict__ Rp, int R2P,
                                                           GemmOut out,
                                                           int32_t* __restrict__ Cint, int tiles_n,
                                                           int ntiles, float qmaxf) {
    constexpr int TMW = 64 * MTW, TNW = 64 * NTW;       // tile height and width
    constexpr int ST = PACKED == PK8 && MTW + NTW == 4 ? 4 : 6;     // stages of packed codes (two workgroups share a CU's LDS)
    constexpr int LDP = 36;             // row stride of a panel chunk (conflict-free 16-byte reads)
    constexpr int OPERAND_LDS = PACKED ? ST * (2 * MTW + 2 * NTW) * pk_block(PACKED) : 2 * (TMW + TNW) * BSTRIDE;
    constexpr int PANEL_LDS = 2 * (TMW + TNW) * LDP * 4;            // two chunks of the panel rows, in the operand tiles' LDS
    constexpr int TILE_LDS = OPERAND_LDS > PANEL_LDS ? OPERAND_LDS : PANEL_LDS;
    __shared__ __align__(16) int8_t tiles[TILE_LDS];
    int8_t* const As[2] = {tiles, tiles + TMW * BSTRIDE};
    int8_t* const Bs[2] = {tiles + 2 * TMW * BSTRIDE, tiles + (2 * TMW + TNW) * BSTRIDE};
    __shared__ __align__(16) float steps[TMW + TNW];    // of the tile's rows, then of its columns
    const int tile = xcd_tile(blockIdx.x, tiles_n, ntiles);
    const int m0 = (tile / tiles_n) * TMW, n0 = (tile % tiles_n) * TNW;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int wm = wave >> 1, wn = wave & 1;
    const int l32 = lane & 31, lh = lane >> 5;

    PackedSum<PACKED> acc[MTW][NTW];
#pragma unroll
    for (int a = 0; a < MTW; ++a)
#pragma unroll
        for (int b = 0; b < NTW; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0;

    // staging: two 16-byte chunks per 64 rows of an operand tile and thread; tiles past the end load zeros or the row's last
    // codes and are never stored
    const int srow0 = tid >> 3, skc = (tid & 7) * 16;
#define LRQ_DECL(S) uint4 S##a0, S##a1, S##a2, S##a3, S##b0, S##b1, S##b2, S##b3
    const int8_t *pa[2 * MTW], *pb[2 * NTW];
#pragma unroll
    for (int u = 0; u < 2 * MTW; ++u) pa[u] = PACKED ? nullptr : code_row(Aq, m0 + srow0 + 32 * u, M, K);
#pragma unroll
    for (int u = 0; u < 2 * NTW; ++u) pb[u] = PACKED ? nullptr : code_row(BqT, n0 + srow0 + 32 * u, N, K);
#define LRQ_LD(P, k0) load16b<WIDE>(P, K, (k0) + skc)
#define LRQ_GLOAD(S, k0)                                                                               \
    S##a0 = LRQ_LD(pa[0], k0); S##b0 = LRQ_LD(pb[0], k0); S##a1 = LRQ_LD(pa[1], k0); S##b1 = LRQ_LD(pb[1], k0); \
    if constexpr (MTW == 2) { S##a2 = LRQ_LD(pa[2], k0); S##a3 = LRQ_LD(pa[3], k0); }                   \
    if constexpr (NTW == 2) { S##b2 = LRQ_LD(pb[2], k0); S##b3 = LRQ_LD(pb[3], k0); }
    // (k0: first column of the set's tile; the branch is the same for the whole workgroup)
#define LRQ_ST(BUF, U, V) *reinterpret_cast<uint4*>(&BUF[(srow0 + 32 * U) * BSTRIDE + skc]) = V
#define LRQ_SSTORE(S, buf, k0)                                                                         \
    if (WIDE && (k0) + BBK > K) {                                                                      \
        const int sh = max(0, (k0) + skc - (K - 16));                                                  \
        S##a0 = tail16(S##a0, sh); S##a1 = tail16(S##a1, sh); S##b0 = tail16(S##b0, sh); S##b1 = tail16(S##b1, sh); \
        if constexpr (MTW == 2) { S##a2 = tail16(S##a2, sh); S##a3 = tail16(S##a3, sh); }               \
        if constexpr (NTW == 2) { S##b2 = tail16(S##b2, sh); S##b3 = tail16(S##b3, sh); }               \
    }                                                                                                  \
    LRQ_ST(As[buf], 0, S##a0); LRQ_ST(Bs[buf], 0, S##b0); LRQ_ST(As[buf], 1, S##a1); LRQ_ST(Bs[buf], 1, S##b1); \
    if constexpr (MTW == 2) { LRQ_ST(As[buf], 2, S##a2); LRQ_ST(As[buf], 3, S##a3); }                   \
    if constexpr (NTW == 2) { LRQ_ST(Bs[buf], 2, S##b2); LRQ_ST(Bs[buf], 3, S##b3); }
    // panel rows of the tile, 32 columns at a time: rows past the end re-read the last one, columns past it the last four
    const int prow = tid >> 3, pcol = (tid & 7) * 4;
    float4 q0, q1, q2, q3, q4, q5, q6, q7;
#define LRQ_PL(U, c) *reinterpret_cast<const float4*>(32 * U < TMW ? Lp + (size_t)min(m0 + prow + 32 * U, M - 1) * R2P + c \
                                                                   : Rp + (size_t)min(n0 + prow + 32 * U - TMW, N - 1) * R2P + c)
#define LRQ_PLOAD(t0)                                                                                  \
    {                                                                                                  \
        const int c = min((t0) + pcol, R2P - 4);                                                       \
        q0 = LRQ_PL(0, c); q1 = LRQ_PL(1, c); q2 = LRQ_PL(2, c); q3 = LRQ_PL(3, c);                    \
        if constexpr (MTW + NTW > 2) { q4 = LRQ_PL(4, c); q5 = LRQ_PL(5, c); }                         \
        if constexpr (MTW + NTW > 3) { q6 = LRQ_PL(6, c); q7 = LRQ_PL(7, c); }                         \
    }
#define LRQ_PST(U) *reinterpret_cast<float4*>((32 * U < TMW ? Ls + (prow + 32 * U) * LDP : Rs + (prow + 32 * U - TMW) * LDP) + pcol) = q##U
    // (without panels sA, sB hold the group maxima, and the tile's steps are formed here)
    float st = 0.f;
    if (tid < TMW) st = sA[min(m0 + tid, M - 1)];
    else if (tid - TMW < TNW) st = sB[min(n0 + tid - TMW, N - 1)];
    if constexpr (PACKED != PK_NONE) {
        if constexpr (COMP) LRQ_PLOAD(0);
        if (tid < TMW + TNW) steps[tid] = COMP ? st : step_of(st, qmaxf);
        packed_products<PACKED, MTW, NTW, 2 * MTW, 2 * NTW, 4, ST>(reinterpret_cast<const uint8_t*>(Aq), reinterpret_cast<const uint8_t*>(BqT),
                                                           m0 >> 5, (M + 31) >> 5, n0 >> 5, (N + 31) >> 5, pk_kblocks(K), 0,
                                                           pk_kblocks(K), reinterpret_cast<uint8_t*>(tiles), wave, lane, wm * MTW,
                                                           wn * NTW, acc);
    } else {
    LRQ_DECL(r0);
    LRQ_DECL(r1);
    auto compute = [&](int buf) {
#pragma unroll
        for (int kk = 0; kk < BBK / 32; ++kk) {
            v4i af[MTW], bf[NTW];
#pragma unroll
            for (int mt = 0; mt < MTW; ++mt)
                af[mt] = *reinterpret_cast<const v4i*>(
                    &As[buf][(wm * 32 * MTW + mt * 32 + l32) * BSTRIDE + kk * 32 + lh * 16]);
#pragma unroll
            for (int nt = 0; nt < NTW; ++nt)
                bf[nt] = *reinterpret_cast<const v4i*>(
                    &Bs[buf][(wn * 32 * NTW + nt * 32 + l32) * BSTRIDE + kk * 32 + lh * 16]);
#pragma unroll
            for (int mt = 0; mt < MTW; ++mt)
#pragma unroll
                for (int nt = 0; nt < NTW; ++nt)
                    acc[mt][nt] = __builtin_amdgcn_mfma_i32_32x32x32_i8(af[mt], bf[nt], acc[mt][nt], 0, 0, 0);
        }
    };
    const int nk = (K + BBK - 1) / BBK;
    LRQ_GLOAD(r0, 0);
    LRQ_GLOAD(r1, BBK);
    if constexpr (COMP) LRQ_PLOAD(0);
    if (tid < TMW + TNW) steps[tid] = COMP ? st : step_of(st, qmaxf);
    LRQ_SSTORE(r0, 0, 0);
    __syncthreads();
    // iteration i: the set that held tile i is free -> load tile i + 2; compute tile i; publish tile i + 1
#define LRQ_GEMM_STEP(J, SCUR, SNEXT)                                  \
    if (kt + J < nk) {                                                 \
        const int i = kt + J;                                          \
        LRQ_GLOAD(SCUR, (i + 2) * BBK);                                \
        compute(J);                                                    \
        if (i + 1 < nk) { LRQ_SSTORE(SNEXT, 1 - J, (i + 1) * BBK); }   \
        __syncthreads();                                               \
    }
    for (int kt = 0; kt < nk; kt += 2) {
        LRQ_GEMM_STEP(0, r0, r1)
        LRQ_GEMM_STEP(1, r1, r0)
    }
    }
#undef LRQ_GEMM_STEP
#undef LRQ_DECL
#undef LRQ_GLOAD
#undef LRQ_LD
#undef LRQ_ST
#undef LRQ_SSTORE

    // ---- epilogue: dequantize, rank-2r update, store ----
    v16f f[MTW][NTW];
#pragma unroll
    for (int mt = 0; mt < MTW; ++mt) {
        const int rbase = m0 + wm * 32 * MTW + mt * 32;
        float sa[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int row = rbase + 8 * (v >> 2) + 4 * lh + (v & 3);
            sa[v] = steps[row - m0];
        }
#pragma unroll
        for (int nt = 0; nt < NTW; ++nt) {
            const int col = n0 + wn * 32 * NTW + nt * 32 + l32;
            const float sb = steps[TMW + col - n0];
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = rbase + 8 * (v >> 2) + 4 * lh + (v & 3);
                if (WCINT && row < M && col < N) Cint[(size_t)row * N + col] = (int32_t)code_sum(acc[mt][nt][v]);
                f[mt][nt][v] = (code_sum(acc[mt][nt][v]) * sa[v]) * sb;
            }
        }
    }
    if constexpr (COMP) {
        // two buffers of 32 columns in the operand tiles' LDS (the K loop's last barrier has released it)
        for (int t0 = 0, buf = 0; t0 < R2P; t0 += 32, buf ^= 1) {
            float* const Ls = reinterpret_cast<float*>(tiles) + buf * ((TMW + TNW) * LDP);
            float* const Rs = Ls + TMW * LDP;
            LRQ_PST(0); LRQ_PST(1); LRQ_PST(2); LRQ_PST(3);
            if constexpr (MTW + NTW > 2) { LRQ_PST(4); LRQ_PST(5); }
            if constexpr (MTW + NTW > 3) { LRQ_PST(6); LRQ_PST(7); }
            if (t0 + 32 < R2P) LRQ_PLOAD(t0 + 32);
            __syncthreads();
            const float* const lp = Ls + (wm * 32 * MTW + l32) * LDP + 4 * lh;
            const float* const rp = Rs + (wn * 32 * NTW + l32) * LDP + 4 * lh;
            const int width = min(R2P - t0, 32);
            for (int t = 0; t < width; t += 8) {       // (R2P % 8 == 0)
                float4 a4[MTW], b4[NTW];
#pragma unroll
                for (int mt = 0; mt < MTW; ++mt) a4[mt] = *reinterpret_cast<const float4*>(lp + 32 * mt * LDP + t);
#pragma unroll
                for (int nt = 0; nt < NTW; ++nt) b4[nt] = *reinterpret_cast<const float4*>(rp + 32 * nt * LDP + t);
#define LRQ_FM(E)                                                                                       \
    _Pragma("unroll") for (int mt = 0; mt < MTW; ++mt) _Pragma("unroll") for (int nt = 0; nt < NTW; ++nt) \
        f[mt][nt] = __builtin_amdgcn_mfma_f32_32x32x2f32(a4[mt].E, b4[nt].E, f[mt][nt], 0, 0, 0);
                LRQ_FM(x)
                LRQ_FM(y)
                LRQ_FM(z)
                LRQ_FM(w)
#undef LRQ_FM
            }
        }
    }
#undef LRQ_PL
#undef LRQ_PLOAD
#undef LRQ_PST
#pragma unroll
    for (int mt = 0; mt < MTW; ++mt)
#pragma unroll
        for (int nt = 0; nt < NTW; ++nt) {
            const int col = n0 + wn * 32 * NTW + nt * 32 + l32;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = m0 + wm * 32 * MTW + mt * 32 + 8 * (v >> 2) + 4 * lh + (v & 3);
                if (row < M && col < N) store_out(out, row, col, f[mt][nt][v]);
            }
        }
}

// Large-tile variant for big problems: 256x256 workgroup tile, one workgroup of 8 waves per
// CU (two waves per SIMD, so one wave's LDS/global waits and barrier stalls are covered by
// the other's MFMAs).  Waves form a 4x2 grid, each 64x128 = 2x4 MFMA tiles (128 accumulator
// registers); per 32-deep MFMA step a wave reads 6 KB of operands from LDS for 8 MFMAs.  A staged
// tile is 128 deep: 144 KB of LDS for the two buffers of both operands.
#define BTM 256
#define BTN 256
#define BCHUNKS (BBK / 16)      // 16-byte chunks per staged row
#define BROWS (512 / BCHUNKS)   // rows covered by one pass of the 512 threads
#define LARGE_LDS (2 * BTM * BSTRIDE)       // of each operand's tiles, reused by the epilogue
struct LargeTile {
    int M, N, m0, n0;
    const float *sA, *sB, *Lp, *Rp;
    int R2P;
    GemmOut out;
    int32_t *Cint, *part;       // part: of a workgroup that holds one range of K (partial)
    bool partial;
    float qmaxf;
};
__device__ __forceinline__ int32_t raw_sum(int a) { return a; }
__device__ __forceinline__ int32_t raw_sum(float a) { return (int32_t)(a * 64.0f); }

// What follows the products of a large tile (v16i sums of bytes, v16f of packed codes).  The tiles' LDS is free.
template <bool COMP, bool WCINT, bool SPLITK, class ACC>
__device__ __forceinline__ void finish_large_tile(const LargeTile& T, ACC (&acc)[2][4], int8_t* ldsA, int8_t* ldsB) {
    const int M = T.M, N = T.N, m0 = T.m0, n0 = T.n0, R2P = T.R2P;
    const float *__restrict__ const sA = T.sA, *__restrict__ const sB = T.sB;
    const float *__restrict__ const Lp = T.Lp, *__restrict__ const Rp = T.Rp;
    const GemmOut& out = T.out;
    float* __restrict__ const C = out.C;
    int32_t *__restrict__ const Cint = T.Cint, *__restrict__ const part = T.part;
    const bool partial = T.partial;
    const float qmaxf = T.qmaxf;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int wm = wave >> 1, wn = wave & 1;
    const int l32 = lane & 31, lh = lane >> 5;
    // ---- epilogue: dequantize, rank-2r update, store ----
    // C == nullptr: only the raw int32 sums are wanted (the dequantization and the update then
    // run later, in rank_update_kernel), and the step vectors are not read.
    const bool want_c = C != nullptr;
    // Without panels sA, sB hold the group maxima, and the tile's steps are formed here, one per thread, in the LDS that the
    // operand tiles have left: a launch that prepared them took 5 us of a call at 4096^3.
    float* const sAl = reinterpret_cast<float*>(ldsA);
    float* const sBl = reinterpret_cast<float*>(ldsB);
    if (!COMP && want_c) {
        if (tid < BTM) sAl[tid] = step_of(sA[min(m0 + tid, M - 1)], qmaxf);
        else sBl[tid - BTM] = step_of(sB[min(n0 + tid - BTM, N - 1)], qmaxf);
        __syncthreads();
    }
    // Wider panels: the float32 matrix cores would take 4 R2P M N flops at 1/16 of the bfloat16 rate, so the tile's panel rows
    // are split into three bfloat16 planes while they are staged (32 columns at a time, in the LDS that the operand tiles have
    // left) and the six plane products of weight >= 2^-16 run on v_mfma_f32_32x32x16_bf16, as in rank_update_bf16_kernel.
    if (COMP && R2P > 64) {
        uint16_t* const Lq = reinterpret_cast<uint16_t*>(ldsA);
        uint16_t* const Rq = reinterpret_cast<uint16_t*>(ldsB);
        constexpr int PL = 256 * PANEL_LD;          // one plane
        static_assert(LARGE_LDS >= 3 * PL * 2, "three planes of a 32-column chunk fit an operand's LDS");
        v16f f[2][4];
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) {
            const int rbase = m0 + wm * 64 + mt * 32;
            float sa[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = rbase + 8 * (v >> 2) + 4 * lh + (v & 3);
                sa[v] = row < M ? sA[row] : 0.f;
            }
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) {
                const int col = n0 + wn * 128 + nt * 32 + l32;
                const float sb = col < N ? sB[col] : 0.f;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int row = rbase + 8 * (v >> 2) + 4 * lh + (v & 3);
                    if (WCINT && row < M && col < N) Cint[(size_t)row * N + col] = raw_sum(acc[mt][nt][v]);
                    f[mt][nt][v] = (code_sum(acc[mt][nt][v]) * sa[v]) * sb;
                }
            }
        }
        for (int t0 = 0; t0 < R2P; t0 += PANEL_KC) {
            __syncthreads();            // nobody reads the operand tiles, or the previous chunk, any more
            // 2 panels x 256 rows x 4 groups of 8 columns, four units per thread
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int unit = tid + 512 * i, r = (unit >> 2) & 255, c8 = (unit & 3) * 8;
                const bool left = i < 2;
                // rows / columns past the end re-read the last one (rows are never stored, columns enter as zeros)
                const float* src = left ? Lp + (size_t)min(m0 + r, M - 1) * R2P : Rp + (size_t)min(n0 + r, N - 1) * R2P;
                stage_planes(src, t0 + c8, R2P, (left ? Lq : Rq) + r * PANEL_LD + c8, PL);
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                v8bf16 a[2][3];
#pragma unroll
                for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                    for (int q = 0; q < 3; ++q)
                        a[mt][q] = *reinterpret_cast<const v8bf16*>(Lq + q * PL + (wm * 64 + mt * 32 + l32) * PANEL_LD + 16 * u + 8 * lh);
#pragma unroll
                for (int nt = 0; nt < 4; ++nt) {
                    v8bf16 b[3];
#pragma unroll
                    for (int q = 0; q < 3; ++q)
                        b[q] = *reinterpret_cast<const v8bf16*>(Rq + q * PL + (wn * 128 + nt * 32 + l32) * PANEL_LD + 16 * u + 8 * lh);
                    // smallest products first; the two row tiles are independent chains
#define LRQ_PP(QA, QB)                                                                                          \
    _Pragma("unroll") for (int mt = 0; mt < 2; ++mt) f[mt][nt] =                                                \
        __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[mt][QA], b[QB], f[mt][nt], 0, 0, 0);
                    LRQ_PP(0, 2)
                    LRQ_PP(1, 1)
                    LRQ_PP(2, 0)
                    LRQ_PP(0, 1)
                    LRQ_PP(1, 0)
                    LRQ_PP(0, 0)
#undef LRQ_PP
                }
            }
        }
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) {
                const int col = n0 + wn * 128 + nt * 32 + l32;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int row = m0 + wm * 64 + mt * 32 + 8 * (v >> 2) + 4 * lh + (v & 3);
                    if (row < M && col < N) store_out(out, row, col, f[mt][nt][v]);
                }
            }
        return;
    }
    // Panels of up to 64 columns: the tile's 256 rows of Lp and of Rp are staged in the LDS that the operand
    // tiles have left (whole-row loads; rows past the end as zeros; row stride R2P + 4 floats: conflict-free
    // 16-byte reads), instead of 32 cache lines per load instruction from global memory.  Same values, same
    // order of the products.
    const int LDP = R2P + 4;
    float* const Ls = reinterpret_cast<float*>(ldsA);
    float* const Rs = reinterpret_cast<float*>(ldsB);
    static_assert(LARGE_LDS >= 256 * 68 * 4 && BTM + BTN == 512, "a 64-column panel tile fits an operand's LDS");
    if (COMP) {
        __syncthreads();        // every wave has read its last operand fragments
        const int q4 = R2P / 4;
        for (int idx = tid; idx < 256 * q4; idx += 512) {
            const int rr = idx / q4, c4 = idx - rr * q4;
            const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
            const float4 lv = m0 + rr < M ? *reinterpret_cast<const float4*>(Lp + (size_t)(m0 + rr) * R2P + 4 * c4) : z;
            const float4 rv = n0 + rr < N ? *reinterpret_cast<const float4*>(Rp + (size_t)(n0 + rr) * R2P + 4 * c4) : z;
            *reinterpret_cast<float4*>(Ls + rr * LDP + 4 * c4) = lv;
            *reinterpret_cast<float4*>(Rs + rr * LDP + 4 * c4) = rv;
        }
        __syncthreads();
    }
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
        const int rbase = m0 + wm * 64 + mt * 32;
        const float* lps = Ls + (wm * 64 + mt * 32 + l32) * LDP + 4 * lh;
        float sa[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int row = rbase + 8 * (v >> 2) + 4 * lh + (v & 3);
            sa[v] = !want_c ? 0.f : (COMP ? sA[min(row, M - 1)] : sAl[row - m0]);
        }
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            const int col = n0 + wn * 128 + nt * 32 + l32;
            const bool col_ok = col < N;
            const float sb = !want_c ? 0.f : (COMP ? sB[min(col, N - 1)] : sBl[col - n0]);
            v16f f;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = rbase + 8 * (v >> 2) + 4 * lh + (v & 3);
                if (WCINT && row < M && col_ok) {
                    if (SPLITK && partial) part[(row - m0) * BTN + (col - n0)] = raw_sum(acc[mt][nt][v]);
                    else Cint[(size_t)row * N + col] = raw_sum(acc[mt][nt][v]);
                }
                f[v] = (code_sum(acc[mt][nt][v]) * sa[v]) * sb;
            }
            if (COMP) {
                const float* rps = Rs + (wn * 128 + nt * 32 + l32) * LDP + 4 * lh;
                for (int t0 = 0; t0 < R2P; t0 += 8) {
                    const float4 a4 = *reinterpret_cast<const float4*>(lps + t0);
                    const float4 b4 = *reinterpret_cast<const float4*>(rps + t0);
                    f = __builtin_amdgcn_mfma_f32_32x32x2f32(a4.x, b4.x, f, 0, 0, 0);
                    f = __builtin_amdgcn_mfma_f32_32x32x2f32(a4.y, b4.y, f, 0, 0, 0);
                    f = __builtin_amdgcn_mfma_f32_32x32x2f32(a4.z, b4.z, f, 0, 0, 0);
                    f = __builtin_amdgcn_mfma_f32_32x32x2f32(a4.w, b4.w, f, 0, 0, 0);
                }
            }
            if (want_c) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int row = rbase + 8 * (v >> 2) + 4 * lh + (v & 3);
                    if (row < M && col_ok) store_out(out, row, col, f[v]);
                }
            }
        }
    }
}

// FULL: M, N multiples of 256 and K a multiple of the tile depth -- operand loads carry no guard at all, so
// nothing consumes a loaded register before it is written to LDS two iterations later.
template <bool COMP, bool WCINT, bool FULL>
__global__ __launch_bounds__(512, 1) void int8_gemm256_kernel(int M, int N, int K,
                                                              const int8_t* __restrict__ Aq,
                                                              const int8_t* __restrict__ BqT,
                                                              const float* __restrict__ sA,
                                                              const float* __restrict__ sB,
                                                              const float* __restrict__ Lp,
                                                              const float* __restrict__ Rp, int R2P,
                                                              GemmOut out,
                                                              int32_t* __restrict__ Cint, int tiles_n,
                                                              int ntiles, float qmaxf) {
    __shared__ __align__(16) int8_t As[2][BTM * BSTRIDE];
    __shared__ __align__(16) int8_t Bs[2][BTN * BSTRIDE];
    const int nk = (K + BBK - 1) / BBK;
    const int tile = xcd_tile(blockIdx.x, tiles_n, ntiles);
    const int m0 = (tile / tiles_n) * BTM, n0 = (tile % tiles_n) * BTN;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int wm = wave >> 1, wn = wave & 1;
    const int l32 = lane & 31, lh = lane >> 5;

    v16i acc[2][4];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0;

    // staging: 2048 16-byte chunks per operand tile, four per thread.  Global loads run two 128-deep
    // K-tiles ahead of the matrix cores in a ring of two register sets (a tile's MFMA time is below
    // global-load latency, so one tile of lookahead stalls every iteration); LDS holds the current
    // and the next tile.  (Measured against 64-deep tiles with a ring of three -- the same depth in
    // flight, twice the barriers per product: 84 against 91 us at 4096^3, 3.99 against 4.29 ms at 16384^3.)
    const int srow0 = tid / BCHUNKS, skc = (tid % BCHUNKS) * 16;
    // The register sets are individually named scalars (not arrays passed by reference):
    // that keeps them in VGPRs; as arrays they were demoted to scratch memory.
    // (FULL: one base per operand and wave-uniform row offsets; otherwise a clamped row pointer per load)
    static_assert(BTM == 4 * BROWS && BTN == BTM, "four staged chunks per thread and operand");
    const int8_t *pa[4], *pb[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        pa[u] = FULL ? nullptr : code_row(Aq, m0 + srow0 + BROWS * u, M, K);
        pb[u] = FULL ? nullptr : code_row(BqT, n0 + srow0 + BROWS * u, N, K);
    }
    auto ldA = [&](int u, int k0) -> uint4 {
        if (FULL)   // tiles past the end of K are loaded (clamped) but never stored or used
            return *reinterpret_cast<const uint4*>(Aq + (size_t)(m0 + srow0 + BROWS * u) * K + min(k0, K - BBK) + skc);
        return load16b<true>(pa[u], K, k0 + skc);
    };
    auto ldB = [&](int u, int k0) -> uint4 {
        if (FULL)
            return *reinterpret_cast<const uint4*>(BqT + (size_t)(n0 + srow0 + BROWS * u) * K + min(k0, K - BBK) + skc);
        return load16b<true>(pb[u], K, k0 + skc);
    };
    auto stA = [&](int u, int buf, uint4 v) {
        *reinterpret_cast<uint4*>(&As[buf][(srow0 + BROWS * u) * BSTRIDE + skc]) = v;
    };
    auto stB = [&](int u, int buf, uint4 v) {
        *reinterpret_cast<uint4*>(&Bs[buf][(srow0 + BROWS * u) * BSTRIDE + skc]) = v;
    };
#define LRQ_DECL(S) uint4 S##a0, S##a1, S##a2, S##a3, S##b0, S##b1, S##b2, S##b3
#define LRQ_GLOAD(S, k0)                                                   \
    S##a0 = ldA(0, k0); S##b0 = ldB(0, k0); S##a1 = ldA(1, k0); S##b1 = ldB(1, k0); \
    S##a2 = ldA(2, k0); S##b2 = ldB(2, k0); S##a3 = ldA(3, k0); S##b3 = ldB(3, k0);
#define LRQ_TAIL(R) R = tail16(R, sh)
#define LRQ_SSTORE(S, buf, k0)                                                     \
    if (!FULL && (k0) + BBK > K) {                                                 \
        const int sh = max(0, (k0) + skc - (K - 16));                              \
        LRQ_TAIL(S##a0); LRQ_TAIL(S##b0); LRQ_TAIL(S##a1); LRQ_TAIL(S##b1);        \
        LRQ_TAIL(S##a2); LRQ_TAIL(S##b2); LRQ_TAIL(S##a3); LRQ_TAIL(S##b3);        \
    }                                                                              \
    stA(0, buf, S##a0); stB(0, buf, S##b0); stA(1, buf, S##a1); stB(1, buf, S##b1); \
    stA(2, buf, S##a2); stB(2, buf, S##b2); stA(3, buf, S##a3); stB(3, buf, S##b3);
    LRQ_DECL(r0);
    LRQ_DECL(r1);
    auto compute = [&](int buf) {
#pragma unroll
        for (int kk = 0; kk < BBK / 32; ++kk) {
            v4i af[2], bf[4];
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
                af[mt] = *reinterpret_cast<const v4i*>(
                    &As[buf][(wm * 64 + mt * 32 + l32) * BSTRIDE + kk * 32 + lh * 16]);
#pragma unroll
            for (int nt = 0; nt < 4; ++nt)
                bf[nt] = *reinterpret_cast<const v4i*>(
                    &Bs[buf][(wn * 128 + nt * 32 + l32) * BSTRIDE + kk * 32 + lh * 16]);
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                for (int nt = 0; nt < 4; ++nt)
                    acc[mt][nt] = __builtin_amdgcn_mfma_i32_32x32x32_i8(af[mt], bf[nt], acc[mt][nt], 0, 0, 0);
        }
    };
    LRQ_GLOAD(r0, 0);
    LRQ_GLOAD(r1, BBK);
    LRQ_SSTORE(r0, 0, 0);
    __syncthreads();
    // iteration i: the set that held tile i is free -> load tile i + 2; compute tile i; publish tile i+1
#define LRQ_GEMM_STEP(J, SCUR, SNEXT)                  \
    if (kt + J < nk) {                                 \
        const int i = kt + J;                          \
        LRQ_GLOAD(SCUR, (i + 2) * BBK);                \
        compute(i & 1);                                \
        if (i + 1 < nk) { LRQ_SSTORE(SNEXT, (i + 1) & 1, (i + 1) * BBK); } \
        __syncthreads();                               \
    }
    for (int kt = 0; kt < nk; kt += 2) {
        LRQ_GEMM_STEP(0, r0, r1)
        LRQ_GEMM_STEP(1, r1, r0)
    }
#undef LRQ_GEMM_STEP
#undef LRQ_DECL
#undef LRQ_GLOAD
#undef LRQ_SSTORE

    finish_large_tile<COMP, WCINT, false>(LargeTile{M, N, m0, n0, sA, sB, Lp, Rp, R2P, out, Cint, nullptr, false, qmaxf}, acc, &As[0][0],
                                          &Bs[0][0]);
}

// The same tiles from packed codes.
// SPLITK (raw sums only, whole tiles and 128-deep steps): workgroups [0, full_tiles) compute one tile each as usual; the remaining
// ntiles - full_tiles tiles are cut into `slices` ranges of K, one workgroup per (tile, range), which leave their int32 partial
// sums in `part` ([tile][range][256][256]) for sum_tile_slices_kernel (integer addition: exact whatever the cut).
template <int FMT, bool COMP, bool WCINT, bool SPLITK = false>
__global__ __launch_bounds__(512, 1) void packed_gemm256_kernel(int M, int N, int K, const uint8_t* __restrict__ A,
                                                                const uint8_t* __restrict__ B, const float* __restrict__ sA,
                                                                const float* __restrict__ sB, const float* __restrict__ Lp,
                                                                const float* __restrict__ Rp, int R2P, GemmOut out,
                                                                int32_t* __restrict__ Cint, int tiles_n, int ntiles, int full_tiles,
                                                                int slices, int32_t* __restrict__ part, float qmaxf) {
    constexpr int ST = FMT == PK8 ? 4 : 6;
    __shared__ __align__(16) int8_t tiles[2 * LARGE_LDS];
    static_assert(ST * 16 * pk_block(FMT) <= 2 * LARGE_LDS, "the stages fit");
    int wg = blockIdx.x, kb0 = 0, nk = pk_kblocks(K);
    const int nkb = nk;
    bool partial = false;
    if constexpr (SPLITK) {
        if (wg >= full_tiles) {
            const int e = wg - full_tiles, lt = e / slices, sl = e - lt * slices;
            wg = full_tiles + lt;
            part += (size_t)e * (BTM * BTN);
            kb0 = (int)((long long)sl * nkb / slices);
            nk = (int)((long long)(sl + 1) * nkb / slices) - kb0;
            partial = true;
        }
    }
    const int tile = xcd_tile(wg, tiles_n, ntiles);
    const int m0 = (tile / tiles_n) * BTM, n0 = (tile % tiles_n) * BTN;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    PackedSum<FMT> acc[2][4];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0;
    packed_products<FMT, 2, 4, 8, 8, 8, ST>(A, B, m0 >> 5, (M + 31) >> 5, n0 >> 5, (N + 31) >> 5, nkb, kb0, nk, reinterpret_cast<uint8_t*>(tiles),
                                       wave, lane, (wave >> 1) * 2, (wave & 1) * 4, acc);
    finish_large_tile<COMP, WCINT, SPLITK>(LargeTile{M, N, m0, n0, sA, sB, Lp, Rp, R2P, out, Cint, part, partial, qmaxf}, acc, tiles,
                                           tiles + LARGE_LDS);
}

// Complete residual compensation (Eq. (gemm_r_split)): the sum of three or four integer products, each with step vectors of
// its own, in one launch: the K tiles of all products form one sequence (loads run two tiles ahead across the boundaries),
// and where a product ends its sums are dequantized and added to a float32 total in registers, in the order and with the
// roundings of one launch per product that reads and writes D.  Waves of 64 x 64 (64 registers of sums and 64 of totals) in a
// WM x 2 grid: 256 x 128 tiles with eight waves, one workgroup per CU, or 128 x 128 with four, two per CU; otherwise the
// staging of the 256 x 256 kernel above.  In the loop it runs at that kernel's rate (2.0 POP/s at 4096^3, bound by the matrix
// cores' sustained rate, LDS traffic and one barrier per K tile in turn); the read-modify-writes of D, step vectors, starts
// and ends of a launch per product fall away.  Calls with four products, one launch per product / this: 4096^3 int8 540 / 376
// us, 5000^3 1142 / 896, 3072^3 414 / 234, 2000^3 216 / 99, 2000 x 2000 x 500 142 / 48, 300^3 68 / 40.
#define TTN 128
struct TermArgs {
    const int8_t *A[2], *B[2];              // codes of the operands and of their residuals (B transposed)
    const float *amaxA[2], *amaxB[2];       // their group maxima
};
template <int WM, bool FULL>
__global__ __launch_bounds__(128 * WM, WM == 4 ? 1 : 2) void int8_terms_kernel(int M, int N, int K, TermArgs t, int terms, float qmaxf, GemmOut out,
                                                            int tiles_n, int ntiles) {
    constexpr int TTM = 64 * WM, THREADS = 128 * WM, ROWS = THREADS / BCHUNKS, LB = TTN / ROWS;     // (TTM / ROWS == 4)
    __shared__ __align__(16) int8_t As[2][TTM * BSTRIDE];
    __shared__ __align__(16) int8_t Bs[2][TTN * BSTRIDE];
    __shared__ __align__(16) float sAs[2][TTM], sBs[2][TTN];
    const int nk = (K + BBK - 1) / BBK, total = nk * terms;
    const int tile = xcd_tile(blockIdx.x, tiles_n, ntiles);
    const int m0 = (tile / tiles_n) * TTM, n0 = (tile % tiles_n) * TTN;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int wm = wave >> 1, wn = wave & 1;
    const int l32 = lane & 31, lh = lane >> 5;
    {
        float l;
        const int ra = tid % TTM, rb = tid % TTN;
        make_scales(t.amaxA[tid / TTM][min(m0 + ra, M - 1)], qmaxf, l, sAs[tid / TTM][ra]);
        if (tid < 2 * TTN) make_scales(t.amaxB[tid / TTN][min(n0 + rb, N - 1)], qmaxf, l, sBs[tid / TTN][rb]);
    }
    v16i acc[2][2];
    v16f f[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) { acc[a][b][v] = 0; f[a][b][v] = 0.f; }
    const int srow0 = tid / BCHUNKS, skc = (tid % BCHUNKS) * 16;
    // offset of a staged row in any code matrix of the operand (rows past the end re-read the last one, never stored)
    size_t ra[FULL ? 1 : 4], rb[FULL ? 1 : LB];
    if constexpr (FULL) {
        ra[0] = (size_t)(m0 + srow0) * K + skc;
        rb[0] = (size_t)(n0 + srow0) * K + skc;
    } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) ra[u] = (size_t)min(m0 + srow0 + ROWS * u, M - 1) * K;
#pragma unroll
        for (int u = 0; u < LB; ++u) rb[u] = (size_t)min(n0 + srow0 + ROWS * u, N - 1) * K;
    }
    auto ld = [&](const int8_t* base, const size_t* row, int u, int k0) -> uint4 {
        if constexpr (FULL) return *reinterpret_cast<const uint4*>(base + (size_t)(ROWS * u) * K + k0 + row[0]);
        else return load16b<true>(base + row[u], K, k0 + skc);
    };
    int lt = 0, lk = 0, st = 0;             // product and column of the next tile to load; column of the next tile to store
    auto next_load = [&] {                  // (past the end: the last tile again, never used)
        if (lk + BBK < K) lk += BBK;
        else if (lt + 1 < terms) { ++lt; lk = 0; }
    };
#define LRQ_DECL(S) uint4 S##a0, S##a1, S##a2, S##a3, S##b0, S##b1, S##b2, S##b3
#define LRQ_GLOAD(S)                                                                                     \
    {                                                                                                    \
        const int8_t *const pa = t.A[lt >> 1], *const pb = t.B[lt & 1];                                  \
        S##a0 = ld(pa, ra, 0, lk); S##b0 = ld(pb, rb, 0, lk); S##a1 = ld(pa, ra, 1, lk);                 \
        S##b1 = ld(pb, rb, 1, lk); S##a2 = ld(pa, ra, 2, lk); S##a3 = ld(pa, ra, 3, lk);                 \
        if (LB == 4) { S##b2 = ld(pb, rb, LB == 4 ? 2 : 0, lk); S##b3 = ld(pb, rb, LB == 4 ? 3 : 0, lk); } \
        next_load();                                                                                     \
    }
#define LRQ_ST(BUF, U, V) *reinterpret_cast<uint4*>(&BUF[(srow0 + ROWS * U) * BSTRIDE + skc]) = V
#define LRQ_SSTORE(S, buf)                                                                               \
    {                                                                                                    \
        if (!FULL && st + BBK > K) {                                                                     \
            const int sh = max(0, st + skc - (K - 16));                                                  \
            S##a0 = tail16(S##a0, sh); S##a1 = tail16(S##a1, sh); S##a2 = tail16(S##a2, sh);             \
            S##a3 = tail16(S##a3, sh); S##b0 = tail16(S##b0, sh); S##b1 = tail16(S##b1, sh);             \
            if (LB == 4) { S##b2 = tail16(S##b2, sh); S##b3 = tail16(S##b3, sh); }                       \
        }                                                                                                \
        LRQ_ST(As[buf], 0, S##a0); LRQ_ST(Bs[buf], 0, S##b0); LRQ_ST(As[buf], 1, S##a1);                 \
        LRQ_ST(Bs[buf], 1, S##b1); LRQ_ST(As[buf], 2, S##a2); LRQ_ST(As[buf], 3, S##a3);                 \
        if (LB == 4) { LRQ_ST(Bs[buf], 2, S##b2); LRQ_ST(Bs[buf], 3, S##b3); }                           \
        st = st + BBK < K ? st + BBK : 0;                                                                \
    }
    auto compute = [&](int buf) {
#pragma unroll
        for (int kk = 0; kk < BBK / 32; ++kk) {
            v4i af[2], bf[2];
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
                af[mt] = *reinterpret_cast<const v4i*>(&As[buf][(wm * 64 + mt * 32 + l32) * BSTRIDE + kk * 32 + lh * 16]);
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
                bf[nt] = *reinterpret_cast<const v4i*>(&Bs[buf][(wn * 64 + nt * 32 + l32) * BSTRIDE + kk * 32 + lh * 16]);
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                for (int nt = 0; nt < 2; ++nt)
                    acc[mt][nt] = __builtin_amdgcn_mfma_i32_32x32x32_i8(af[mt], bf[nt], acc[mt][nt], 0, 0, 0);
        }
    };
    // D <- alpha * product + beta * D, the next products with beta = 1 and the total in D's place
    auto add_product = [&](int term) {
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const float4 s4 = *reinterpret_cast<const float4*>(&sAs[term >> 1][wm * 64 + mt * 32 + 8 * g + 4 * lh]);
                const float sa[4] = {s4.x, s4.y, s4.z, s4.w};
#pragma unroll
                for (int nt = 0; nt < 2; ++nt) {
                    const float sb = sBs[term & 1][wn * 64 + nt * 32 + l32];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int v = 4 * g + e;
                        f[mt][nt][v] = out.alpha * (((float)acc[mt][nt][v] * sa[e]) * sb) + f[mt][nt][v];
                        acc[mt][nt][v] = 0;
                    }
                }
                __builtin_amdgcn_sched_barrier(0);      // (eight entries at a time: the steps of all would not fit in registers)
            }
    };
    if (out.beta != 0.f) {
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {
                const int col = n0 + wn * 64 + nt * 32 + l32;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int row = m0 + wm * 64 + mt * 32 + 8 * (v >> 2) + 4 * lh + (v & 3);
                    if (row < M && col < N) f[mt][nt][v] = out.beta * out.C[(size_t)row * out.ldc + col];
                }
            }
    }
    LRQ_DECL(r0);
    LRQ_DECL(r1);
    LRQ_GLOAD(r0);
    LRQ_GLOAD(r1);
    LRQ_SSTORE(r0, 0);
    __syncthreads();
    int left = nk, term = 0;                // tiles left of the current product
    // iteration i: the set that held tile i is free -> load tile i + 2; compute tile i; publish tile i + 1
#define LRQ_TERM_STEP(J, SCUR, SNEXT)                                \
    if (i0 + J < total) {                                            \
        LRQ_GLOAD(SCUR);                                             \
        compute(J);                                                  \
        if (i0 + J + 1 < total) { LRQ_SSTORE(SNEXT, 1 - J); }        \
        if (--left == 0) { add_product(term); ++term; left = nk; }   \
        __syncthreads();                                             \
    }
    for (int i0 = 0; i0 < total; i0 += 2) {
        LRQ_TERM_STEP(0, r0, r1)
        LRQ_TERM_STEP(1, r1, r0)
    }
#undef LRQ_TERM_STEP
#undef LRQ_DECL
#undef LRQ_GLOAD
#undef LRQ_ST
#undef LRQ_SSTORE
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            const int col = n0 + wn * 64 + nt * 32 + l32;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = m0 + wm * 64 + mt * 32 + 8 * (v >> 2) + 4 * lh + (v & 3);
                if (row < M && col < N) out.C[(size_t)row * out.ldc + col] = f[mt][nt][v];
            }
        }
}

// Four products of the codes (0) and the residuals' codes (1) of both operands, packed: a 128 x 128 tile of D needs 128 rows of each of
// the four code matrices, which stacked are the operands of one 256 x 256 tile of the kernel above, a product per quadrant.  So
// every operand tile is read and staged once for two products, the matrix cores see 64 x 128 tiles per wave, and the quadrants
// meet in LDS at the end, added in the order (and with the roundings) of one launch per product.  Four products of random codes, us,
// int8_terms_kernel / this with bytes / with six bits: 300^3 16.5 / 14.7 / 13.5, 1024^3 26.2 / 22.4 / 18.8, 1537 x 1021 x 2311 79.5 /
// 40.4 / 31.5, 2000^3 62.4 / 41.8 / 32.8, 3000^3 205 / 143 / 106, 4096^3 312 / 274 / 195, 5000^3 736 / 529 / 378, 8192^3 2239 / 1926 /
// 1314.  (Three products would leave a quadrant idle: int8_terms_kernel.)
template <int FMT>
__global__ __launch_bounds__(512, 1) void packed_terms_kernel(int M, int N, int K, TermArgs t, float qmaxf, GemmOut out, int tiles_n,
                                                              int ntiles) {
    constexpr int ST = FMT == PK8 ? 4 : 6, T = 128, LD = T + 8;     // (+ 8: the two row groups of a wave's store on different banks)
    __shared__ __align__(16) uint8_t stages[2 * LARGE_LDS];
    __shared__ __align__(16) float steps[4 * T];
    static_assert(ST * 16 * pk_block(FMT) <= 2 * LARGE_LDS && 2 * T * LD * 4 <= 2 * LARGE_LDS, "stages and two quadrants fit");
    const int tile = xcd_tile(blockIdx.x, tiles_n, ntiles);
    const int m0 = (tile / tiles_n) * T, n0 = (tile % tiles_n) * T;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int wm = wave >> 1, wn = wave & 1, l32 = lane & 31, lh = lane >> 5;
    {
        const int lvl = (tid >> 7) & 1, e = tid & 127;
        steps[tid] = step_of(tid < 256 ? t.amaxA[lvl][min(m0 + e, M - 1)] : t.amaxB[lvl][min(n0 + e, N - 1)], qmaxf);
    }
    PackedSum<FMT> acc[2][4];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0;
    packed_products<FMT, 2, 4, 8, 8, 8, ST, true>(reinterpret_cast<const uint8_t*>(t.A[0]), reinterpret_cast<const uint8_t*>(t.B[0]), m0 >> 5,
                                                  (M + 31) >> 5, n0 >> 5, (N + 31) >> 5, pk_kblocks(K), 0, pk_kblocks(K), stages, wave,
                                                  lane, wm * 2, wn * 4, acc, reinterpret_cast<const uint8_t*>(t.A[1]),
                                                  reinterpret_cast<const uint8_t*>(t.B[1]));
    float* const quad = reinterpret_cast<float*>(stages);
    const int crow = tid >> 5, ccol = (tid & 31) * 4;           // of this thread's sixteenth of the rows: crow + 16 i
    float4 f[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) f[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    const int cols = min(4, N - n0 - ccol);                     // columns of this thread's groups inside D
    if (out.beta != 0.f) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float* p = out.C + (size_t)min(m0 + crow + 16 * i, M - 1) * out.ldc + n0 + ccol;
            if (cols > 0) f[i].x = out.beta * p[0];
            if (cols > 1) f[i].y = out.beta * p[1];
            if (cols > 2) f[i].z = out.beta * p[2];
            if (cols > 3) f[i].w = out.beta * p[3];
        }
    }
#pragma unroll
    for (int level = 0; level < 2; ++level) {
        if (level) __syncthreads();
        if ((wm >> 1) == level) {
            const int rbase = (wm & 1) * 64 + 4 * lh;
            float* const q = quad + wn * (T * LD);
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) {
                const float sb = steps[256 + wn * T + nt * 32 + l32];
#pragma unroll
                for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int row = rbase + mt * 32 + 8 * (v >> 2) + (v & 3);
                        q[row * LD + nt * 32 + l32] = out.alpha * ((code_sum(acc[mt][nt][v]) * steps[level * T + row]) * sb);
                    }
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const float4 x = *reinterpret_cast<const float4*>(quad + b * (T * LD) + (crow + 16 * i) * LD + ccol);
                f[i].x = x.x + f[i].x; f[i].y = x.y + f[i].y; f[i].z = x.z + f[i].z; f[i].w = x.w + f[i].w;
            }
    }
    const bool whole = cols == 4 && (out.ldc & 3) == 0 && ((uintptr_t)out.C & 15) == 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int row = m0 + crow + 16 * i;
        if (row >= M) continue;
        float* p = out.C + (size_t)row * out.ldc + n0 + ccol;
        if (whole) *reinterpret_cast<float4*>(p) = f[i];
        else {
            if (cols > 0) p[0] = f[i].x;
            if (cols > 1) p[1] = f[i].y;
            if (cols > 2) p[2] = f[i].z;
            if (cols > 3) p[3] = f[i].w;
        }
    }
}

// The epilogue of the GEMM as a kernel of its own, for the schedule in which the integer
// product runs early (next to the small kernels of the factorizations) and leaves its raw
// int32 sums in C's memory: C <- float(Cint) sA_i sB_j + Lp . Rp^T in place, with the same
// products accumulated in the same order as the fused epilogue (bit-identical results).
// 128x128 tile per workgroup, 4 waves of 64x64 (2x2 MFMA tiles).  The MFMA runs on the
// transposed tile (Rp rows as the A operand, Lp rows as B), so that a lane owns ONE row of C
// and four groups of 4 consecutive columns: C is read and written with 16-byte accesses
// (needs N % 4 == 0).  A wave first issues all its loads -- its four tiles of sums and, per 64
// panel columns, the panel rows of both row tiles and both column tiles -- without branches,
// and then runs the four accumulation chains interleaved, so neither load latency nor the
// latency of dependent MFMAs is exposed.
__global__ __launch_bounds__(256, 2) void rank_update_kernel(int M, int N, float* __restrict__ C,
                                                          const float* __restrict__ sA,
                                                          const float* __restrict__ sB,
                                                          const float* __restrict__ Lp,
                                                          const float* __restrict__ Rp, int R2P, int tiles_n,
                                                          float alpha) {
    __shared__ __align__(16) float pl[2][128][68];      // Lp and Rp rows of the tile, 64 columns, padded
    const int m0 = (blockIdx.x / tiles_n) * 128, n0 = (blockIdx.x % tiles_n) * 128;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int wm = wave >> 1, wn = wave & 1;
    const int l32 = lane & 31, lh = lane >> 5;
    const int rb0 = m0 + wm * 64, cb0 = n0 + wn * 64;
    // D[i][j] of tile (mt, nt): j = l32 is the row of C, i = 8 g + 4 lh + e its column (v = 4 g + e)
    int row[2], colb[2][4];         // this lane's C rows and first columns of its groups (clamped)
    bool row_ok[2], col_ok[2][4];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        row_ok[t] = rb0 + t * 32 + l32 < M;
        row[t] = min(rb0 + t * 32 + l32, M - 1);
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int c = cb0 + t * 32 + 8 * g + 4 * lh;
            col_ok[t][g] = c < N;
            colb[t][g] = min(c, N - 4);
        }
    }
    v16f f[2][2];
    int4 raw[2][2][4];
    float4 sb[2][4];
    float sa[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        sa[t] = sA[row[t]];
#pragma unroll
        for (int g = 0; g < 4; ++g) sb[t][g] = *reinterpret_cast<const float4*>(sB + colb[t][g]);
    }
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                raw[mt][nt][g] = *reinterpret_cast<const int4*>(C + (size_t)row[mt] * N + colb[nt][g]);
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                f[mt][nt][4 * g + 0] = ((float)raw[mt][nt][g].x * sa[mt]) * sb[nt][g].x;
                f[mt][nt][4 * g + 1] = ((float)raw[mt][nt][g].y * sa[mt]) * sb[nt][g].y;
                f[mt][nt][4 * g + 2] = ((float)raw[mt][nt][g].z * sa[mt]) * sb[nt][g].z;
                f[mt][nt][4 * g + 3] = ((float)raw[mt][nt][g].w * sa[mt]) * sb[nt][g].w;
            }
    // The panel rows of the tile go through LDS, 64 columns at a time: the workgroup loads each row once,
    // 16 lanes per 256-byte row, instead of every wave fetching its operands with 16-byte loads that touch
    // 32 cache lines per instruction (measured on this access pattern: 36 instead of 41 us).
    for (int t0 = 0; t0 < R2P; t0 += 64) {      // R2P % 8 == 0
        if (t0 > 0) __syncthreads();            // the previous chunk is no longer read
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int idx = threadIdx.x + 256 * i, r = idx >> 4, c = (idx & 15) * 4;
            const int col = t0 + c;
            const bool in = col < R2P;           // panel columns past R2P enter as zeros
            const int cc = min(col, R2P - 4);
            // rows / columns past the end re-read the last one (never stored)
            const float4 x = *reinterpret_cast<const float4*>(Lp + (size_t)min(m0 + r, M - 1) * R2P + cc);
            const float4 y = *reinterpret_cast<const float4*>(Rp + (size_t)min(n0 + r, N - 1) * R2P + cc);
            *reinterpret_cast<float4*>(&pl[0][r][c]) = make_float4(in ? x.x : 0.f, in ? x.y : 0.f, in ? x.z : 0.f, in ? x.w : 0.f);
            *reinterpret_cast<float4*>(&pl[1][r][c]) = make_float4(in ? y.x : 0.f, in ? y.y : 0.f, in ? y.z : 0.f, in ? y.w : 0.f);
        }
        __syncthreads();
        float4 a4[2][8], b4[2][8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                a4[t][u] = *reinterpret_cast<const float4*>(&pl[0][wm * 64 + t * 32 + l32][8 * u + 4 * lh]);
                b4[t][u] = *reinterpret_cast<const float4*>(&pl[1][wn * 64 + t * 32 + l32][8 * u + 4 * lh]);
            }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                for (int nt = 0; nt < 2; ++nt) {    // A operand: panel row of the column, B operand: of the row
                    f[mt][nt] = __builtin_amdgcn_mfma_f32_32x32x2f32(b4[nt][u].x, a4[mt][u].x, f[mt][nt], 0, 0, 0);
                    f[mt][nt] = __builtin_amdgcn_mfma_f32_32x32x2f32(b4[nt][u].y, a4[mt][u].y, f[mt][nt], 0, 0, 0);
                    f[mt][nt] = __builtin_amdgcn_mfma_f32_32x32x2f32(b4[nt][u].z, a4[mt][u].z, f[mt][nt], 0, 0, 0);
                    f[mt][nt] = __builtin_amdgcn_mfma_f32_32x32x2f32(b4[nt][u].w, a4[mt][u].w, f[mt][nt], 0, 0, 0);
                }
        }
    }
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                if (row_ok[mt] && col_ok[nt][g])
                    *reinterpret_cast<float4*>(C + (size_t)row[mt] * N + colb[nt][g]) =
                        make_float4(alpha * f[mt][nt][4 * g + 0], alpha * f[mt][nt][4 * g + 1],
                                    alpha * f[mt][nt][4 * g + 2], alpha * f[mt][nt][4 * g + 3]);
}

// The same update for wide panels (2r > 64), where the float32 matrix cores are the limit (4 R2P flops per output:
// 0.87 ms of matrix-core time at 16384^2 and r = 64).  The panel rows are split into three bfloat16 planes while
// they are staged in LDS (exact: a float32 is the sum of its three planes) and the six plane products of weight
// >= 2^-16 run on v_mfma_f32_32x32x16_bf16 with float32 accumulation: 192 instead of 512 matrix-core cycles per
// 16 panel columns.  The same products in the same order as the large-tile kernel's epilogue (the same bits); the
// smaller tiles keep the float32 instructions, another rounding order.  Operand layout (lane l): A[i = l%32][k = 8(l/32) .. +8],
// B[k = 8(l/32) .. +8][j = l%32]; D as for the 32x32 float32 instruction.
__global__ __launch_bounds__(256, 2) void rank_update_bf16_kernel(int M, int N, float* __restrict__ C,
                                                                  const float* __restrict__ sA,
                                                                  const float* __restrict__ sB,
                                                                  const float* __restrict__ Lp,
                                                                  const float* __restrict__ Rp, int R2P, int tiles_n,
                                                                  float alpha) {
    __shared__ __align__(16) uint16_t pp[2][3][128 * PANEL_LD];     // [Lp | Rp][plane][row][column of the chunk]
    const int m0 = (blockIdx.x / tiles_n) * 128, n0 = (blockIdx.x % tiles_n) * 128;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int wm = wave >> 1, wn = wave & 1;
    const int l32 = lane & 31, lh = lane >> 5;
    const int rb0 = m0 + wm * 64, cb0 = n0 + wn * 64;
    int row[2], colb[2][4];
    bool row_ok[2], col_ok[2][4];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        row_ok[t] = rb0 + t * 32 + l32 < M;
        row[t] = min(rb0 + t * 32 + l32, M - 1);
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int c = cb0 + t * 32 + 8 * g + 4 * lh;
            col_ok[t][g] = c < N;
            colb[t][g] = min(c, N - 4);
        }
    }
    v16f f[2][2];
    {
        int4 raw[2][2][4];
        float4 sb[2][4];
        float sa[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            sa[t] = sA[row[t]];
#pragma unroll
            for (int g = 0; g < 4; ++g) sb[t][g] = *reinterpret_cast<const float4*>(sB + colb[t][g]);
        }
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    raw[mt][nt][g] = *reinterpret_cast<const int4*>(C + (size_t)row[mt] * N + colb[nt][g]);
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    f[mt][nt][4 * g + 0] = ((float)raw[mt][nt][g].x * sa[mt]) * sb[nt][g].x;
                    f[mt][nt][4 * g + 1] = ((float)raw[mt][nt][g].y * sa[mt]) * sb[nt][g].y;
                    f[mt][nt][4 * g + 2] = ((float)raw[mt][nt][g].z * sa[mt]) * sb[nt][g].z;
                    f[mt][nt][4 * g + 3] = ((float)raw[mt][nt][g].w * sa[mt]) * sb[nt][g].w;
                }
    }
    for (int t0 = 0; t0 < R2P; t0 += PANEL_KC) {       // R2P % 8 == 0
        if (t0 > 0) __syncthreads();                // the previous chunk is no longer read
        // 2 panels x 128 rows x 4 groups of 8 columns = 1024 units, four per thread: load, split, store the planes
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int unit = threadIdx.x + 256 * i;
            const int pnl = unit >> 9, r = (unit >> 2) & 127, c8 = (unit & 3) * 8;
            const float* src = pnl == 0 ? Lp + (size_t)min(m0 + r, M - 1) * R2P : Rp + (size_t)min(n0 + r, N - 1) * R2P;
            stage_planes(src, t0 + c8, R2P, &pp[pnl][0][r * PANEL_LD + c8], 128 * PANEL_LD);     // (rows past the end: the last one again)
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < PANEL_KC / 16; ++u) {
            Planes3 a[2], b[2];     // a: Lp rows of the two row tiles (B operand), b: Rp rows of the two column tiles (A operand)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int oa = (wm * 64 + t * 32 + l32) * PANEL_LD + 16 * u + 8 * lh;
                const int ob = (wn * 64 + t * 32 + l32) * PANEL_LD + 16 * u + 8 * lh;
                a[t].p1 = *reinterpret_cast<const v8bf16*>(&pp[0][0][oa]);
                a[t].p2 = *reinterpret_cast<const v8bf16*>(&pp[0][1][oa]);
                a[t].p3 = *reinterpret_cast<const v8bf16*>(&pp[0][2][oa]);
                b[t].p1 = *reinterpret_cast<const v8bf16*>(&pp[1][0][ob]);
                b[t].p2 = *reinterpret_cast<const v8bf16*>(&pp[1][1][ob]);
                b[t].p3 = *reinterpret_cast<const v8bf16*>(&pp[1][2][ob]);
            }
            // the six plane products, smallest first; the four tiles are independent chains
#define LRQ_RU_PP(PB, PA)                                                                                   \
    _Pragma("unroll") for (int mt = 0; mt < 2; ++mt) _Pragma("unroll") for (int nt = 0; nt < 2; ++nt)        \
        f[mt][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[nt].PB, a[mt].PA, f[mt][nt], 0, 0, 0);
            LRQ_RU_PP(p3, p1)
            LRQ_RU_PP(p2, p2)
            LRQ_RU_PP(p1, p3)
            LRQ_RU_PP(p2, p1)
            LRQ_RU_PP(p1, p2)
            LRQ_RU_PP(p1, p1)
#undef LRQ_RU_PP
        }
    }
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                if (row_ok[mt] && col_ok[nt][g])
                    *reinterpret_cast<float4*>(C + (size_t)row[mt] * N + colb[nt][g]) =
                        make_float4(alpha * f[mt][nt][4 * g + 0], alpha * f[mt][nt][4 * g + 1],
                                    alpha * f[mt][nt][4 * g + 2], alpha * f[mt][nt][4 * g + 3]);
}

// ---------------------------------------------------------------------------
// Panels of the rank-2r update (compensation terms of Algorithm 2 regrouped):
//   C = C0 + [U Sigma | A~ W] . [V^T B~ + (V^T W) Gamma Z^T ; Gamma Z^T]
// panel_prep: step vectors of both operands, the planes of W and V as matrix-core operands, and X = V^T W in k-slices; the code
// products and the panels follow in one launch (passes.hip).
// ---------------------------------------------------------------------------

// Xp[ks][t][u] = sum over the ks-th slice of k of Vt[t][k] W[k][u] (r x r per slice), float64
// accumulation, for the workgroup (t, ks).  Thread (kg, u) walks k = kg, kg + G, ... so a
// wavefront reads whole rows of W (coalesced) against a broadcast element of Vt, eight loads
// deep; the G partial sums are merged through LDS in fixed order.  The slices are summed
// (fixed order) where X is used.
template <int RU>
__device__ __forceinline__ void vtw_block(const float* __restrict__ Vt, const float* __restrict__ W, int K,
                                          int r, int kslice, int t, int ks, float* __restrict__ Xp,
                                          double* __restrict__ part) {
    constexpr int G = 256 / RU;
    const int u = threadIdx.x % RU, kg = threadIdx.x / RU;
    const int uc = min(u, r - 1);
    const int kb = ks * kslice, ke = min(K, kb + kslice);
    const float* vrow = Vt + (size_t)t * K;
    double acc = 0.0;
    for (int k0 = kb + kg; k0 < ke; k0 += 8 * G) {
        float v[8], w[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int k = min(k0 + j * G, K - 1);
            v[j] = vrow[k];
            w[j] = W[(size_t)k * r + uc];
        }
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (k0 + j * G < ke) acc = fma((double)v[j], (double)w[j], acc);
    }
    part[kg * RU + u] = acc;
    __syncthreads();
    if (kg == 0 && u < r) {
        double sum = 0.0;
#pragma unroll
        for (int g = 0; g < G; ++g) sum += part[g * RU + u];
        Xp[((size_t)ks * r + t) * r + u] = (float)sum;
    }
}

struct PrepArgs {
    const float *amaxA, *amaxB, *W, *Vt;
    float *lamA, *sA, *lamB, *sB, *Xp;
    uint16_t *Wf, *Vf;
    int M, Mp, N, Np, K, Kp, r, RP, kslice, nslices;
    float qmaxf;
    int nbA, nbB, nbP;      // workgroups of the first three sections
};

// Workgroup ranges: [0, nbA) steps of A, [nbA, nbA+nbB) steps of B, then nbP workgroups that
// write the zero-padded bfloat16 planes of W (K x r) and V = Vt^T in operand order (see FACTOR_PIECE), then
// r * nslices workgroups of V^T W.
__global__ __launch_bounds__(256) void panel_prep_kernel(PrepArgs a) {
    __shared__ double part[256];
    int b = blockIdx.x;
    if (b < a.nbA + a.nbB) {
        const bool isA = b < a.nbA;
        const int i = (isA ? b : b - a.nbA) * 256 + threadIdx.x;
        const int n = isA ? a.M : a.N, npad = isA ? a.Mp : a.Np;
        if (i >= npad) return;
        float l = 0.0f, st = 0.0f;
        if (i < n) make_scales((isA ? a.amaxA : a.amaxB)[i], a.qmaxf, l, st);
        (isA ? a.lamA : a.lamB)[i] = l;
        (isA ? a.sA : a.sB)[i] = st;
        return;
    }
    b -= a.nbA + a.nbB;
    if (b < a.nbP) {
        // one lane's eight k of an operand, of both factors
        const int idx = b * 256 + threadIdx.x, NT = a.RP / 16;
        if (idx >= a.Kp / 64 * NT * 128) return;
        const int lane = idx & 63, h = (idx >> 6) & 1, blk = idx >> 7;           // blk: k block and column tile
        const int c = 16 * (blk % NT) + (lane & 15), k0 = 64 * (blk / NT) + 16 * (lane >> 4) + 8 * h;
        float w[8], v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int k = min(k0 + e, a.K - 1), cc = min(c, a.r - 1);
            const bool in = c < a.r && k0 + e < a.K;
            const float wv = a.W[(size_t)k * a.r + cc], vv = a.Vt[(size_t)cc * a.K + k];
            w[e] = in ? wv : 0.f;
            v[e] = in ? vv : 0.f;
        }
        const Planes3 pw = split_planes<3>(w), pv = split_planes<3>(v);
        const size_t at = (size_t)(blk * 6 + h) * FACTOR_PIECE + lane * 8;
        *reinterpret_cast<v8bf16*>(a.Wf + at) = pw.p1;
        *reinterpret_cast<v8bf16*>(a.Wf + at + 2 * FACTOR_PIECE) = pw.p2;
        *reinterpret_cast<v8bf16*>(a.Wf + at + 4 * FACTOR_PIECE) = pw.p3;
        *reinterpret_cast<v8bf16*>(a.Vf + at) = pv.p1;
        *reinterpret_cast<v8bf16*>(a.Vf + at + 2 * FACTOR_PIECE) = pv.p2;
        *reinterpret_cast<v8bf16*>(a.Vf + at + 4 * FACTOR_PIECE) = pv.p3;
        return;
    }
    b -= a.nbP;
    const int t = b % a.r, ks = b / a.r;
    if (a.r <= 32)      vtw_block<32>(a.Vt, a.W, a.K, a.r, a.kslice, t, ks, a.Xp, part);
    else if (a.r <= 64) vtw_block<64>(a.Vt, a.W, a.K, a.r, a.kslice, t, ks, a.Xp, part);
    else                vtw_block<128>(a.Vt, a.W, a.K, a.r, a.kslice, t, ks, a.Xp, part);
}

int vtw_slices(int K) { return max(1, min(LRQ_VTW_MAX_SLICES, K / 256)); }

int launch_panel_prep(int M, int N, int K, int r, int RP, float qmaxf, const float* amaxA, const float* amaxB,
                      const float* W, const float* Vt, float* lamA, float* sA, float* lamB, float* sB,
                      uint16_t* Wf, uint16_t* Vf, float* Xp, hipStream_t st) {
    PrepArgs a;
    a.amaxA = amaxA; a.amaxB = amaxB; a.W = W; a.Vt = Vt;
    a.lamA = lamA; a.sA = sA; a.lamB = lamB; a.sB = sB; a.Xp = Xp;
    a.Wf = Wf; a.Vf = Vf; a.Kp = (K + 63) / 64 * 64;
    a.M = M; a.Mp = (M + 3) / 4 * 4; a.N = N; a.Np = (N + 3) / 4 * 4; a.K = K; a.r = r; a.RP = RP;
    a.qmaxf = qmaxf;
    a.nbA = ceil_div(a.Mp, 256);
    a.nbB = ceil_div(a.Np, 256);
    a.nbP = ceil_div(a.Kp / 64 * (RP / 16) * 128, 256);
    a.kslice = ceil_div(K, vtw_slices(K));
    a.nslices = ceil_div(K, a.kslice);
    const int total = a.nbA + a.nbB + a.nbP + r * a.nslices;
    hipLaunchKernelGGL(panel_prep_kernel, dim3(total), dim3(256), 0, st, a);
    LRQ_CHECK_LAUNCH();
    return LRQMM_OK;
}

static void dispatch_gemm256(bool comp, bool wcint, dim3 grid, hipStream_t st, int M, int N, int K,
                             const int8_t* Aq, const int8_t* BqT, const float* sA, const float* sB,
                             const float* Lp, const float* Rp, int R2P, GemmOut C, int32_t* Cint, int tiles_n,
                             int ntiles, float qmaxf, int packed) {
    const bool full = aligned16(Aq) && aligned16(BqT) && (M % BTM == 0) && (N % BTN == 0) && (K % BBK == 0);
#define LRQ_PACKED(FMT, COMP, WC)                                                                            \
    hipLaunchKernelGGL((packed_gemm256_kernel<FMT, COMP, WC>), grid, dim3(512), 0, st, M, N, K,              \
                       reinterpret_cast<const uint8_t*>(Aq), reinterpret_cast<const uint8_t*>(BqT), sA, sB, Lp, Rp, R2P, C, Cint, \
                       tiles_n, ntiles, ntiles, 1, nullptr, qmaxf)
#define LRQ_GEMM(COMP, WC)                                                                                   \
    do {                                                                                                     \
        if (full)                                                                                            \
            hipLaunchKernelGGL((int8_gemm256_kernel<COMP, WC, true>), grid, dim3(512), 0, st, M, N, K, Aq,   \
                               BqT, sA, sB, Lp, Rp, R2P, C, Cint, tiles_n, ntiles, qmaxf);                   \
        else                                                                                                 \
            hipLaunchKernelGGL((int8_gemm256_kernel<COMP, WC, false>), grid, dim3(512), 0, st, M, N, K,      \
                               Aq, BqT, sA, sB, Lp, Rp, R2P, C, Cint, tiles_n, ntiles, qmaxf);               \
    } while (0)
    if (packed) {           // (Cint: raw sums)
        if (packed == PK6) { if (comp) LRQ_PACKED(PK6, true, false); else if (wcint) LRQ_PACKED(PK6, false, true); else LRQ_PACKED(PK6, false, false); }
        else               { if (comp) LRQ_PACKED(PK8, true, false); else if (wcint) LRQ_PACKED(PK8, false, true); else LRQ_PACKED(PK8, false, false); }
    } else if (comp) {
        if (wcint) LRQ_GEMM(true, true); else LRQ_GEMM(true, false);
    } else {
        if (wcint) LRQ_GEMM(false, true); else LRQ_GEMM(false, false);
    }
#undef LRQ_GEMM
#undef LRQ_PACKED
}

template <bool WIDE, int MTW, int NTW, int PACKED>
static void dispatch_gemm(bool comp, bool wcint, dim3 grid, hipStream_t st, int M, int N, int K,
                          const int8_t* Aq, const int8_t* BqT, const float* sA, const float* sB,
                          const float* Lp, const float* Rp, int R2P, GemmOut C, int32_t* Cint, int tiles_n,
                          int ntiles, float qmaxf) {
#define LRQ_GEMM(COMP, WC) hipLaunchKernelGGL((int8_gemm_kernel<WIDE, COMP, WC, MTW, NTW, PACKED>), grid, dim3(256), 0, st, M, N, K, \
                                              Aq, BqT, sA, sB, Lp, Rp, R2P, C, Cint, tiles_n, ntiles, qmaxf)
    if constexpr (PACKED != PK_NONE) {      // (without Cint)
        if (comp) LRQ_GEMM(true, false); else LRQ_GEMM(false, false);
    } else if (comp) {
        if (wcint) LRQ_GEMM(true, true); else LRQ_GEMM(true, false);
    } else {
        if (wcint) LRQ_GEMM(false, true); else LRQ_GEMM(false, false);
    }
#undef LRQ_GEMM
}

// Tiles [first, ntiles) (in xcd_tile order) of C_int <- sum over the K ranges of their partial sums.
__global__ __launch_bounds__(256) void sum_tile_slices_kernel(int32_t* __restrict__ Cint, int N, int tiles_n, int ntiles,
                                                              int first, const int32_t* __restrict__ part, int slices) {
    const int tile = xcd_tile(first + blockIdx.y, tiles_n, ntiles);
    const int m0 = (tile / tiles_n) * BTM, n0 = (tile % tiles_n) * BTN;
    const int e = blockIdx.x * 256 + threadIdx.x;            // 16-byte group of the tile
    const int row = e / (BTN / 4), c4 = e % (BTN / 4);
    const int4* src = reinterpret_cast<const int4*>(part + (size_t)blockIdx.y * slices * (BTM * BTN)) + e;
    int4 acc = make_int4(0, 0, 0, 0);
    for (int s0 = 0; s0 < slices; s0 += 8) {                 // eight loads in flight
        int4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = src[(size_t)min(s0 + u, slices - 1) * (BTM * BTN / 4)];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (s0 + u < slices) { acc.x += v[u].x; acc.y += v[u].y; acc.z += v[u].z; acc.w += v[u].w; }
    }
    *reinterpret_cast<int4*>(Cint + (size_t)(m0 + row) * N + n0 + 4 * c4) = acc;
}

namespace {
struct SumsPlan { int tiles_n, ntiles, left, slices; };
// Which tiles of the raw-sum product are cut along K when only `resident` CUs are free.
SumsPlan plan_sums(int M, int N, int K, const int8_t* Aq, const int8_t* BqT, int resident) {
    const bool full = aligned16(Aq) && aligned16(BqT) && int8_gemm_large_tiles(M, N) && M % BTM == 0 && N % BTN == 0 && K % BBK == 0;
    SumsPlan p = {N / BTN, (M / BTM) * (N / BTN), 0, 1};
    // (with many rounds the last one matters little, and the free CUs change along the way)
    if (full && resident > 0 && p.ntiles > resident && p.ntiles < 4 * resident) {
        p.left = p.ntiles % resident;
        // as many ranges as fill the chip once, each at least four K-tiles deep
        if (p.left > 0) p.slices = max(1, min(min(K / BBK / 4, resident / p.left), LRQ_SUMS_MAX_PARTS / p.left));
    }
    if (p.slices < 2) p.left = 0;
    return p;
}
}  // namespace

size_t int8_gemm_sums_scratch_bytes(int M, int N, int K) {
    // (whole tiles only; counted for ragged problems too, which contain smaller ones of whole tiles)
    const bool shape = int8_gemm_large_tiles(M / BTM * BTM, N / BTN * BTN) && K >= 8 * BBK;
    return shape ? (size_t)LRQ_SUMS_MAX_PARTS * BTM * BTN * sizeof(int32_t) : 0;
}

int launch_int8_gemm_sums(int M, int N, int K, const int8_t* Aq, const int8_t* BqT, int32_t* Cint, int resident,
                          int32_t* part, hipStream_t st, int packed) {
    if (packed == PK_NONE) return LRQMM_ERR_UNSUPPORTED;
    const SumsPlan p = part ? plan_sums(M, N, K, Aq, BqT, resident) : SumsPlan{0, 0, 0, 1};
    if (p.left == 0)
        return launch_int8_gemm(M, N, K, Aq, BqT, nullptr, nullptr, nullptr, nullptr, 0, GemmOut{nullptr, N, 1.0f, 0.0f},
                                Cint, 0.0f, st, packed);
    const int full_tiles = p.ntiles - p.left;
#define LRQ_SUMS(FMT)                                                                                                                 \
    hipLaunchKernelGGL((packed_gemm256_kernel<FMT, false, true, true>), dim3(full_tiles + p.left * p.slices), dim3(512), 0, st, M, N, \
                       K, reinterpret_cast<const uint8_t*>(Aq), reinterpret_cast<const uint8_t*>(BqT), nullptr, nullptr, nullptr,     \
                       nullptr, 0, GemmOut{nullptr, N, 1.0f, 0.0f}, Cint, p.tiles_n, p.ntiles, full_tiles, p.slices, part, 0.0f)
    if (packed == PK6) LRQ_SUMS(PK6);
    else               LRQ_SUMS(PK8);
#undef LRQ_SUMS
    LRQ_CHECK_LAUNCH();
    return LRQMM_OK;
}

int launch_int8_gemm_sums_finish(int M, int N, int K, const int8_t* Aq, const int8_t* BqT, int32_t* Cint, int resident,
                                 const int32_t* part, hipStream_t st) {
    const SumsPlan p = part ? plan_sums(M, N, K, Aq, BqT, resident) : SumsPlan{0, 0, 0, 1};
    if (p.left == 0) return LRQMM_OK;
    hipLaunchKernelGGL(sum_tile_slices_kernel, dim3(BTM * BTN / 4 / 256, p.left), dim3(256), 0, st, Cint, N, p.tiles_n,
                       p.ntiles, p.ntiles - p.left, part, p.slices);
    LRQ_CHECK_LAUNCH();
    return LRQMM_OK;
}

// Six bits for codes of at most five whose sums stay within 2^24, bytes otherwise.  Products of random 8-bit codes at rank 0,
// us, from rows of bytes (staged through registers) / from blocks of bytes (copied to LDS as they are): 300^3 4.3 / 4.0, 1024^3 5.9 /
// 5.7, 2000^3 20.8 / 16.9, 1537 x 1021 x 2311 19.6 / 11.2 (rows of an odd length), 512 x 4096 x 4096 19.8 / 16.4, 3072 x 1536 x 2048
// 25.1 / 19.1, 3000^3 53.4 / 44.7, 5000^3 164 / 138, 8192^3 507 / 474; at 4096^3 and beyond the chip's power bounds both (77 to 87).
int packed_format(int bits, int K) { return bits <= 5 && ((long long)K << (2 * (bits - 1))) <= (1ll << 24) ? PK6 : PK8; }

// Direct quantization: a workgroup of the packing kernel takes eight rows of A through LDS, four of more than 4096, which costs a tall A
// with short rows or with such long ones more than a narrow product gains.  Rank 0, 8 bits, rows of bytes / packed, us: 100352 x 64 K = 64
// 35.7 / 41.0, 256 41.3 / 46.7, 512 61.5 / 65.8, 768 95.5 / 90.7; 100352 x 512 128 81.7 / 86.6, 384 125 / 132, 512 143 / 144; 40000 x 768 384 59.7 / 63.3,
// 512 65.7 / 67.0; 40000 x 1024 512 84.7 / 88.1, 768 112 / 114; 100352 x 1024 256 155 / 156, 512 215 / 213; 100352 x 2048 64 239 / 215; long rows 16384
// x 64 4112 82.0 / 106, 8000 170 / 178, 12000 253 / 261; 16384 x 300 4864 132 / 150, 8192 221 / 231, 12000 347 / 328; 5000 x 256 4864 50.4 / 58.0, 12000 121 /
// 128; 3200 x 64 4112 36.1 / 39.0; 3000 x 64 8000 56.1 / 55.0.  4 bits: 100352 x 64 K = 384 48.0 / 52.5, 512 60 / 59; 100352 x 512 256 104 / 107,
// 384 125 / 125; 16384 x 256 4112 102 / 120, 8000 202 / 194; 8192 x 256 8192 104 / 112.  Up to 8192 short rows either takes the same time, which is that of the launches.
// Rows of bytes that are no multiple of four read slower, so that these stay only where nothing but A counts: 100352 x 16 207 40.8 / 44.1, 333
// 47.8 / 50.7, 461 57.0 / 54.7; 100352 x 64 333 50.8 / 53.3; 100352 x 256 207 64.8 / 65.4; 40000 x 16 207 22.9 / 23.8; 16384 x 64 5001 111 / 120; rows of
// less than 16, read byte by byte, nowhere: 40000 x 16 K = 11 29.7 / 21.1.
int direct_format(int M, int N, int K, int bits) {
    const int format = packed_format(bits, K);
    const bool six = format == PK6;
    if (K < 16) return format;
    if (K % 4 != 0) return N <= 64 && ((M >= 65536 && K <= 384) || (M >= 16384 && K > 4096)) ? PK_NONE : format;
    if (K > 4096) {
        const int widest = K <= 6144 ? 384 : six ? (M < 16384 && K <= 8192 ? 256 : 64) : K <= 8192 ? 384 : 256;
        return M >= 3072 && N <= widest ? PK_NONE : format;
    }
    return M >= 16384 && (six ? N <= 512 && K <= 384 : N <= 768 && K <= 512) ? PK_NONE : format;
}

long long int8_gemm_tiles(int M, int N) { return (long long)ceil_div(M, BTM) * ceil_div(N, BTN); }
// The large-tile kernel pays from half a round of its tiles on (raw sums, where it is the only one that is asked for)
bool int8_gemm_large_tiles(int M, int N) { return M >= BTM && N >= BTN && int8_gemm_tiles(M, N) >= GEMM_CUS / 2; }
// ... and with the result in C where the 128 x 128 tiles would no longer all be resident, two per CU: up to 512 of them those
// are the faster kernel, from a third round on they are not.  lrqmm_gemm at K = 4096, large / 128 x 128 tiles, us, ranks 0, 16
// and 40: 483 (2570 x 2830) 57.5 / 49.1, 91.5 / 73.4, 116 / 101; 512 (4096 x 2048) 54.7 / 47.3, 88.8 / 72.0, 114 / 101; 516
// (33024 x 256) 54.9 / 68.4, 130 / 138, 206 / 223; 528 (2816 x 3072) 54.9 / 64.9, 89.1 / 93.7, 114 / 125; 576 (3072^2) 55.2 /
// 64.9, 89.1 / 93.5, 113 / 125.  At K = 256 512 tiles 16.6 / 12.3, 43.2 / 32.1, 56.6 / 48.8, 528 16.1 / 16.0, 43.2 / 38.0, 56.8
// / 58.5.
static bool large_tiles_into_c(int M, int N) {
    return int8_gemm_large_tiles(M, N) && (long long)ceil_div(M, 128) * ceil_div(N, 128) > 2 * GEMM_CUS;
}

// The early-GEMM schedule needs the large-tile kernel and 16-byte accesses to the rows of C.
bool rank_update_usable(int M, int N, const float* C) {
    return int8_gemm_large_tiles(M, N) && N % 4 == 0 && ((uintptr_t)C & 15) == 0;
}

int launch_rank_update(int M, int N, float* C, const float* sA, const float* sB, const float* Lp, const float* Rp,
                       int R2P, float alpha, hipStream_t st) {
    const int tiles_n = ceil_div(N, 128);
    if (R2P > 64)       // wide panels: bound by the float32 matrix cores, so the plane products on the bf16 ones
        hipLaunchKernelGGL(rank_update_bf16_kernel, dim3(ceil_div(M, 128) * tiles_n), dim3(256), 0, st, M, N, C, sA, sB,
                           Lp, Rp, R2P, tiles_n, alpha);
    else
        hipLaunchKernelGGL(rank_update_kernel, dim3(ceil_div(M, 128) * tiles_n), dim3(256), 0, st, M, N, C, sA, sB, Lp,
                           Rp, R2P, tiles_n, alpha);
    LRQ_CHECK_LAUNCH();
    return LRQMM_OK;
}

// Few tiles with a long reduction stay with one launch per product and its smaller tiles: 256 x 256 x 6000 160 us against 188
// (4 tiles); 256 x 4096 x 4096 170 against 157 (64 tiles).
bool int8_terms_usable(int M, int N, int K) {
    return K >= 16 && (K <= 2048 || (long long)ceil_div(M, 128) * ceil_div(N, TTN) >= 32);
}

// int8_terms_kernel: 256-row tiles, one per CU, where they fill their last round to 3/4, 256 / 128 rows, us: 2000^3 (0.50) 113 / 99, 2560^3
// (0.78) 132 / 142, 3072^3 (0.56) 256 / 234, 3500^3 (0.77) 349 / 381, 4096^3 (1) 377 / 401, 5000^3 (0.78) 895 / 903
static bool tall_terms(int M, int N) {
    const long long tiles = (long long)ceil_div(M, 256) * ceil_div(N, TTN);
    return 4 * tiles >= 3 * GEMM_CUS * ((tiles + GEMM_CUS - 1) / GEMM_CUS);
}

// The format of the codes of four products: packed_terms_kernel reads less and multiplies faster, but nothing covers the end of its
// tiles (one workgroup per CU, the quadrants through LDS), so rows of bytes stay the better form of short reductions.  How short depends
// on the rounds of 128 x 128 tiles that each of the kernels makes of D (of int8_terms_kernel's a 256-row tile counts for two, and
// so do two tiles that share a CU).  Whole calls, rows of bytes / packed, us:
//   one round, up to 256 tiles: 2000^2 8 bits K = 256 31.6 / 34.8, 384 36.4 / 38.6, 512 41.5 / 41.9, 768 51.7 / 49.1; 4 bits 256 31.9 / 33.8, 384
//     36.2 / 36.5, 512 41.2 / 39.2; 1024^2 the same limits
//   as many rounds: 4096^2 (4 and 4) 8 bits K = 128 46.0 / 71.7, 512 75.5 / 100, 1024 114.5 / 134, 2048 196 / 200, 3072 278 / 275; 4 bits 512
//     71.0 / 87.3, 1024 109 / 110, 1536 148 / 133; 2560^2, 4000^2, 8192^2 and 100352 x 64 about the same limits
//   fewer: 3000^2 (3 and 4) 8 bits K = 512 65.2 / 75.6, 1024 95.8 / 97.7, 1536 132 / 124; 4 bits 512 62.2 / 66.6, 768 77.0 / 74.7; 3072^2,
//     5000^2 and 6144^2 within 200 of K
//   half as many (outputs of up to 128 rows, where 256-row tiles are half empty): 64 x 50000 8 bits K = 64 45.7 / 43.0, 512 129 / 114
// Rows of bytes that are no multiple of 16, and of an odd number of them even more, read slower, and the limits lie lower:
//   one round: 2000^2 8 bits K = 200 32.5 / 34.1, 500 42.8 / 41.9, 63 30.7 / 29.8, 461 46.1 / 41.0; 300^2 129 29.9 / 27.5
//   as many: 4096^2 8 bits K = 700 104 / 114, 1500 173 / 167, 461 94.9 / 99.6, 1001 151 / 134; 4 bits 500 77.2 / 86.5, 700 97.2 / 96.2, 333 75.6 / 80.9, 461
//     87.5 / 85.8
//   fewer: 5000^2 8 bits K = 500 141 / 156, 700 180 / 180, 333 138 / 141, 461 166 / 156; 4 bits 500 131 / 135, 700 171 / 152, 207 108 / 117, 333 131 / 126
int terms_format(int M, int N, int K, int bits) {
    static const int limits[3][2][3] = {        // [one round, fewer, as many][bytes, six bits][K a multiple of 16, of 4, of neither]
        {{512, 256, 0}, {384, 192, 0}}, {{1408, 704, 352}, {896, 544, 288}}, {{2560, 1280, 640}, {1024, 704, 448}}};
    const int format = packed_format(bits, K);
    const long long tiles = (long long)ceil_div(M, 128) * ceil_div(N, 128), tall = (long long)ceil_div(M, 256) * ceil_div(N, 128);
    const long long rounds = (tiles + GEMM_CUS - 1) / GEMM_CUS;
    const long long byte_rounds = tall_terms(M, N) ? 2 * ((tall + GEMM_CUS - 1) / GEMM_CUS)
                                                   : tiles <= GEMM_CUS ? 1 : 2 * ((tiles + 2 * GEMM_CUS - 1) / (2 * GEMM_CUS));
    if (rounds > 1 && 2 * rounds <= byte_rounds) return format;
    return K >= limits[rounds == 1 ? 0 : rounds < byte_rounds ? 1 : 2][format == PK6][K % 16 == 0 ? 0 : K % 4 == 0 ? 1 : 2] ? format : PK_NONE;
}

int launch_int8_terms(int M, int N, int K, const int8_t* const A[2], const float* const amaxA[2], const int8_t* const B[2],
                      const float* const amaxB[2], int terms, float qmaxf, GemmOut out, hipStream_t st, int packed) {
    if (!int8_terms_usable(M, N, K) || (packed && terms != 4)) return LRQMM_ERR_UNSUPPORTED;
    TermArgs t = {{A[0], A[1]}, {B[0], B[1]}, {amaxA[0], amaxA[1]}, {amaxB[0], amaxB[1]}};
    if (packed) {
        const int tn = ceil_div(N, 128), nt = ceil_div(M, 128) * tn;
        if (packed == PK6) hipLaunchKernelGGL(packed_terms_kernel<PK6>, dim3(nt), dim3(512), 0, st, M, N, K, t, qmaxf, out, tn, nt);
        else               hipLaunchKernelGGL(packed_terms_kernel<PK8>, dim3(nt), dim3(512), 0, st, M, N, K, t, qmaxf, out, tn, nt);
        LRQ_CHECK_LAUNCH();
        return LRQMM_OK;
    }
    const int tiles_n = ceil_div(N, TTN);
    const bool tall = tall_terms(M, N);
    const int ttm = tall ? 256 : 128, ntiles = ceil_div(M, ttm) * tiles_n;
    const bool full = aligned16(A[0]) && aligned16(A[1]) && aligned16(B[0]) && aligned16(B[1]) && M % ttm == 0 && N % TTN == 0 && K % BBK == 0;
#define LRQ_TERMS(WM, FULL)                                                                                                  \
    hipLaunchKernelGGL((int8_terms_kernel<WM, FULL>), dim3(ntiles), dim3(128 * WM), 0, st, M, N, K, t, terms, qmaxf, out, tiles_n, \
                       ntiles)
    if (tall) { if (full) LRQ_TERMS(4, true); else LRQ_TERMS(4, false); }
    else      { if (full) LRQ_TERMS(2, true); else LRQ_TERMS(2, false); }
#undef LRQ_TERMS
    LRQ_CHECK_LAUNCH();
    return LRQMM_OK;
}

// K == 0: every sum is empty.  One thread per output element.
__global__ __launch_bounds__(256) void empty_product_kernel(int M, int N, GemmOut out, int32_t* __restrict__ Cint) {
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (size_t)M * N) return;
    const int row = (int)(idx / N), col = (int)(idx % N);
    if (Cint) Cint[idx] = 0;
    if (out.C) store_out(out, row, col, 0.0f);
}

int launch_empty_product(int M, int N, GemmOut C, int32_t* Cint, hipStream_t st) {
    const size_t total = (size_t)M * N;
    if (total == 0) return LRQMM_OK;
    hipLaunchKernelGGL(empty_product_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, M, N, C, Cint);
    LRQ_CHECK_LAUNCH();
    return LRQMM_OK;
}

int launch_int8_gemm(int M, int N, int K, const int8_t* Aq, const int8_t* BqT, const float* sA,
                     const float* sB, const float* Lp, const float* Rp, int R2P, GemmOut C, int32_t* Cint,
                     float qmaxf, hipStream_t st, int packed) {
    // the GEMM kernels issue their first operand loads unconditionally: an empty reduction never reaches them
    if (K <= 0) return launch_empty_product(M, N, C, Cint, st);
    // (the 16-byte load path clamps its address to K - 16, so it needs at least one whole group)
    const bool wide = K >= 16;
    const bool comp = Lp != nullptr;
    // big problems: 256x256 tiles, one workgroup per CU
    const bool large = (C.C ? large_tiles_into_c(M, N) : int8_gemm_large_tiles(M, N)) && wide;
    if (packed && Cint && (C.C || !large)) return LRQMM_ERR_UNSUPPORTED;        // (packed codes: the result or the raw sums)
    if (large) {
        const int btiles = (int)int8_gemm_tiles(M, N);
        const int btn = ceil_div(N, BTN);
        dim3 bgrid(btiles);
        dispatch_gemm256(comp, Cint != nullptr, bgrid, st, M, N, K, Aq, BqT, sA, sB, Lp, Rp, R2P, C, Cint, btn, btiles, qmaxf, packed);
        LRQ_CHECK_LAUNCH();
        return LRQMM_OK;
    }
    // Smaller outputs: the largest of the smaller tiles of which there are at least 256, one per CU.  Calls with 128 x 128 tiles throughout / with this rule: 4 tiles of
    // 128 x 128 (256^3) 87 / 81 us, 104 (1537 x 1021 x 2311) 279 / 258, 128 (512 x 4096 x 4096 layer) 233 / 222;
    // 256 (2000^3) is the same path.
    // At most 64 columns: 64 rows too, four workgroups per CU (128 x 64 / 64 x 64: 100352 x 64 x 576 213.5 / 208.8 us a call).
    int mtw = N <= 64 ? 1 : 2, ntw = mtw;
    auto tiles = [&] { return (long long)ceil_div(M, 64 * mtw) * ceil_div(N, 64 * ntw); };
    if (tiles() < GEMM_MIN_TILES) mtw = 1;
    if (tiles() < GEMM_MIN_TILES) ntw = 1;
    if (!wide) mtw = ntw = 2;           // (K < 16: one staged tile)
    const int tiles_n = ceil_div(N, 64 * ntw), ntiles = (int)tiles();
    dim3 grid(ntiles);
#define LRQ_DG(W, MT, NT, PK) dispatch_gemm<W, MT, NT, PK>(comp, Cint != nullptr, grid, st, M, N, K, Aq, BqT, sA, sB, Lp, Rp, R2P, C, Cint, tiles_n, ntiles, qmaxf)
#define LRQ_DGS(W, PK)                                       \
    do {                                                    \
        if (mtw == 2 && ntw == 2) LRQ_DG(W, 2, 2, PK);      \
        else if (ntw == 2)        LRQ_DG(W, 1, 2, PK);      \
        else                      LRQ_DG(W, 1, 1, PK);      \
    } while (0)
    if (packed == PK6)      LRQ_DGS(true, PK6);
    else if (packed == PK8) LRQ_DGS(true, PK8);
    else if (!wide)         LRQ_DG(false, 2, 2, PK_NONE);
    else                    LRQ_DGS(true, PK_NONE);
#undef LRQ_DGS
#undef LRQ_DG
    LRQ_CHECK_LAUNCH();
    return LRQMM_OK;
}
