// Residual products over the whole reduction (paper: Background 2.1 / Algorithm 1, the products R Z, R^T Q and Q^T R of the
// randomized range finder): the passes of passes.hip in a form that leaves no partial sums.
//
// A workgroup takes 16 RT results (rows of X, or columns in the transposed pass) over the whole reduction.  Its eight waves take
// every eighth 32-deep step of the reduction on their own: X straight from memory, the residuals split into bfloat16 planes in
// registers (see resid_mul_n_bf16_kernel for the plane arithmetic), the other operand as planes in operand order (STEP_PIECE),
// which its producer, orth_apply_kernel, has left: no LDS and no barrier before the waves' sums meet at the end.  There the
// workgroup holds whole rows of the result, so it also forms their float64 Gram matrix: a product needs no launch that adds
// partial results.
//
// What bounds it: the read of X (7.0 TB/s from the memory-side cache with 128 or 256 such workgroups) for few sketch columns; the
// planes, which every workgroup reads whole (100 to 119 GB/s a CU from the L2s, 6 bytes a value), and the matrix cores beyond.
#pragma once
#include <type_traits>
#include "kernels.h"

namespace {

struct FullJob {
    const float *X, *lam, *sc;
    const void* W;              // the other operand, in the order of steps
    float* Y;                   // n x LP; several ranges: [ranges][n][LP]
    double* gpart;              // [blocks][LP][LP], of a single range
    int ldx, n, len;            // results, reduction
    int rt, nb;                 // tiles of 16 results per workgroup, workgroups of a range
    int group;                  // tiles per Gram partial
    int ranges, chunk;          // of the reduction, whole steps per range (the last range also takes what is left over)
};

template <int V>
__device__ __forceinline__ void load_vec(const float* __restrict__ p, float (&v)[V]) {
    typedef float vu __attribute__((ext_vector_type(V), aligned(4)));
    const vu t = *reinterpret_cast<const vu*>(p);
#pragma unroll
    for (int i = 0; i < V; ++i) v[i] = t[i];
}
template <>
__device__ __forceinline__ void load_vec<1>(const float* __restrict__ p, float (&v)[1]) { v[0] = *p; }

// T: the transposed pass.  OUTER: the scales go with the results (else with the reduction).  Two steps of a wave are in flight.  With four
// (three for 48 columns and more) these were 126, 186 and 238 registers for 16, 32 and 48 columns, of 512 that a SIMD has for two such waves:
// beside 48 columns no wave of the other chain's passes fitted a CU (1024 x 4096 x 4096 l = 40 352 us in place of 324, 512 x 4096 x 4096 330
// / 313).  More steps gain nothing either where a call has the chip to itself, four / two, us: 256 x 512 x 8192 l = 8 147.0 / 141.3, 24
// 204.5 / 195.7, 2000^3 24 170.7 / 165.8, 40 235.1 / 230.0, 1000 x 700 x 6000 24 220.7 / 209.0, 300 x 5000 x 1200 24 164.4 / 158.6; the exception
// is 4096 x 512 x 4096 l = 24 in two chains, 224.5 / 231.4.
// Scales that go with the reduction are loaded one value a lane and handed to the lanes through a few words of LDS of the wave's
// own: loads return in order, so every load of a step has to be issued as far ahead as its X, and eight lambdas and eight
// steps a lane would take 16 registers for each step in flight.
template <int NT, int RT, bool T, bool OUTER, int PL>
__device__ __forceinline__ void full_body(const FullJob& job, QuantParams q, int blk, int range, float* __restrict__ const lds) {
    constexpr int LP = 16 * NT, OB = 16 * RT, LD = LP + 4, U = 2;
    const float* __restrict__ const X = job.X;
    const float* __restrict__ const lam = job.lam;
    const float* __restrict__ const sc = job.sc;
    const int ldx = job.ldx, n = job.n, len = job.len;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int r = lane & 15, g = lane >> 4;
    const int o0 = blk * OB;
    // A lane's operands.  k-slot e of lane group g: reduction index 4 g + (e & 3) + 16 (e >> 2) of the step.
    // N: tile t is rows o0 + 16 t ..; T: tile t is columns {o0 + RT c + t}, so a lane's RT columns are adjacent (the lane that would
    // cross the end takes the last RT columns and stores what lies at or beyond its own first one).
    auto first_col = [&](int c) { return max(0, min(o0 + RT * c, n - RT)); };
    uint32_t xoff[T ? 1 : RT];
    if (T) xoff[0] = (uint32_t)(4 * g) * (uint32_t)ldx + (uint32_t)(first_col(r) - o0);
    else {
#pragma unroll
        for (int t = 0; t < RT; ++t) xoff[t] = (uint32_t)min(16 * t + r, n - 1 - o0) * (uint32_t)ldx + (uint32_t)(4 * g);
    }
    const float* const xb = T ? X + o0 : X + (size_t)o0 * ldx;       // wave-uniform
    float lo[RT], so[RT];           // OUTER
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        const int o = T ? first_col(r) + t : min(o0 + 16 * t + r, n - 1);
        lo[t] = OUTER ? lam[o] : 0.f;
        so[t] = OUTER ? sc[o] : 0.f;
    }
    // Float32 matrix cores round after every four products: four sums, so that the order of addition stays as shallow as that of short
    // ranges (100352 x 64 x 576, l = 8: distance of C from float64 with one sum 3.10e-7, with four 2.90e-7, passes.hip 2.88e-7).
    constexpr int SUMS = PL == 0 ? 4 : 1;
    v4f acc[RT][NT * SUMS];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int nt = 0; nt < NT * SUMS; ++nt) acc[t][nt] = (v4f){0.f, 0.f, 0.f, 0.f};

    struct Step {
        float x[RT][8];
        float scale;            // lane l: lambda of reduction index l (l < 32), step of l - 32
        v8bf16 b[NT][PL ? PL : 1];
        float w[PL ? 1 : 8];
    };
    struct Resid {
        Planes3 p;
        float r[PL ? 1 : 8];
    };
    float* const sl = lds + 4 * OB * LD + wave * 64;
    const float* const scq = lane < 32 ? lam : sc;
    // whole steps: constant lane offsets from wave-uniform bases
    auto load_x = [&](Step& f, int step) {
        const int k0 = 32 * step;
        if (T) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float v[RT];
                load_vec<RT>(xb + (size_t)(k0 + (e & 3) + 16 * (e >> 2)) * ldx + (int)xoff[0], v);
#pragma unroll
                for (int t = 0; t < RT; ++t) f.x[t][e] = v[t];
            }
        } else {
#pragma unroll
            for (int t = 0; t < RT; ++t)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const float4 v = load4u(xb + k0 + 16 * h + xoff[t]);
                    f.x[t][4 * h] = v.x; f.x[t][4 * h + 1] = v.y; f.x[t][4 * h + 2] = v.z; f.x[t][4 * h + 3] = v.w;
                }
        }
        if (!OUTER) f.scale = scq[k0 + (lane & 31)];
    };
    // the step that reaches past the reduction: clamped, the planes are zero there
    auto load_x_tail = [&](Step& f, int step) {
        const int k0 = 32 * step;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int k = min(k0 + 4 * g + (e & 3) + 16 * (e >> 2), len - 1);
#pragma unroll
            for (int t = 0; t < RT; ++t)
                f.x[t][e] = T ? X[(size_t)k * ldx + first_col(r) + t] : X[(size_t)min(o0 + 16 * t + r, n - 1) * ldx + k];
        }
        if (!OUTER) f.scale = scq[min(k0 + (lane & 31), len - 1)];
    };
    auto load_b = [&](Step& f, int step) {
        if constexpr (PL == 0) {
            const float4* w = reinterpret_cast<const float4*>(static_cast<const float*>(job.W) + (size_t)step * 512 + lane * 8);
            const float4 a = w[0], b = w[1];
            f.w[0] = a.x; f.w[1] = a.y; f.w[2] = a.z; f.w[3] = a.w;
            f.w[4] = b.x; f.w[5] = b.y; f.w[6] = b.z; f.w[7] = b.w;
            return;
        }
        const uint16_t* w = static_cast<const uint16_t*>(job.W) + (size_t)step * (NT * 3 * STEP_PIECE) + lane * 8;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int p = 0; p < PL; ++p) f.b[nt][p] = *reinterpret_cast<const v8bf16*>(w + (nt * 3 + p) * STEP_PIECE);
    };
    auto residuals = [&](const Step& f, Resid (&ap)[RT]) {
        float lk[8], sk[8];
        if constexpr (!OUTER) {
            sl[lane] = f.scale;
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const float4 a = *reinterpret_cast<const float4*>(sl + 16 * h + 4 * g), b = *reinterpret_cast<const float4*>(sl + 32 + 16 * h + 4 * g);
                lk[4 * h] = a.x; lk[4 * h + 1] = a.y; lk[4 * h + 2] = a.z; lk[4 * h + 3] = a.w;
                sk[4 * h] = b.x; sk[4 * h + 1] = b.y; sk[4 * h + 2] = b.z; sk[4 * h + 3] = b.w;
            }
            __builtin_amdgcn_wave_barrier();
        }
        auto form = [&](auto mode) {            // one uniform branch on the rounding mode per step
            constexpr int RM = decltype(mode)::value;
#pragma unroll
            for (int t = 0; t < RT; ++t) {
                float res[8];
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    res[e] = quant_residual_m<RM>(f.x[t][e], OUTER ? lo[t] : lk[e], OUTER ? so[t] : sk[e], q);
                if constexpr (PL > 0) ap[t].p = split_planes<PL>(res);
                else {
#pragma unroll
                    for (int e = 0; e < 8; ++e) ap[t].r[e] = res[e];
                }
            }
        };
        if (q.round_mode == 0) form(std::integral_constant<int, 0>{});
        else form(std::integral_constant<int, 1>{});
    };
    auto products = [&](const Step& f, const Resid (&ap)[RT]) {
        if constexpr (PL == 0) {
#pragma unroll
            for (int e = 0; e < 8; ++e)
#pragma unroll
                for (int t = 0; t < RT; ++t) acc[t][e % SUMS] = __builtin_amdgcn_mfma_f32_16x16x4f32(ap[t].r[e], f.w[e], acc[t][e % SUMS], 0, 0, 0);
        }
#define LRQ_FP(PA, PB)                                                                                          \
    _Pragma("unroll") for (int nt = 0; nt < NT; ++nt) _Pragma("unroll") for (int t = 0; t < RT; ++t)             \
        acc[t][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ap[t].p.PA, f.b[nt][PB], acc[t][nt], 0, 0, 0);
        if constexpr (PL >= 3) {
            LRQ_FP(p3, 0)
            LRQ_FP(p2, 1)
            LRQ_FP(p1, 2)
        }
        if constexpr (PL >= 2) {
            LRQ_FP(p2, 0)
            LRQ_FP(p1, 1)
        }
        if constexpr (PL >= 1) { LRQ_FP(p1, 0) }
#undef LRQ_FP
    };
    // this wave's steps of the range: begin + wave, + 8, ...; only the last step of all may be short
    const int begin = range * job.chunk, whole = min(len >> 5, begin + job.chunk) - begin;
    const bool last = range == job.ranges - 1 && (len & 31) != 0;
    const int cnt = (whole - wave + 7) >> 3;
    const int first = begin + min(wave, whole - 1);         // (a wave without a whole step loads another's; whole > 0)
    auto step_of = [&](int i) { return first + 8 * max(0, min(i, cnt - 1)); };
    Step f[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {       // (no branch: the waits below count the loads that are in flight)
        const int s = step_of(u);
        load_x(f[u], s);
        __builtin_amdgcn_sched_barrier(0);
        load_b(f[u], s);
        __builtin_amdgcn_sched_barrier(0);
    }
    int i = 0;
    for (; i + U <= cnt; i += U) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int s = step_of(i + U + u);       // (past the end: the wave's last step again, not used)
            Resid ap[RT];
            residuals(f[u], ap);
            load_x(f[u], s);
            __builtin_amdgcn_sched_barrier(0);
            products(f[u], ap);
            load_b(f[u], s);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (i + u < cnt) {
            Resid ap[RT];
            residuals(f[u], ap);
            products(f[u], ap);
        }
    if (last && (whole & 7) == wave) {
        load_x_tail(f[0], begin + whole);
        load_b(f[0], begin + whole);
        Resid ap[RT];
        residuals(f[0], ap);
        products(f[0], ap);
    }
    if constexpr (SUMS == 4) {
#pragma unroll
        for (int t = 0; t < RT; ++t) acc[t][0] = (acc[t][0] + acc[t][1]) + (acc[t][2] + acc[t][3]);
    }
    // The eight waves' sums meet in LDS: waves 4 to 7 leave theirs, 0 to 3 add their own, then four sums a value.
    auto each = [&](auto fn) {
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = 4 * g + v;
                int o = 16 * t + row;
                bool own = true;
                if (T) {
                    const int skip = o0 + RT * row - first_col(row);
                    o = RT * row + t - skip;
                    own = t >= skip;
                }
                if (own) {
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) fn(lds + (wave & 3) * (OB * LD) + o * LD + 16 * nt + r, acc[t][nt][v]);
                }
            }
    };
    if (wave >= 4) each([](float* p, float a) { *p = a; });
    __syncthreads();
    if (wave < 4) each([](float* p, float a) { *p += a; });
    __syncthreads();
    float* const Y = job.Y + (size_t)range * n * LP;
    for (int e = threadIdx.x; e < OB * LP / 4; e += 512) {
        const int o = e / (LP / 4), c = e % (LP / 4) * 4;
        float4 p[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) p[w] = *reinterpret_cast<const float4*>(lds + w * (OB * LD) + o * LD + c);
        const float4 v = make_float4((p[0].x + p[1].x) + (p[2].x + p[3].x), (p[0].y + p[1].y) + (p[2].y + p[3].y),
                                     (p[0].z + p[1].z) + (p[2].z + p[3].z), (p[0].w + p[1].w) + (p[2].w + p[3].w));
        const bool in = o0 + o < n;
        if (in) *reinterpret_cast<float4*>(Y + (size_t)(o0 + o) * LP + c) = v;
        *reinterpret_cast<float4*>(lds + o * LD + c) = in ? v : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    if (job.ranges > 1) return;         // partial results (launch_reduce_gram adds them up)
    __syncthreads();
    // Gram matrices of these rows, `group` tiles each, as in reduce_gram_kernel
    typedef double v4d __attribute__((ext_vector_type(4)));
    constexpr int NP = NT * (NT + 1) / 2;
    const int groups = min(RT / job.group, (n - o0 + 16 * job.group - 1) / (16 * job.group));
    for (int i = wave; i < NP * groups; i += 8) {
        const int grp = i / NP;
        int ta = 0, o = i % NP;
        while (o >= NT - ta) { o -= NT - ta; ++ta; }        // row ta of the upper triangle
        const int tb = ta + o;
        v4d ga = (v4d){0.0, 0.0, 0.0, 0.0};
        const float* row = lds + (16 * job.group * grp + g) * LD + r;
        for (int st = 0; st < job.group; ++st, row += 16 * LD) {
#pragma unroll
            for (int k = 0; k < 16; k += 4)
                ga = __builtin_amdgcn_mfma_f64_16x16x4f64((double)row[k * LD + 16 * ta], (double)row[k * LD + 16 * tb], ga, 0, 0, 0);
        }
        double* const gp = job.gpart + (size_t)(blk * (RT / job.group) + grp) * LP * LP;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int gi = 16 * ta + 4 * v + g, gj = 16 * tb + r;
            gp[gi * LP + gj] = ga[v];
            if (ta != tb) gp[gj * LP + gi] = ga[v];
        }
    }
}

constexpr int full_lds(int NT, int RT) { return 4 * 16 * RT * (16 * NT + 4) + 512; }

// Neighbouring strips of the transposed pass share lines of X: they go to the same XCD (workgroup i runs on XCD i % 8).
__device__ __forceinline__ int strip_of(int id, int nb) {
    const int per = nb >> 3, rest = nb & 7, x = id & 7, i = id >> 3;
    return x * per + min(x, rest) + i;
}

// Workgroups [0, nb0) work on job a (scales by row), the rest on job b (scales by column).
template <int NT, bool T, int PL, int RTA, int RTB>
__global__ __launch_bounds__(512, 2) void full_pair_kernel(FullJob a, FullJob b, int nb0, QuantParams q) {
    __shared__ __align__(16) float lds[full_lds(NT, RTA > RTB ? RTA : RTB)];
    if ((int)blockIdx.x < nb0) {
        const int id = blockIdx.x % a.nb, range = blockIdx.x / a.nb;
        full_body<NT, RTA, T, !T, PL>(a, q, T ? strip_of(id, a.nb) : id, range, lds);
    } else {
        const int id = (blockIdx.x - nb0) % b.nb, range = (blockIdx.x - nb0) / b.nb;
        full_body<NT, RTB, T, T, PL>(b, q, T ? strip_of(id, b.nb) : id, range, lds);
    }
}

// Tiles of 16 results per Gram partial: by the factor's own length, so that its Gram matrix does not depend on how a launch deals
// the tiles to workgroups.
inline int full_group(int n, int LP) { return LP == 16 || n <= 4096 ? 1 : 2; }

template <int NT, bool T, int PL>
int dispatch_full(FullJob (&j)[2], QuantParams q, hipStream_t st) {
    // As few tiles a workgroup as leave every CU one, the operand with more workgroups first.  Both operands at two tiles where either
    // is, us per call in place of (and half the kernels): 3072 x 1536 x 2048 24 columns 185 / 181, 40 258 / 252, 80 472 / 461, 2311 x 2600 x
    // 1800 8 130 / 126, 24 193 / 185, 40 262 / 254; squares of 2100 to 2700 1 % faster.  (The order of addition is the same.)
    auto blocks = [&](int i) { return j[i].n ? ceil_div(j[i].n, 16 * j[i].rt) * j[i].ranges : 0; };
    while (blocks(0) + blocks(1) > 256) {
        const int i = blocks(0) >= blocks(1) ? 0 : 1;
        if (j[i].rt >= 2) break;
        j[i].rt *= 2;
    }
    for (int i = 0; i < 2; ++i) j[i].nb = j[i].n ? ceil_div(j[i].n, 16 * j[i].rt) : 1;       // (an absent job: never indexed)
    const int nb0 = blocks(0);
    const dim3 grid(nb0 + blocks(1));
    const int ra = j[0].n ? j[0].rt : j[1].rt, rb = j[1].n ? j[1].rt : j[0].rt;
#define LRQ_FULL(RA, RB) hipLaunchKernelGGL((full_pair_kernel<NT, T, PL, RA, RB>), grid, dim3(512), 0, st, j[0], j[1], nb0, q)
    if (ra == 1 && rb == 1)      LRQ_FULL(1, 1);
    else if (ra == 2 && rb == 2) LRQ_FULL(2, 2);
    else if (ra == 1 && rb == 2) LRQ_FULL(1, 2);
    else if (ra == 2 && rb == 1) LRQ_FULL(2, 1);
    else return LRQMM_ERR_UNSUPPORTED;
#undef LRQ_FULL
    LRQ_CHECK_LAUNCH();
    return LRQMM_OK;
}

template <bool T>
int launch_full_t(const PassOperand* op, int nop, QuantParams q, int LP, hipStream_t st, int planes) {
    if (planes < 2) return LRQMM_ERR_UNSUPPORTED;
    FullJob j[2] = {};
    for (int i = 0; i < nop; ++i) {
        const PassOperand& o = op[i];
        const int n = T ? o.cols : o.rows, len = T ? o.rows : o.cols, group = full_group(n, LP), ranges = T ? o.ft : o.fn;
        if (ranges < 1) return LRQMM_ERR_UNSUPPORTED;
        const int chunk = ceil_div(len >> 5, ranges);
        float* const out = ranges > 1 ? o.partial : (T ? o.W : o.Y);
        j[o.axis] = {o.X, o.lam, o.s, o.steps, out, o.gpart, o.ldx, n, len, group, 0, group, ceil_div(len >> 5, chunk), chunk};
    }
    if (LP == 16) return planes == 3 ? dispatch_full<1, T, 0>(j, q, st) : dispatch_full<1, T, 2>(j, q, st);
#define LRQ_FULL_NT(NTV) case NTV: return planes == 3 ? dispatch_full<NTV, T, 3>(j, q, st) : dispatch_full<NTV, T, 2>(j, q, st)
    switch (LP / 16) {
        LRQ_FULL_NT(2); LRQ_FULL_NT(3); LRQ_FULL_NT(4); LRQ_FULL_NT(5);
        default: return LRQMM_ERR_UNSUPPORTED;
    }
#undef LRQ_FULL_NT
}

}  // namespace
