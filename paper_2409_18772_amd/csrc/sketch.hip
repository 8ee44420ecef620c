// Launches of the sketch and of small preparations (see sketch.h).
#include "sketch.h"

// Workgroups [0, nb) fill a sketch; the following ones (if any) derive the step vectors lambda = qmax/amax, s = amax/qmax of the
// operand it is for: the preparation of a factorization is one launch.
__global__ void fill_sketch_kernel(SketchFill f, int nb, const float* __restrict__ amax, int n, int npad, float qmaxf,
                                   float* __restrict__ lam, float* __restrict__ s) {
    if ((int)blockIdx.x >= nb) {
        const int i = ((int)blockIdx.x - nb) * blockDim.x + threadIdx.x;
        if (i >= npad) return;
        float l = 0.0f, st = 0.0f;
        if (i < n) make_scales(amax[i], qmaxf, l, st);
        lam[i] = l;
        s[i] = st;
        return;
    }
    fill_sketch_entry(f, (size_t)blockIdx.x * blockDim.x + threadIdx.x);
}

__global__ void pad_copy_kernel(const float* __restrict__ src, int rows, int cols, int ld,
                                float* __restrict__ dst) {
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t total = (size_t)rows * ld;
    if (idx >= total) return;
    const int i = (int)(idx / ld), j = (int)(idx % ld);
    dst[idx] = (j < cols) ? src[(size_t)i * cols + j] : 0.0f;
}

int launch_fill_sketch(uint64_t seed, int stream_id, int rows, int cols, int ld, float* omega,
                       hipStream_t st) {
    return launch_sketch_and_scales(seed, stream_id, rows, cols, ld, omega, nullptr, 0, 0, 0.f, nullptr, nullptr,
                                    st);
}

int launch_sketch_and_scales(uint64_t seed, int stream_id, int rows, int cols, int ld, float* omega,
                             const float* amax, int n, int npad, float qmaxf, float* lam, float* s,
                             hipStream_t st) {
    const SketchFill f = make_fill(seed, stream_id, rows, cols, ld, omega);
    const int nb = fill_blocks(f), nb_scale = amax ? (npad + 255) / 256 : 0;
    if (nb + nb_scale == 0) return LRQMM_OK;
    hipLaunchKernelGGL(fill_sketch_kernel, dim3(nb + nb_scale), dim3(256), 0, st, f, nb, amax, n, npad, qmaxf, lam, s);
    LRQ_CHECK_LAUNCH();
    return LRQMM_OK;
}

int launch_pad_copy(const float* src, int rows, int cols, int ld, float* dst, hipStream_t st) {
    const size_t total = (size_t)rows * ld;
    if (total == 0) return LRQMM_OK;
    hipLaunchKernelGGL(pad_copy_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, src, rows,
                       cols, ld, dst);
    LRQ_CHECK_LAUNCH();
    return LRQMM_OK;
}
