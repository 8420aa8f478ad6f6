// Second pass of a chain whose n range is split over blocks: every range has left its fp32 result
// (for a softmax normalised by its own row sum, with the base-2 logarithm of that sum beside it)
// in the workspace; here the ranges are put together and rounded once.
//
//     E[i,:] = sum_s w_s P_s[i,:] / sum_s w_s,   w_s = 2^(lse_s - max lse)      (softmax)
//     E[i,:] = sum_s P_s[i,:]                                                   (plain)
//
// Bound by the bytes of the partial results (from L2 / the memory-side cache) and by being a launch:
// a lane owns four columns of a row, its ranges are requested four at a time, and a
// wave reads whole row segments.
#include <hip/hip_runtime.h>

#include "mcf_internal.h"

namespace mcf {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

template <typename T, bool SOFTMAX>
__global__ __launch_bounds__(256) void combine_kernel(const CombineParams p) {
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int quads = p.L >> 2;
    const int64_t row = idx / quads; // over all batches
    if (row >= p.rows) return;
    const int col = (int)(idx - row * quads) * 4;
    const float *src = p.part + row * p.pitch;
    float m = -INFINITY;
    if (SOFTMAX) {
        const float *lse = src + p.L;
        for (int s = 0; s < p.n_split; ++s) m = fmaxf(m, lse[s * p.split_stride]);
        if (m == -INFINITY) m = 0.f; // a row that sees no column: every weight is zero
    }
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    float wsum = 0.f;
#pragma unroll 4
    for (int s = 0; s < p.n_split; ++s) {
        const float *q = src + s * p.split_stride;
        const f32x4 v = *(const f32x4 *)(q + col);
        const float w = SOFTMAX ? __builtin_amdgcn_exp2f(q[p.L] - m) : 1.f;
        wsum += w;
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = SOFTMAX ? __builtin_fmaf(w, v[e], acc[e]) : acc[e] + v[e];
    }
    const float inv = SOFTMAX ? (wsum > 0.f ? 1.0f / wsum : 0.f) : 1.f;
    const int64_t b = row / p.M, i = row - b * p.M;
    const int64_t at = b * p.se_b + i * p.se_r + col;
    if (p.out_f32) {
        f32x4 r;
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = acc[e] * inv;
        *(f32x4 *)((float *)p.E + at) = r;
    } else {
        typedef T T4 __attribute__((ext_vector_type(4)));
        T4 r;
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = (T)(acc[e] * inv);
        *(T4 *)((T *)p.E + at) = r;
    }
}

} // namespace

int launch_combine(const CombineParams &p, int dtype, int softmax, void *stream) {
    const int64_t threads = p.rows * (p.L >> 2);
    const dim3 grid((unsigned)((threads + 255) / 256)), block(256);
    hipStream_t st = (hipStream_t)stream;
    if (dtype == MCF_F16) {
        if (softmax) hipLaunchKernelGGL((combine_kernel<_Float16, true>), grid, block, 0, st, p);
        else hipLaunchKernelGGL((combine_kernel<_Float16, false>), grid, block, 0, st, p);
    } else {
        if (softmax) hipLaunchKernelGGL((combine_kernel<__bf16, true>), grid, block, 0, st, p);
        else hipLaunchKernelGGL((combine_kernel<__bf16, false>), grid, block, 0, st, p);
    }
    return (int)hipGetLastError();
}

} // namespace mcf
