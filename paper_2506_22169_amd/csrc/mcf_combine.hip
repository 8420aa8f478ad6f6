// Second pass of a chain whose n range is split over blocks: every range has left its fp32 result
// (for a softmax normalised by its own row sum, with the base-2 logarithm of that sum beside it)
// in the workspace; here the ranges are put together and rounded once.
//
//     E[i,:] = sum_s w_s P_s[i,:] / sum_s w_s,   w_s = 2^(lse_s - max lse)      (softmax)
//     E[i,:] = sum_s P_s[i,:]                                                   (plain)
//
// Bound by being a launch: what its blocks wait for one after the other.  So a lane finds its row and its four columns with
// constants of the host in place of 64-bit divisions, and requests the logarithms and the values of up to four ranges (G) at once,
// of eight where there are more than four.  A wave reads whole row segments.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "mcf_internal.h"

namespace mcf {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// n / d of division_magic's constants
__device__ __forceinline__ uint32_t quotient(uint32_t n, uint32_t magic, int shift) { return magic ? __umulhi(n, magic) >> shift : n; }

template <typename T, bool SOFTMAX, int G>
__global__ __launch_bounds__(256) void combine_kernel(const CombineParams p) {
    const uint32_t r = quotient(threadIdx.x, p.quads_magic, p.quads_shift); // row of the block
    const int col = (int)(threadIdx.x - r * (uint32_t)(p.L >> 2)) * 4;
    const uint32_t row = blockIdx.x * (uint32_t)p.block_rows + r; // over all batches
    if (r >= (uint32_t)p.block_rows || row >= (uint32_t)p.rows) return;
    const float *src = p.part + (int64_t)row * p.pitch;
    f32x4 v[G];
    float lse[G];
    const auto fetch = [&](int s0, bool values) __attribute__((always_inline)) { // (beyond the last range: the last once more, unused)
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const float *q = src + (s0 + g < p.n_split ? s0 + g : p.n_split - 1) * p.split_stride;
            if (values) v[g] = *(const f32x4 *)(q + col);
            lse[g] = SOFTMAX ? q[p.L] : 0.f;
        }
        // (all of them here: left alone, the values are not requested before the logarithms have come)
        if (values) {
            if constexpr (G == 4) asm volatile("" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(lse[0]), "+v"(lse[1]), "+v"(lse[2]), "+v"(lse[3]));
            else
                asm volatile("" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]), "+v"(v[6]), "+v"(v[7]), "+v"(lse[0]), "+v"(lse[1]),
                             "+v"(lse[2]), "+v"(lse[3]), "+v"(lse[4]), "+v"(lse[5]), "+v"(lse[6]), "+v"(lse[7]));
        }
    };
    float m = -INFINITY;
    if (SOFTMAX) {
        for (int s0 = G; s0 < p.n_split; s0 += G) {
            fetch(s0, false);
#pragma unroll
            for (int g = 0; g < G; ++g) m = fmaxf(m, lse[g]);
        }
    }
    fetch(0, true);
    if (SOFTMAX) {
#pragma unroll
        for (int g = 0; g < G; ++g) m = fmaxf(m, lse[g]);
        if (m == -INFINITY) m = 0.f; // a row that sees no column: every weight is zero
    }
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    float wsum = 0.f;
    for (int s0 = 0;;) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (s0 + g >= p.n_split) continue;
            const float w = SOFTMAX ? __builtin_amdgcn_exp2f(lse[g] - m) : 1.f;
            wsum += w;
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] = SOFTMAX ? __builtin_fmaf(w, v[g][e], acc[e]) : acc[e] + v[g][e];
        }
        if ((s0 += G) >= p.n_split) break;
        fetch(s0, true);
    }
    const float inv = SOFTMAX ? (wsum > 0.f ? 1.0f / wsum : 0.f) : 1.f;
    const uint32_t b = quotient(row, p.m_magic, p.m_shift), i = row - b * (uint32_t)p.M;
    const int64_t at = b * p.se_b + i * p.se_r + col;
    if (p.out_f32) {
        f32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = acc[e] * inv;
        *(f32x4 *)((float *)p.E + at) = o;
    } else {
        typedef T T4 __attribute__((ext_vector_type(4)));
        T4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (T)(acc[e] * inv);
        *(T4 *)((T *)p.E + at) = o;
    }
}

} // namespace

int launch_combine(const CombineParams &p, int dtype, int softmax, void *stream) {
    const dim3 grid((unsigned)((p.rows + p.block_rows - 1) / p.block_rows)), block(256);
    hipStream_t st = (hipStream_t)stream;
    const auto run = [&](auto more) {
        constexpr int G = decltype(more)::value ? 8 : 4;
        if (dtype == MCF_F16) {
            if (softmax) hipLaunchKernelGGL((combine_kernel<_Float16, true, G>), grid, block, 0, st, p);
            else hipLaunchKernelGGL((combine_kernel<_Float16, false, G>), grid, block, 0, st, p);
        } else {
            if (softmax) hipLaunchKernelGGL((combine_kernel<__bf16, true, G>), grid, block, 0, st, p);
            else hipLaunchKernelGGL((combine_kernel<__bf16, false, G>), grid, block, 0, st, p);
        }
    };
    if (p.n_split > 4) run(std::true_type{});
    else run(std::false_type{});
    return (int)hipGetLastError();
}

} // namespace mcf
