// The second stage of the backward pass' coefficient sums, for its own kernel and for the one that adds an MLP block's
// weight gradients.  Device code only.
#ifndef GRKAN_STAGE2_H_
#define GRKAN_STAGE2_H_

#include <hip/hip_runtime.h>

#include "grkan_walk.h"

namespace grkan {

// Stage 2.  One workgroup per group, of one wavefront when the group has at
// most 64 workspace rows and of four otherwise (the flat walk leaves one row
// per stage-1 workgroup; reading hundreds of rows with 64 lanes is a chain of
// dependent memory latencies).  Thread t adds rows t, t + T, ... in double; the
// T thread sums go through LDS, each block of 64 of them is added in thread
// order, then the blocks in block order.  Every order is fixed by T and the row
// count; dA / dB are overwritten.
// With one numerator row shared by the groups (G_shared > 0) the workgroups below
// G_shared write dB only, and M + 1 more, of four wavefronts, add one numerator
// sum each over the rows of all groups the same way.
constexpr int kStage2MaxThreads = 4 * kWave;

__device__ __forceinline__ uint16_t to_bf16(float v) { return __builtin_bit_cast(uint16_t, static_cast<__bf16>(v)); }

// A coefficient's gradient in the coefficients' type.
__device__ __forceinline__ void store_coef_grad(void *p, int32_t i, double v, int32_t bf16)
{
    if (bf16)
        static_cast<uint16_t *>(p)[i] = to_bf16((float)v);
    else
        static_cast<float *>(p)[i] = (float)v;
}

// What workgroup g does; all its threads come here.
template <int M, int N>
__device__ __forceinline__ void stage2_block(const float *__restrict__ partial, int32_t rows_per_group, void *__restrict__ dA,
                                             void *__restrict__ dB, int32_t G_shared, int32_t bf16, const int g)
{
    constexpr int kNumCoef = M + 1 + N;
    constexpr int kBlocks = kStage2MaxThreads / kWave;
    __shared__ double thread_sum[kNumCoef][kStage2MaxThreads];
    __shared__ double block_sum[kNumCoef][kBlocks];
    const int tid = threadIdx.x;
    const int T = blockDim.x; // 64 or 256
    if (G_shared > 0 && g >= G_shared) {
        const int k = g - G_shared;
        if (bf16) {
            // bfloat16: every group's gradient is rounded, then the rounded ones are added in float32 (what
            // converting and summing the groups' gradients gives); a wavefront takes every T / 64th group
            float t = 0.0f;
            for (int c = tid / kWave; c < G_shared; c += T / kWave) {
                double s = 0.0;
#pragma unroll 4
                for (int r = tid & (kWave - 1); r < rows_per_group; r += kWave)
                    s += (double)partial[((int64_t)c * rows_per_group + r) * kNumCoef + k];
                for (int d = kWave / 2; d > 0; d /= 2)
                    s += __shfl_xor(s, d);
                t += __builtin_bit_cast(float, (uint32_t)to_bf16((float)s) << 16);
            }
            if ((tid & (kWave - 1)) == 0)
                block_sum[0][tid / kWave] = (double)t;
            __syncthreads();
            if (tid == 0) {
                float v = 0.0f;
                for (int b = 0; b < T / kWave; ++b)
                    v += (float)block_sum[0][b];
                store_coef_grad(dA, k, (double)v, bf16);
            }
            return;
        }
        double s = 0.0;
#pragma unroll 8
        for (int64_t r = tid; r < (int64_t)G_shared * rows_per_group; r += T)
            s += (double)partial[r * kNumCoef + k];
        thread_sum[0][tid] = s;
        __syncthreads();
        if (tid < T / kWave) {
            double t = 0.0;
            for (int l = 0; l < kWave; ++l)
                t += thread_sum[0][tid * kWave + l];
            block_sum[0][tid] = t;
        }
        __syncthreads();
        if (tid == 0) {
            double t = 0.0;
            for (int b = 0; b < T / kWave; ++b)
                t += block_sum[0][b];
            store_coef_grad(dA, k, t, bf16);
        }
        return;
    }
    const float *base = partial + (size_t)g * rows_per_group * kNumCoef;

    double s[kNumCoef];
#pragma unroll
    for (int k = 0; k < kNumCoef; ++k)
        s[k] = 0.0;
#pragma unroll 4
    for (int r = tid; r < rows_per_group; r += T) {
#pragma unroll
        for (int k = 0; k < kNumCoef; ++k)
            s[k] += (double)base[(size_t)r * kNumCoef + k];
    }
#pragma unroll
    for (int k = 0; k < kNumCoef; ++k)
        thread_sum[k][tid] = s[k];
    __syncthreads();
    const int nblocks = T / kWave;
    if (tid < kNumCoef * nblocks) {
        const int k = tid / nblocks, b = tid - k * nblocks;
        double t = 0.0;
        for (int l = 0; l < kWave; ++l)
            t += thread_sum[k][b * kWave + l];
        block_sum[k][b] = t;
    }
    __syncthreads();
    if (tid < kNumCoef) {
        double t = 0.0;
        for (int b = 0; b < nblocks; ++b)
            t += block_sum[tid][b];
        if (tid > M)
            store_coef_grad(dB, g * N + (tid - (M + 1)), t, bf16);
        else if (G_shared == 0)
            store_coef_grad(dA, g * (M + 1) + tid, t, bf16);
    }
}

} // namespace grkan
#endif // GRKAN_STAGE2_H_
