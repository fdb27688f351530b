// Device helpers of the kernels that put tiles of bfloat16 through LDS and the matrix cores.  Device code only.
#ifndef GRKAN_TILE_H_
#define GRKAN_TILE_H_

#include <hip/hip_runtime.h>

#include <type_traits>

#include "grkan_elem.h"

namespace grkan {
namespace tile {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

typedef const __attribute__((address_space(1))) char *gcptr_t;
typedef __attribute__((address_space(1))) char *gptr_t;

__device__ __forceinline__ uint64_t uniform_u64(uint64_t v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ u32x4 gload16(uint64_t base, uint32_t off)
{
    return *(const __attribute__((address_space(1))) u32x4 *)((gcptr_t)base + off);
}
__device__ __forceinline__ void gstore16(uint64_t base, uint32_t off, u32x4 v)
{
    *(__attribute__((address_space(1))) u32x4 *)((gptr_t)base + off) = v;
}
__device__ __forceinline__ u32x4 lds_read16(uint32_t at)
{
    return *(const __attribute__((address_space(3))) u32x4 *)(uintptr_t)at;
}
__device__ __forceinline__ void lds_write16(uint32_t at, u32x4 v)
{
    *(__attribute__((address_space(3))) u32x4 *)(uintptr_t)at = v;
}
// lane (i, g) of a wavefront gets column i, rows 4 g .. 4 g + 3 of what the lanes address (8 bytes each: lane l row l / 4)
__device__ __forceinline__ s16x4 lds_read_transposed(uint32_t at)
{
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(uintptr_t)at);
}
__device__ __forceinline__ void fence_schedule() { __builtin_amdgcn_sched_barrier(0); }
__device__ __forceinline__ void keep_in_loop(uint32_t &v) { asm volatile("" : "+v"(v)); }

template <int I, int E, typename F> __device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (I < E) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, E>(f);
    }
}

__device__ __forceinline__ float low(uint32_t w) { return __builtin_bit_cast(float, w << 16); }
__device__ __forceinline__ float high(uint32_t w) { return __builtin_bit_cast(float, w & 0xffff0000u); }
__device__ __forceinline__ uint32_t pack(float a, float b)
{
    f32x2 v;
    v[0] = a;
    v[1] = b;
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// F of eight bfloat16, every step of all of them before the next (as the fused layer's prologue computes it).
__device__ __forceinline__ u32x4 rational8(const u32x4 &w, const Coef<5, 4> &c)
{
    float x[8], p[8], q[8];
#pragma unroll
    for (int e = 0; e < 8; ++e)
        x[e] = e % 2 == 0 ? low(w[e / 2]) : high(w[e / 2]);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        p[e] = fmaf(c.a[5], x[e], c.a[4]);
        q[e] = fmaf(c.b[3], x[e], c.b[2]);
    }
    fence_schedule();
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        p[e] = fmaf(p[e], x[e], c.a[3]);
        q[e] = fmaf(q[e], x[e], c.b[1]);
    }
    fence_schedule();
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        p[e] = fmaf(p[e], x[e], c.a[2]);
        q[e] = fmaf(q[e], x[e], c.b[0]);
    }
    fence_schedule();
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        p[e] = fmaf(p[e], x[e], c.a[1]);
        q[e] = fmaf(fabsf(q[e]), fabsf(x[e]), 1.0f);
    }
    fence_schedule();
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        p[e] = fmaf(p[e], x[e], c.a[0]);
        q[e] = __builtin_amdgcn_rcpf(q[e]);
    }
    fence_schedule();
    u32x4 y;
#pragma unroll
    for (int j = 0; j < 4; ++j)
        y[j] = pack(p[2 * j] * q[2 * j], p[2 * j + 1] * q[2 * j + 1]);
    return y;
}

// LDS-direct load: 16 bytes per lane from "uniform base + lane offset" to LDS bytes lds_at + 16 lane ..
// In assembly because the compiler, seeing such a load in flight, waits for all of them in front of LDS reads that have nothing to
// do with it; they are waited for by count in front of a barrier instead.  The instruction writes no registers.  s_nop: m0 and a
// base formed by a vector instruction need up to five wait states.
__device__ __forceinline__ void load_to_lds(uint64_t base, uint32_t lane_off, uint32_t lds_at)
{
    asm volatile("s_nop 4\n\tglobal_load_lds_dwordx4 %1, %2" : : "{m0}"(lds_at), "v"(lane_off), "s"(base) : "memory");
}
// All but the last N of a wavefront's loads have landed, and its LDS reads too.
template <int N> __device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory"); }

} // namespace tile
} // namespace grkan
#endif // GRKAN_TILE_H_
