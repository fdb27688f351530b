// GR-KAN group-wise rational function on gfx950 (MI355X): kernels and C ABI.
//
// The function and its gradients are those of the FlashKAT paper
// (Eq. "pade"; Eq. "grad_a", "grad_b", "grad_x", summed as in Eq. "accum" and
// "accum2").  The paper's own backward kernel (its Algorithm 2) accumulates the
// coefficient gradients per thread block and then issues one atomic add per
// block; here there are no atomics at all:
//
//   stage 1  Each lane streams 128-bit vectors of x and dy, writes dx, and
//            keeps the m + 1 + n partial sums (ten for the paper's degrees) in
//            registers for the whole kernel.
//            Group walk (long, line-aligned group segments): one wavefront =
//            one group, coefficients in scalar registers; the wavefront folds
//            its sums with DPP row/bank operations, the workgroup folds its
//            wavefronts through LDS.  Flat walk (short segments): wavefronts
//            read whole rows or column blocks of whole groups, each lane holds
//            the coefficients of its fixed column's group, and the workgroup
//            folds lanes -> runs -> groups through LDS.  Either way one row of m + 1 + n floats per (workgroup,
//            group) goes to a workspace.
//   stage 2  one wavefront per group adds that group's workspace rows in a
//            fixed order (in double) and overwrites dA / dB.
//
// Every order is fixed by the launch geometry, which is a pure function of
// shape, alignment and device, so dA / dB are bit-identical from run to run.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdlib>
#include <mutex>
#include <tuple>
#include <type_traits>
#include <vector>

#include "grkan_elem.h"
#include "grkan_plan.h"
#include "grkan_stage2.h"

namespace grkan {

// Global-memory (address space 1) byte pointers.  The loop-carried chunk base
// is wave-uniform; passing its two halves through readfirstlane keeps it in
// scalar registers, so that the memory instructions take the "scalar base +
// 32-bit lane offset" form and the vector ALU does no address arithmetic in the
// steady state.  The explicit address space keeps these global_* instructions
// (a pointer rebuilt from integers would otherwise be treated as generic).
typedef const __attribute__((address_space(1))) char *gcptr_t;
typedef __attribute__((address_space(1))) char *gptr_t;

// Marks a lane value as redefined at this point (no instruction is emitted).  Used on the 32-bit lane
// offset at the top of the streaming loops: its zero-extension then stays inside the loop body, where
// the address "scalar base + 32-bit lane offset" is recognised as such; hoisted out of the loop it would
// become a 64-bit lane value and every access would pay a 64-bit vector addition.
__device__ __forceinline__ void keep_in_loop(uint32_t &v) { asm volatile("" : "+v"(v)); }

// The instruction scheduler may not move anything across this point.  Placed after the prefetch loads:
// left alone, the scheduler sinks them into the arithmetic of the chunk before (dozens of instructions
// later), which shortens the time they have to arrive.
__device__ __forceinline__ void issue_before_what_follows() { __builtin_amdgcn_sched_barrier(0); }

__device__ __forceinline__ uint64_t uniform_u64(uint64_t v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// --------------------------------------------------------------------------
// vector memory access: VEC elements of IO per lane, one instruction
// --------------------------------------------------------------------------
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

// tags of the two 16-bit I/O formats (the arithmetic is float32 for both)
struct bf16_t {
    uint16_t bits;
};
struct f16_t {
    uint16_t bits;
};

// two 16-bit elements of one 32-bit word -> float32 (element 0 in the low half)
template <typename IO> __device__ __forceinline__ void widen_pair(uint32_t w, float &lo, float &hi)
{
    if constexpr (std::is_same_v<IO, bf16_t>) {
        // bfloat16 -> float32 is a 16-bit shift
        lo = __builtin_bit_cast(float, w << 16);
        hi = __builtin_bit_cast(float, w & 0xffff0000u);
    } else {
        const f16x2 h = __builtin_bit_cast(f16x2, w);
        lo = (float)h[0];
        hi = (float)h[1];
        // keep the two conversions as instructions of their own: folded into mixed-precision FMAs
        // (one per use of x) they cost the backward kernel registers and time
        asm volatile("" : "+v"(lo), "+v"(hi));
    }
}

// two float32 -> one word of two 16-bit elements, round to nearest even
template <typename IO> __device__ __forceinline__ uint32_t narrow_pair(float lo, float hi)
{
    f32x2 f;
    f[0] = lo;
    f[1] = hi;
    if constexpr (std::is_same_v<IO, bf16_t>)
        return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));
    else
        return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, f16x2));
}

template <typename IO> __device__ __forceinline__ float widen_one(uint16_t v)
{
    if constexpr (std::is_same_v<IO, bf16_t>)
        return __builtin_bit_cast(float, (uint32_t)v << 16);
    else
        return (float)__builtin_bit_cast(_Float16, v);
}

template <typename IO> __device__ __forceinline__ uint16_t narrow_one(float v)
{
    if constexpr (std::is_same_v<IO, bf16_t>)
        return __builtin_bit_cast(uint16_t, static_cast<__bf16>(v));
    else
        return __builtin_bit_cast(uint16_t, static_cast<_Float16>(v));
}

template <int BYTES> struct RawOf;
template <> struct RawOf<16> { using type = u32x4; };
template <> struct RawOf<8> { using type = u32x2; };
template <> struct RawOf<4> { using type = uint32_t; };
template <> struct RawOf<2> { using type = uint16_t; };

template <int BYTES> __device__ __forceinline__ uint32_t raw_word(const typename RawOf<BYTES>::type &r, int i)
{
    if constexpr (BYTES == 16 || BYTES == 8)
        return r[i];
    else
        return (uint32_t)r;
}

// A lane's vector as it sits in memory (raw bits), so that a prefetched vector
// can sit in registers untouched while the wave works on the current one:
// converting at load time would make the wave wait for the data immediately.
template <typename IO, int VEC> using RawT = typename RawOf<(int)sizeof(IO) * VEC>::type;

// LOOSE: the vector is aligned to its elements only (the overlapped walk; global memory instructions take
// any byte address on this target).
template <typename IO, int VEC, bool LOOSE = false> __device__ __forceinline__ RawT<IO, VEC> load_raw(gcptr_t p)
{
    using Raw = RawT<IO, VEC>;
    if constexpr (LOOSE) {
        typedef Raw LooseRaw __attribute__((aligned(sizeof(IO))));
        return *(const __attribute__((address_space(1))) LooseRaw *)p;
    } else {
        return __builtin_nontemporal_load((const __attribute__((address_space(1))) Raw *)p);
    }
}

// Reads a loaded vector at this point (no instruction is emitted), so that the wait for its load is
// placed here and not at its first real use further down.
template <typename IO, int VEC> __device__ __forceinline__ void arrived(const RawT<IO, VEC> &r)
{
    const uint32_t w = raw_word<(int)sizeof(IO) * VEC>(r, 0);
    asm volatile("" : : "v"(w));
}

template <typename IO, int VEC> __device__ __forceinline__ void unpack(const RawT<IO, VEC> &r, float (&out)[VEC])
{
    constexpr int BYTES = (int)sizeof(IO) * VEC;
    if constexpr (sizeof(IO) == 4) {
#pragma unroll
        for (int i = 0; i < VEC; ++i)
            out[i] = __builtin_bit_cast(float, raw_word<BYTES>(r, i));
    } else if constexpr (VEC == 1) {
        out[0] = widen_one<IO>(r);
    } else {
        // two elements per 32-bit word
#pragma unroll
        for (int i = 0; i < VEC / 2; ++i)
            widen_pair<IO>(raw_word<BYTES>(r, i), out[2 * i], out[2 * i + 1]);
    }
}

template <typename IO, int VEC, bool LOOSE = false> __device__ __forceinline__ void load_vec(gcptr_t p, float (&out)[VEC])
{
    unpack<IO, VEC>(load_raw<IO, VEC, LOOSE>(p), out);
}

template <typename IO, int VEC, bool LOOSE = false>
__device__ __forceinline__ void store_vec(gptr_t p, const float (&in)[VEC])
{
    constexpr int BYTES = (int)sizeof(IO) * VEC;
    using Raw = typename RawOf<BYTES>::type;
    Raw r;
    if constexpr (sizeof(IO) == 4) {
        if constexpr (VEC == 1) {
            r = __builtin_bit_cast(uint32_t, in[0]);
        } else {
#pragma unroll
            for (int i = 0; i < VEC; ++i)
                r[i] = __builtin_bit_cast(uint32_t, in[i]);
        }
    } else if constexpr (VEC == 1) {
        r = narrow_one<IO>(in[0]);
    } else {
#pragma unroll
        for (int i = 0; i < VEC / 2; ++i) {
            const uint32_t w = narrow_pair<IO>(in[2 * i], in[2 * i + 1]);
            if constexpr (VEC == 2)
                r = w;
            else
                r[i] = w;
        }
    }
    if constexpr (LOOSE) {
        typedef Raw LooseRaw __attribute__((aligned(sizeof(IO))));
        *(__attribute__((address_space(1))) LooseRaw *)p = r;
    } else {
        __builtin_nontemporal_store(r, (__attribute__((address_space(1))) Raw *)p);
    }
}

// --------------------------------------------------------------------------
// kernels
// --------------------------------------------------------------------------
struct FwdArgs {
    const char *x;
    char *y;
    CoefRows coef;
    int32_t dgc; // channels per coefficient group (walk.dg is the walk's: a whole row in the flat walk)
    Walk walk;
};

struct BwdArgs {
    const char *x;
    const char *dy;
    char *dx;
    CoefRows coef;
    float *partial; // [G][workspace rows per group][m + 1 + n]
    int32_t dgc;    // channels per coefficient group (walk.dg is the walk's: a whole row in the flat walk,
                    // a column block of the group when the plan splits groups)
    Walk walk;
};

// Forward.  In fixed-column mode a wave prefetches: the loads of its next chunk
// are issued before the arithmetic on the current one, so every resident wave
// always has one chunk of loads in flight.  The persistent grid is then sized
// so that the chip as a whole keeps about 4 MB of loads in flight (measured
// optimum of this memory system for a streaming read/write mix; both deeper
// per-wave prefetch and more resident waves were measured slower).
// LOOSE: the overlapped walk (a flat walk whose vectors are aligned to their elements only).  CBF: bfloat16
// coefficients.
template <typename IO, int VEC, bool FIXED, bool LANECOEF, int M, int N, bool LOOSE = false, bool CBF = false>
__global__ __launch_bounds__(kThreadsPerWg) void grkan_fwd_kernel(const FwdArgs a)
{
    static_assert(FIXED || !LANECOEF, "per-lane coefficients need fixed columns");
    static_assert(LANECOEF || !LOOSE, "the overlapped walk is a flat walk");
    const Walk &p = a.walk;
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const WaveId id = wave_id(p, (int32_t)blockIdx.x, wv);
    // group walk: the coefficient group that holds the wave's column block (scalar registers; the
    // block is the group itself unless the plan splits groups); flat walk: the group of this lane's
    // fixed column inside the wave's block of whole groups (vector registers)
    int cg;
    if constexpr (LANECOEF)
        cg = (int)(((uint32_t)id.g * (uint32_t)p.dg + fixed_col_elem(p, fixed_lane_col(p, id.w, lane).ccol, LOOSE)) /
                   (uint32_t)a.dgc);
    else
        cg = p.dg == a.dgc ? id.g : (int)((uint32_t)id.g * (uint32_t)p.dg / (uint32_t)a.dgc);
    const Coef<M, N> c = load_coef<M, N, !LANECOEF, CBF>(a.coef, cg);
    const int32_t n_it = full_visits(p, id.w);
    const bool tail = owns_tail(p, id.w) && lane < p.rem;
    constexpr int64_t ES = sizeof(IO);
    constexpr bool WIDE = sizeof(IO) == 4; // see aden_of
    const uint64_t x0 = reinterpret_cast<uint64_t>(a.x);
    const uint64_t y0 = reinterpret_cast<uint64_t>(a.y);

    auto one = [&](uint64_t off) {
        float xv[VEC], yv[VEC];
        load_vec<IO, VEC, LOOSE>((gcptr_t)(x0 + off), xv);
#pragma unroll
        for (int e = 0; e < VEC; ++e)
            yv[e] = fwd_elem<WIDE, M, N>(xv[e], c);
        store_vec<IO, VEC, LOOSE>((gptr_t)(y0 + off), yv);
    };

    if constexpr (FIXED) {
        const uint64_t base0 = (uint64_t)(fixed_base0(p, id.g, id.w) * ES);
        const uint64_t step = (uint64_t)(fixed_step(p) * ES);
        uint32_t lo = fixed_lane_offset(p, id.w, lane, LOOSE) * (uint32_t)ES;
        // chunk `i` of this wave: scalar base + lane offset
        auto xin = [&](int32_t i) { return (gcptr_t)uniform_u64(x0 + base0 + (uint64_t)(uint32_t)i * step) + lo; };
        auto yout = [&](int32_t i) { return (gptr_t)uniform_u64(y0 + base0 + (uint64_t)(uint32_t)i * step) + lo; };

        // chunk i: raw bits in, results out
        auto work = [&](const RawT<IO, VEC> &rx, int32_t i) {
            float xs[VEC], yv[VEC];
            unpack<IO, VEC>(rx, xs);
#pragma unroll
            for (int e = 0; e < VEC; ++e)
                yv[e] = fwd_elem<WIDE, M, N>(xs[e], c);
            store_vec<IO, VEC, LOOSE>(yout(i), yv);
        };
        if (n_it > 0) {
            // Two register sets take turns, so nothing is copied from "next" to "current" and the loop
            // body has no conditional load.  Per half trip: issue the loads of the following chunk
            // (raw, untouched), work on the current one, then wait for those loads before issuing any
            // more - one chunk of loads in flight per wave, which is what the persistent grid is sized for.
            RawT<IO, VEC> ra = load_raw<IO, VEC, LOOSE>(xin(0));
            arrived<IO, VEC>(ra); // the loop is entered, like re-entered, with nothing to wait for
            int32_t it = 0;
            for (; it + 2 < n_it; it += 2) {
                keep_in_loop(lo);
                const RawT<IO, VEC> rb = load_raw<IO, VEC, LOOSE>(xin(it + 1));
                issue_before_what_follows();
                work(ra, it);
                arrived<IO, VEC>(rb);
                ra = load_raw<IO, VEC, LOOSE>(xin(it + 2));
                issue_before_what_follows();
                work(rb, it + 1);
                arrived<IO, VEC>(ra);
            }
            if (it + 1 < n_it) {
                const RawT<IO, VEC> rb = load_raw<IO, VEC, LOOSE>(xin(it + 1));
                issue_before_what_follows();
                work(ra, it);
                work(rb, it + 1);
            } else {
                work(ra, it);
            }
        }
        if (tail)
            one(base0 + (uint64_t)(uint32_t)n_it * step + lo);
    } else {
        LanePos s = lane_start(p, id.w, lane);
        for (int32_t it = 0; it < n_it; ++it) {
            one((uint64_t)(elem_offset(p, id.g, s) * ES));
            lane_advance(p, s);
        }
        if (tail)
            one((uint64_t)(elem_offset(p, id.g, s) * ES));
    }
}

// Backward, stage 1 (see the file header).
template <typename IO, int VEC, bool FIXED, bool LANECOEF, int M, int N, bool LOOSE = false, bool CBF = false>
__global__ __launch_bounds__(kThreadsPerWg) void grkan_bwd_stage1_kernel(const BwdArgs a)
{
    static_assert(FIXED || !LANECOEF, "per-lane coefficients need fixed columns");
    static_assert(LANECOEF || !LOOSE, "the overlapped walk is a flat walk");
    const Walk &p = a.walk;
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const WaveId id = wave_id(p, (int32_t)blockIdx.x, wv);
    int cg;
    if constexpr (LANECOEF)
        cg = (int)(((uint32_t)id.g * (uint32_t)p.dg + fixed_col_elem(p, fixed_lane_col(p, id.w, lane).ccol, LOOSE)) /
                   (uint32_t)a.dgc);
    else
        cg = p.dg == a.dgc ? id.g : (int)((uint32_t)id.g * (uint32_t)p.dg / (uint32_t)a.dgc);
    const Coef<M, N> c = load_coef<M, N, !LANECOEF, CBF>(a.coef, cg);
    const int32_t n_it = full_visits(p, id.w);
    const bool tail = owns_tail(p, id.w) && lane < p.rem;
    constexpr int64_t ES = sizeof(IO);
    constexpr bool WIDE = sizeof(IO) == 4; // see aden_of
    const uint64_t x0 = reinterpret_cast<uint64_t>(a.x);
    const uint64_t dy0 = reinterpret_cast<uint64_t>(a.dy);
    const uint64_t dx0 = reinterpret_cast<uint64_t>(a.dx);
    // elements at the front of this lane's vectors that another lane counts (overlapped walk)
    const int skip = LOOSE ? (int)overlap_skip(p, fixed_lane_col(p, id.w, lane).ccol) : 0;

    constexpr int kNumCoef = M + 1 + N; // sums per group
    float acc[kNumCoef];
#pragma unroll
    for (int k = 0; k < kNumCoef; ++k)
        acc[k] = 0.0f;

    auto one = [&](uint64_t off) {
        float xv[VEC], dv[VEC], ov[VEC];
        load_vec<IO, VEC, LOOSE>((gcptr_t)(x0 + off), xv);
        load_vec<IO, VEC, LOOSE>((gcptr_t)(dy0 + off), dv);
#pragma unroll
        for (int e = 0; e < VEC; ++e)
            ov[e] = bwd_elem<WIDE, M, N, LOOSE>(xv[e], dv[e], c, acc, e < skip);
        store_vec<IO, VEC, LOOSE>((gptr_t)(dx0 + off), ov);
    };

    if constexpr (FIXED) {
        const uint64_t base0 = (uint64_t)(fixed_base0(p, id.g, id.w) * ES);
        const uint64_t step = (uint64_t)(fixed_step(p) * ES);
        uint32_t lo = fixed_lane_offset(p, id.w, lane, LOOSE) * (uint32_t)ES;
        // chunk `i` of this wave: scalar base + lane offset
        auto xin = [&](int32_t i) { return (gcptr_t)uniform_u64(x0 + base0 + (uint64_t)(uint32_t)i * step) + lo; };
        auto dyin = [&](int32_t i) { return (gcptr_t)uniform_u64(dy0 + base0 + (uint64_t)(uint32_t)i * step) + lo; };
        auto dxout = [&](int32_t i) { return (gptr_t)uniform_u64(dx0 + base0 + (uint64_t)(uint32_t)i * step) + lo; };

        // chunk i: raw bits in, dx out, sums updated
        auto work = [&](const RawT<IO, VEC> &rx, const RawT<IO, VEC> &rd, int32_t i) {
            float xs[VEC], ds[VEC], ov[VEC];
            unpack<IO, VEC>(rx, xs);
            unpack<IO, VEC>(rd, ds);
#pragma unroll
            for (int e = 0; e < VEC; ++e)
                ov[e] = bwd_elem<WIDE, M, N, LOOSE>(xs[e], ds[e], c, acc, e < skip);
            store_vec<IO, VEC, LOOSE>(dxout(i), ov);
        };
        if (n_it > 0) {
            // Two register sets take turns, so nothing is copied from "next" to "current" and the loop
            // body has no conditional load.  Per half trip: issue the loads of the following chunk
            // (raw, untouched), work on the current one, then wait for those loads before issuing any
            // more - one chunk of loads in flight per wave, which is what the persistent grid is sized for.
            RawT<IO, VEC> xa = load_raw<IO, VEC, LOOSE>(xin(0));
            RawT<IO, VEC> da = load_raw<IO, VEC, LOOSE>(dyin(0));
            arrived<IO, VEC>(xa); // the loop is entered, like re-entered, with nothing to wait for
            arrived<IO, VEC>(da);
            int32_t it = 0;
            for (; it + 2 < n_it; it += 2) {
                keep_in_loop(lo);
                const RawT<IO, VEC> xb = load_raw<IO, VEC, LOOSE>(xin(it + 1));
                const RawT<IO, VEC> db = load_raw<IO, VEC, LOOSE>(dyin(it + 1));
                issue_before_what_follows();
                work(xa, da, it);
                arrived<IO, VEC>(xb);
                arrived<IO, VEC>(db);
                xa = load_raw<IO, VEC, LOOSE>(xin(it + 2));
                da = load_raw<IO, VEC, LOOSE>(dyin(it + 2));
                issue_before_what_follows();
                work(xb, db, it + 1);
                arrived<IO, VEC>(xa);
                arrived<IO, VEC>(da);
            }
            if (it + 1 < n_it) {
                const RawT<IO, VEC> xb = load_raw<IO, VEC, LOOSE>(xin(it + 1));
                const RawT<IO, VEC> db = load_raw<IO, VEC, LOOSE>(dyin(it + 1));
                issue_before_what_follows();
                work(xa, da, it);
                work(xb, db, it + 1);
            } else {
                work(xa, da, it);
            }
        }
        if (tail)
            one(base0 + (uint64_t)(uint32_t)n_it * step + lo);
    } else {
        LanePos s = lane_start(p, id.w, lane);
        for (int32_t it = 0; it < n_it; ++it) {
            one((uint64_t)(elem_offset(p, id.g, s) * ES));
            lane_advance(p, s);
        }
        if (tail)
            one((uint64_t)(elem_offset(p, id.g, s) * ES));
    }

    negate_b_sums<M, N>(acc);
    if constexpr (!LANECOEF) {
        // registers -> wavefront (DPP) -> workgroup (LDS) -> one workspace row per group
        __shared__ float wave_part[kWavesPerWg][kNumCoef];
#pragma unroll
        for (int k = 0; k < kNumCoef; ++k) {
            const float s = wave_sum(acc[k]);
            if (lane == 0)
                wave_part[wv][k] = s;
        }
        __syncthreads();
        const int tid = threadIdx.x;
        if (tid < p.k * kNumCoef) {
            const int gl = tid / kNumCoef;
            const int kc = tid - gl * kNumCoef;
            // waves gl, gl + k, gl + 2k, ... of this workgroup hold group (bundle * k + gl)
            float s = 0.0f;
            for (int sub = 0; sub < p.ns; ++sub)
                s += wave_part[sub * p.k + gl][kc];
            const int32_t bundle = (int32_t)blockIdx.x % p.nb;
            const int32_t wgi = (int32_t)blockIdx.x / p.nb;
            const int64_t g = (int64_t)bundle * p.k + gl;
            a.partial[(g * p.wg_per_bundle + wgi) * kNumCoef + kc] = s;
        }
    } else {
        // Flat walk: the 256 lanes of the workgroup hold consecutive vectors of
        // the rows of its column block, so lanes of one coefficient group form
        // runs of vt = d_g / vec lanes (a group can own several runs when the
        // block's row is shorter than the workgroup).  registers -> LDS -> one sum
        // per run (fixed lane order) -> one sum per group (fixed run order) -> one
        // workspace row per workgroup for every group of the block, zeros
        // included, so that stage 2 needs no map of who wrote what.
        __shared__ float lane_part[kNumCoef][kThreadsPerWg];
        __shared__ float run_part[kThreadsPerWg + 1][kNumCoef];
        const int tid = threadIdx.x;
#pragma unroll
        for (int k = 0; k < kNumCoef; ++k)
            lane_part[k][tid] = acc[k];
        __syncthreads();
        const uint32_t vt = LOOSE ? (uint32_t)p.gvecs : (uint32_t)a.dgc / (uint32_t)p.vec; // lanes per run
        const uint32_t V = (uint32_t)p.v;                       // vectors per row of the walk's column block
        const uint32_t Gb = (uint32_t)p.dg / (uint32_t)a.dgc;   // coefficient groups per column block
        const uint32_t c0 = ((uint32_t)id.wg_index * kThreadsPerWg) % V; // column of lane 0
        const uint32_t u0 = c0 / vt;                            // first (unwrapped) run
        const uint32_t n_runs = (c0 + kThreadsPerWg - 1) / vt - u0 + 1;
        for (uint32_t item = tid; item < n_runs * kNumCoef; item += kThreadsPerWg) {
            const uint32_t r = item / kNumCoef, k = item - r * kNumCoef;
            const uint32_t first = (u0 + r) * vt; // unwrapped column where run r starts
            const uint32_t lo = first > c0 ? first - c0 : 0;
            const uint32_t hi = first + vt - c0 < (uint32_t)kThreadsPerWg ? first + vt - c0 : (uint32_t)kThreadsPerWg;
            float s = 0.0f;
            for (uint32_t l = lo; l < hi; ++l)
                s += lane_part[k][l];
            run_part[r][k] = s;
        }
        __syncthreads();
        for (uint32_t item = tid; item < Gb * kNumCoef; item += kThreadsPerWg) {
            const uint32_t g = item / kNumCoef, k = item - g * kNumCoef;
            // run r belongs to group (u0 + r) mod Gb of this block
            float s = 0.0f;
            for (uint32_t r = (g + Gb - u0 % Gb) % Gb; r < n_runs; r += Gb)
                s += run_part[r][k];
            const int64_t gg = (int64_t)id.g * Gb + g; // the group's index in A, B and the workspace
            a.partial[(gg * p.wg_per_bundle + id.wg_index) * kNumCoef + k] = s;
        }
    }
}

static int stage2_threads(int32_t rows_per_group) { return rows_per_group > kWave ? kStage2MaxThreads : kWave; }

template <int M, int N>
__global__ __launch_bounds__(kStage2MaxThreads) void grkan_bwd_stage2_kernel(const float *__restrict__ partial,
                                                                             int32_t rows_per_group,
                                                                             void *__restrict__ dA,
                                                                             void *__restrict__ dB,
                                                                             int32_t G_shared, int32_t bf16)
{
    stage2_block<M, N>(partial, rows_per_group, dA, dB, G_shared, bf16, (int)blockIdx.x);
}

// --------------------------------------------------------------------------
// host side
// --------------------------------------------------------------------------
struct DeviceInfo {
    bool ready = false;
    int num_cu = 0;
};

static std::mutex g_mu;
static DeviceInfo g_dev[64];

static bool device_info(int *dev_out, DeviceInfo *out)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64)
        return false;
    std::lock_guard<std::mutex> lock(g_mu);
    if (!g_dev[dev].ready) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
            return false;
        g_dev[dev].num_cu = n;
        g_dev[dev].ready = true;
    }
    *dev_out = dev;
    *out = g_dev[dev];
    return true;
}

// Experiment overrides of the persistent grid sizes (workgroups per compute
// unit; 0 = the built-in choice).  The two environment variables are read once,
// when the library is loaded; grkan_tuning_override replaces them at run time.
static int env_int(const char *name)
{
    const char *s = std::getenv(name);
    if (!s || !*s)
        return 0;
    const int v = std::atoi(s);
    return v > 0 ? v : 0;
}

static std::atomic<int> g_fwd_wg_per_cu{env_int("GRKAN_FWD_WG_PER_CU")};
static std::atomic<int> g_bwd_wg_per_cu{env_int("GRKAN_BWD_WG_PER_CU")};

static int32_t common_alignment(std::initializer_list<const void *> ptrs)
{
    uintptr_t bits = 16;
    for (const void *q : ptrs)
        bits |= reinterpret_cast<uintptr_t>(q);
    return (int32_t)(bits & (~bits + 1)); // lowest set bit, at most 16
}

// Kernel selection: the variant for (degrees, dtype, vector width, walk mode)
// as a plain function pointer, so that one code path can both query its
// occupancy and launch it.
using FwdKernel = void (*)(const FwdArgs);
using BwdKernel = void (*)(const BwdArgs);
using Stage2Kernel = void (*)(const float *, int32_t, void *, void *, int32_t, int32_t);

template <typename IO, int VEC, int M, int N, bool CBF> static FwdKernel fwd_variant(bool fixed, bool lane_coef)
{
    if (lane_coef)
        return grkan_fwd_kernel<IO, VEC, true, true, M, N, false, CBF>;
    return fixed ? grkan_fwd_kernel<IO, VEC, true, false, M, N, false, CBF>
                 : grkan_fwd_kernel<IO, VEC, false, false, M, N, false, CBF>;
}
template <typename IO, int VEC, int M, int N, bool CBF> static BwdKernel bwd_variant(bool fixed, bool lane_coef)
{
    if (lane_coef)
        return grkan_bwd_stage1_kernel<IO, VEC, true, true, M, N, false, CBF>;
    return fixed ? grkan_bwd_stage1_kernel<IO, VEC, true, false, M, N, false, CBF>
                 : grkan_bwd_stage1_kernel<IO, VEC, false, false, M, N, false, CBF>;
}

// What a launch needs of the kernel besides the degrees.
struct Pick {
    grkan_dtype_t io;
    int vec;
    bool fixed, lane_coef, overlapped, coef_bf16;
};

template <typename IO, int M, int N, bool CBF = false> static FwdKernel fwd_of_type(const Pick &k)
{
    constexpr int kFull = 16 / (int)sizeof(IO);
    if (k.overlapped) // full vectors only
        return grkan_fwd_kernel<IO, kFull, true, true, M, N, true, CBF>;
    if constexpr (kFull == 8)
        if (k.vec == 8)
            return fwd_variant<IO, 8, M, N, CBF>(k.fixed, k.lane_coef);
    switch (k.vec) {
    case 4: return fwd_variant<IO, 4, M, N, CBF>(k.fixed, k.lane_coef);
    case 2: return fwd_variant<IO, 2, M, N, CBF>(k.fixed, k.lane_coef);
    case 1: return fwd_variant<IO, 1, M, N, CBF>(k.fixed, k.lane_coef);
    }
    return nullptr;
}

template <typename IO, int M, int N, bool CBF = false> static BwdKernel bwd_of_type(const Pick &k)
{
    constexpr int kFull = 16 / (int)sizeof(IO);
    if (k.overlapped)
        return grkan_bwd_stage1_kernel<IO, kFull, true, true, M, N, true, CBF>;
    if constexpr (kFull == 8)
        if (k.vec == 8)
            return bwd_variant<IO, 8, M, N, CBF>(k.fixed, k.lane_coef);
    switch (k.vec) {
    case 4: return bwd_variant<IO, 4, M, N, CBF>(k.fixed, k.lane_coef);
    case 2: return bwd_variant<IO, 2, M, N, CBF>(k.fixed, k.lane_coef);
    case 1: return bwd_variant<IO, 1, M, N, CBF>(k.fixed, k.lane_coef);
    }
    return nullptr;
}

template <int M, int N> static FwdKernel select_fwd(const Pick &k)
{
    switch (k.io) {
    case GRKAN_F32: return fwd_of_type<float, M, N>(k);
    case GRKAN_BF16: return k.coef_bf16 ? fwd_of_type<bf16_t, M, N, true>(k) : fwd_of_type<bf16_t, M, N>(k);
    case GRKAN_F16: return fwd_of_type<f16_t, M, N>(k);
    }
    return nullptr;
}

template <int M, int N> static BwdKernel select_bwd(const Pick &k)
{
    switch (k.io) {
    case GRKAN_F32: return bwd_of_type<float, M, N>(k);
    case GRKAN_BF16: return k.coef_bf16 ? bwd_of_type<bf16_t, M, N, true>(k) : bwd_of_type<bf16_t, M, N>(k);
    case GRKAN_F16: return bwd_of_type<f16_t, M, N>(k);
    }
    return nullptr;
}

// The degrees the library is built for.  (5, 4) is the paper's; (3, 2) and
// (7, 6) are the neighbouring "numerator one degree above the denominator"
// units of the same family.
struct DegreeOps {
    int m, n;
    FwdKernel (*fwd)(const Pick &);
    BwdKernel (*bwd)(const Pick &);
    Stage2Kernel stage2;
};

template <int M, int N> static constexpr DegreeOps degree_entry()
{
    static_assert(M + 1 + N <= kMaxCoef, "workspace rows are sized for kMaxCoef sums");
    return DegreeOps{M, N, select_fwd<M, N>, select_bwd<M, N>, grkan_bwd_stage2_kernel<M, N>};
}

static const DegreeOps kDegrees[] = {degree_entry<5, 4>(), degree_entry<3, 2>(), degree_entry<7, 6>()};

static const DegreeOps *degree_ops(int m, int n)
{
    for (const DegreeOps &d : kDegrees)
        if (d.m == m && d.n == n)
            return &d;
    return nullptr;
}

// Workgroups of a kernel that fit on one compute unit at once (cached per
// kernel and device).  A persistent grid larger than that would leave
// workgroups queued behind the resident ones.
static int resident_wg_per_cu(const void *kernel, int dev)
{
    static std::mutex mu;
    static std::vector<std::tuple<const void *, int, int>> cache;
    std::lock_guard<std::mutex> lock(mu);
    for (const auto &e : cache)
        if (std::get<0>(e) == kernel && std::get<1>(e) == dev)
            return std::get<2>(e);
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, kThreadsPerWg, 0) != hipSuccess || n <= 0)
        return 0;
    cache.emplace_back(kernel, dev, n);
    return n;
}

// Workgroups (of 4 waves) per compute unit the persistent grids are sized for.
// With one chunk of loads in flight per wave (1 KB forward, 2 KB backward),
// 4 and 2 workgroups per unit put about 4 MB of loads in flight on 256 units,
// which is where the HBM-bound kernels were measured fastest (a backward pass
// that sweeps whole rows as one stream - no column blocks - measured best at 3).  The 16-bit backward pass moves
// half the bytes for the same arithmetic: with degrees (3, 2) it is bound by HBM like the others and takes 2; with (5, 4)
// and (7, 6) by the vector ALU, and takes every wave slot it can get (requests are clamped to the kernel's real
// occupancy) - but in the flat walk, where each workgroup more is one more workspace row for each of its groups,
// no more than leave every wave about four chunks.  Measured in us with 2 / 3 / 4 / as many as fit:
//   bf16 (3,2) [25216, 3072] 78.6 / 81.8 / 84.0 / 85.6     bf16 (5,4) [25216, 3072] 96.7 / 93.6 / 94.5 / 93.3
//   flat walk, bf16 (5,4): [25216, 192] 15.1 / 15.6 / 15.7 / 17.6   [25216, 384] 19.2 / 18.9 / 18.7 / 22.1
//   [25216, 3072] in 64 groups - / - / 101 / 99
// The overrides above apply to every walk.
struct Want {
    int group_walk;
    int flat_blocks; // flat walk over column blocks
    int flat_rows;   // one sweep over whole rows
};

static Want fwd_want(grkan_dtype_t)
{
    const int e = g_fwd_wg_per_cu.load(std::memory_order_relaxed);
    return e ? Want{e, e, e} : Want{4, 4, 4};
}

static Want bwd_want(grkan_dtype_t io, int m, int64_t rows, int32_t D, int num_cu)
{
    const int e = g_bwd_wg_per_cu.load(std::memory_order_relaxed);
    if (e)
        return Want{e, e, e};
    if (io == GRKAN_F32 || m <= 3)
        return Want{2, 2, 3};
    const int64_t vectors = rows * (int64_t)D / (16 / elem_size(io));
    const int64_t fit = vectors / kThreadsPerWg * 2 / (9 * (int64_t)num_cu); // 4.5 chunks for every wave
    const int flat = fit < 3 ? 3 : fit > 8 ? 8 : (int)fit;
    return Want{8, flat, flat};
}

// Plans the launch with the wanted workgroups per unit, then clamps to what
// the selected kernel can keep resident and re-plans if needed.  may_overlap: no output shares memory with an
// input, so that an element may be computed by two lanes.
template <typename Select>
static grkan_status_t plan_resident(int64_t rows, int32_t D, int32_t G, grkan_dtype_t io, int32_t align,
                                    const DeviceInfo &info, int dev, Want want, bool forward, Select select,
                                    bool may_overlap, bool coef_bf16, grkan_plan_t *pl, Walk *walk, const void **kernel)
{
    int per_cu = want.group_walk;
    if (may_overlap && make_overlapped(rows, D, G, io, info.num_cu, want.flat_rows, forward, pl, walk)) {
        *kernel = reinterpret_cast<const void *>(select(Pick{io, pl->vec, true, true, true, coef_bf16}));
        const int fit = resident_wg_per_cu(*kernel, dev);
        if (fit <= 0)
            return GRKAN_ERR_LAUNCH;
        if (fit >= want.flat_rows || make_overlapped(rows, D, G, io, info.num_cu, fit, forward, pl, walk))
            return GRKAN_OK;
    }
    grkan_status_t st = make_plan(rows, D, G, io, align, info.num_cu, per_cu, forward, pl, walk);
    if (st != GRKAN_OK)
        return st;
    // one sweep over whole rows (flat walk without column blocks, or a single unsplit group) against
    // several interleaved column streams: the two were measured best at different grid sizes
    const bool rows_walk = (pl->lane_coef ? pl->column_split : G * pl->column_split) == 1;
    const int other = rows_walk ? want.flat_rows : pl->lane_coef ? want.flat_blocks : per_cu;
    if (other != per_cu) {
        grkan_plan_t alt;
        if (make_plan(rows, D, G, io, align, info.num_cu, other, forward, &alt, nullptr) == GRKAN_OK &&
            alt.lane_coef == pl->lane_coef) {
            per_cu = other;
            st = make_plan(rows, D, G, io, align, info.num_cu, per_cu, forward, pl, walk);
            if (st != GRKAN_OK)
                return st;
        }
    }
    *kernel = reinterpret_cast<const void *>(
        select(Pick{io, pl->vec, pl->fixed_col != 0, pl->lane_coef != 0, false, coef_bf16}));
    if (!*kernel)
        return GRKAN_ERR_LAUNCH;
    const int fit = resident_wg_per_cu(*kernel, dev);
    if (fit <= 0)
        return GRKAN_ERR_LAUNCH;
    if (fit < per_cu) {
        const int32_t was_flat = pl->lane_coef;
        st = make_plan(rows, D, G, io, align, info.num_cu, fit, forward, pl, walk);
        if (st != GRKAN_OK)
            return st;
        *kernel = reinterpret_cast<const void *>(
            select(Pick{io, pl->vec, pl->fixed_col != 0, pl->lane_coef != 0, false, coef_bf16}));
        if (!*kernel || (pl->lane_coef != was_flat && resident_wg_per_cu(*kernel, dev) <= 0))
            return GRKAN_ERR_LAUNCH;
    }
    return GRKAN_OK;
}

static grkan_status_t check_common(int64_t rows, int32_t D, int32_t G, int32_t m, int32_t n, grkan_dtype_t io,
                                   const DegreeOps **ops)
{
    *ops = degree_ops(m, n);
    if (!*ops)
        return GRKAN_ERR_DEGREE;
    return check_shape(rows, D, G, io);
}

// rows of `coefs` floats, one per (group, workgroup that holds a part of it)
static size_t workspace_for(const grkan_plan_t &pl, int32_t G, int coefs)
{
    return (size_t)G * (size_t)pl.partials_per_group * (size_t)coefs * sizeof(float);
}

} // namespace grkan

using namespace grkan;

extern "C" size_t grkan_bwd_workspace_bytes(int64_t rows, int32_t D, int32_t G, grkan_dtype_t io)
{
    if (check_shape(rows, D, G, io) != GRKAN_OK)
        return 0;
    int dev;
    DeviceInfo info;
    if (!device_info(&dev, &info))
        return 0;
    size_t need = 16; // never zero, so that callers can always allocate it
    // the query names no degrees: the bound covers every built (m, n), whose kernels differ in occupancy
    for (const DegreeOps &ops : kDegrees) {
        const Want want = bwd_want(io, ops.m, rows, D, info.num_cu);
        for (int align = elem_size(io); align <= 16; align *= 2) {
            grkan_plan_t pl;
            const void *kernel = nullptr;
            for (int v = 0; v < (io == GRKAN_BF16 ? 4 : 2); ++v) {
                const int overlap = v & 1, coef_bf16 = v >> 1;
                if (plan_resident(rows, D, G, io, align, info, dev, want, false, ops.bwd, overlap != 0, coef_bf16 != 0,
                                  &pl, nullptr, &kernel) != GRKAN_OK)
                    return 0;
                const size_t b = workspace_for(pl, G, ops.m + 1 + ops.n);
                need = b > need ? b : need;
            }
        }
    }
    return need;
}

extern "C" void grkan_tuning_override(int32_t fwd_wg_per_cu, int32_t bwd_wg_per_cu)
{
    g_fwd_wg_per_cu.store(fwd_wg_per_cu > 0 ? fwd_wg_per_cu : 0, std::memory_order_relaxed);
    g_bwd_wg_per_cu.store(bwd_wg_per_cu > 0 ? bwd_wg_per_cu : 0, std::memory_order_relaxed);
}

extern "C" grkan_status_t grkan_device_query(int32_t *out)
{
    if (!out)
        return GRKAN_ERR_NULL;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess)
        return GRKAN_ERR_LAUNCH;
    const hipDeviceAttribute_t what[4] = {hipDeviceAttributeMultiprocessorCount, hipDeviceAttributeClockRate,
                                          hipDeviceAttributeMemoryClockRate, hipDeviceAttributeMemoryBusWidth};
    for (int i = 0; i < 4; ++i) {
        int v = 0;
        if (hipDeviceGetAttribute(&v, what[i], dev) != hipSuccess)
            return GRKAN_ERR_LAUNCH;
        out[i] = v;
    }
    return GRKAN_OK;
}

namespace grkan {

// The coefficient operands of a call: float32 or bfloat16, the numerator one row per group or one for all.
static CoefRows coef_rows(const void *A, const void *B, int32_t m, bool shared, grkan_dtype_t dtype)
{
    return CoefRows{A, B, shared ? 0 : m + 1, dtype == GRKAN_BF16};
}

static bool disjoint(const void *p, const void *q, size_t bytes)
{
    const uintptr_t a = reinterpret_cast<uintptr_t>(p), b = reinterpret_cast<uintptr_t>(q);
    return a + bytes <= b || b + bytes <= a;
}

static grkan_status_t fwd_impl(const void *x, const CoefRows &coef, void *y, int64_t rows, int32_t D, int32_t G, int32_t m,
                               int32_t n, grkan_dtype_t io, void *hip_stream)
{
    const DegreeOps *ops = nullptr;
    grkan_status_t st = check_common(rows, D, G, m, n, io, &ops);
    if (st != GRKAN_OK)
        return st;
    if (!coef.A || !coef.B || (rows > 0 && (!x || !y)))
        return GRKAN_ERR_NULL;
    const int es = elem_size(io);
    if ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(y)) % es != 0 ||
        (reinterpret_cast<uintptr_t>(coef.A) | reinterpret_cast<uintptr_t>(coef.B)) % (coef.bf16 ? 2 : 4) != 0)
        return GRKAN_ERR_ALIGN;
    if (rows == 0)
        return GRKAN_OK;

    int dev;
    DeviceInfo info;
    if (!device_info(&dev, &info))
        return GRKAN_ERR_LAUNCH;
    grkan_plan_t pl;
    FwdArgs a;
    const void *kernel = nullptr;
    const size_t bytes = (size_t)rows * (size_t)D * (size_t)es;
    st = plan_resident(rows, D, G, io, common_alignment({x, y}), info, dev, fwd_want(io), true, ops->fwd,
                       disjoint(x, y, bytes), coef.bf16 != 0, &pl, &a.walk, &kernel);
    if (st != GRKAN_OK)
        return st;
    a.x = static_cast<const char *>(x);
    a.y = static_cast<char *>(y);
    a.coef = coef;
    a.dgc = D / G;
    void *args[] = {&a};
    const hipError_t e = hipLaunchKernel(kernel, dim3(pl.grid), dim3(kThreadsPerWg), args, 0,
                                         static_cast<hipStream_t>(hip_stream));
    return e == hipSuccess ? GRKAN_OK : GRKAN_ERR_LAUNCH;
}

} // namespace grkan

extern "C" grkan_status_t grkan_fwd(const void *x, const float *A, const float *B, void *y,
                                    int64_t rows, int32_t D, int32_t G, int32_t m, int32_t n,
                                    grkan_dtype_t io, void *hip_stream)
{
    return fwd_impl(x, coef_rows(A, B, m, false, GRKAN_F32), y, rows, D, G, m, n, io, hip_stream);
}

extern "C" grkan_status_t grkan_fwd_model(const void *x, const void *A, const void *B, void *y,
                                          int64_t rows, int32_t D, int32_t G, int32_t m, int32_t n,
                                          grkan_dtype_t io, grkan_dtype_t coef_dtype, int32_t shared_numerator,
                                          void *hip_stream)
{
    if (coef_dtype != GRKAN_F32 && !(coef_dtype == GRKAN_BF16 && io == GRKAN_BF16))
        return GRKAN_ERR_DTYPE;
    return fwd_impl(x, coef_rows(A, B, m, shared_numerator != 0, coef_dtype), y, rows, D, G, m, n, io, hip_stream);
}

namespace grkan {

// Scratch of the allocation-free entry point: the workspace rows of stage 1,
// in a fixed array in device memory (one copy per GPU the library runs on, held
// until the process ends).  In host code the array's name is only a handle for
// the symbol; its address on a device comes from hipGetSymbolAddress, once per
// device, and only that pointer is ever handed to a kernel.
constexpr size_t kScratchBytes = (size_t)4 << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

static std::mutex g_scratch_mu;
static void *g_scratch_ptr[64]; // per device, filled on the first call there

// `dev` must be the current device.
static grkan_status_t scratch_of_device(int dev, void **out)
{
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr)
            return GRKAN_ERR_LAUNCH;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return GRKAN_OK;
}

// The three backward entry points.  Where the workspace comes from: a buffer of the caller's, the library's
// fixed array, or the caller's allocation function, asked once the launch is planned.
struct Workspace {
    void *ptr;
    size_t bytes;
    bool own_scratch;
    grkan_alloc_t alloc;
    void *alloc_context;
};

grkan_status_t run_stage2(const float *partial, int32_t rows_per_group, const CoefRows &coef, void *dA, void *dB, int32_t G,
                          int32_t m, int32_t n, hipStream_t stream)
{
    const DegreeOps *const ops = degree_ops(m, n);
    if (!ops)
        return GRKAN_ERR_DEGREE;
    int32_t G_shared = coef.a_stride == 0 ? G : 0;
    int32_t bf16 = coef.bf16;
    void *args[] = {&partial, &rows_per_group, &dA, &dB, &G_shared, &bf16};
    const int threads = G_shared > 0 ? kStage2MaxThreads : stage2_threads(rows_per_group);
    const hipError_t e = hipLaunchKernel(reinterpret_cast<const void *>(ops->stage2),
                                         dim3((unsigned)G + (G_shared > 0 ? (unsigned)(m + 1) : 0u)), dim3(threads), args, 0,
                                         stream);
    return e == hipSuccess ? GRKAN_OK : GRKAN_ERR_LAUNCH;
}

static grkan_status_t bwd_impl(const void *x, const void *dy, const CoefRows &coef, void *dx, void *dA, void *dB,
                               const Workspace &ws, int64_t rows, int32_t D, int32_t G, int32_t m, int32_t n,
                               grkan_dtype_t io, void *hip_stream, CoefSums *later = nullptr)
{
    const DegreeOps *ops = nullptr;
    grkan_status_t st = check_common(rows, D, G, m, n, io, &ops);
    if (st != GRKAN_OK)
        return st;
    if (!coef.A || !coef.B || !dA || !dB || (rows > 0 && (!x || !dy || !dx)))
        return GRKAN_ERR_NULL;
    const int es = elem_size(io);
    if ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(dy) | reinterpret_cast<uintptr_t>(dx)) % es != 0 ||
        (reinterpret_cast<uintptr_t>(coef.A) | reinterpret_cast<uintptr_t>(coef.B) | reinterpret_cast<uintptr_t>(dA) |
         reinterpret_cast<uintptr_t>(dB)) % (coef.bf16 ? 2 : 4) != 0)
        return GRKAN_ERR_ALIGN;

    int dev;
    DeviceInfo info;
    if (!device_info(&dev, &info))
        return GRKAN_ERR_LAUNCH;
    grkan_plan_t pl;
    BwdArgs a;
    const void *kernel = nullptr;
    const size_t bytes = (size_t)rows * (size_t)D * (size_t)es;
    bool may_overlap = disjoint(x, dx, bytes) && disjoint(dy, dx, bytes);
    const Want want = bwd_want(io, m, rows, D, info.num_cu);
    st = plan_resident(rows, D, G, io, common_alignment({x, dy, dx}), info, dev, want, false, ops->bwd, may_overlap,
                       coef.bf16 != 0, &pl, &a.walk, &kernel);
    if (st != GRKAN_OK)
        return st;
    size_t need = workspace_for(pl, G, m + 1 + n);
    // a workspace that is too small for the overlapped walk may do for the other
    const size_t limit = ws.own_scratch ? kScratchBytes : ws.alloc ? SIZE_MAX : ws.bytes;
    if (a.walk.gvecs > 0 && need > limit) {
        st = plan_resident(rows, D, G, io, common_alignment({x, dy, dx}), info, dev, want, false, ops->bwd, false,
                           coef.bf16 != 0, &pl, &a.walk, &kernel);
        if (st != GRKAN_OK)
            return st;
        need = workspace_for(pl, G, m + 1 + n);
    }
    void *workspace = ws.ptr;
    if (ws.own_scratch) {
        if (need > kScratchBytes)
            return GRKAN_ERR_SCRATCH_LIMIT;
        st = scratch_of_device(dev, &workspace);
        if (st != GRKAN_OK)
            return st;
    } else if (ws.alloc) {
        workspace = need > 0 ? ws.alloc(need, ws.alloc_context) : nullptr;
        if (need > 0 && (!workspace || reinterpret_cast<uintptr_t>(workspace) % 16 != 0))
            return GRKAN_ERR_WORKSPACE;
    } else if (need > 0 &&
               (!workspace || ws.bytes < need || reinterpret_cast<uintptr_t>(workspace) % 16 != 0)) {
        return GRKAN_ERR_WORKSPACE;
    }

    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    a.x = static_cast<const char *>(x);
    a.dy = static_cast<const char *>(dy);
    a.dx = static_cast<char *>(dx);
    a.coef = coef;
    a.partial = static_cast<float *>(workspace);
    a.dgc = D / G;
    if (pl.grid > 0) {
        void *args[] = {&a};
        if (hipLaunchKernel(kernel, dim3(pl.grid), dim3(kThreadsPerWg), args, 0, stream) != hipSuccess)
            return GRKAN_ERR_LAUNCH;
    }
    // Stage 1 writes every workspace row stage 2 reads (one per workgroup and group, zeros included),
    // so nothing has to be cleared beforehand; with no rows there are no workspace rows and stage 2
    // writes zeros.
    if (later) {
        *later = CoefSums{a.partial, pl.partials_per_group, coef, dA, dB, G};
        return GRKAN_OK;
    }
    return run_stage2(a.partial, pl.partials_per_group, coef, dA, dB, G, m, n, stream);
}

grkan_status_t bwd_model_stage1(const void *x, const void *dy, const CoefRows &coef, void *dx, void *dA, void *dB, grkan_alloc_t alloc,
                                void *alloc_context, int64_t rows, int32_t D, int32_t G, CoefSums *later, hipStream_t stream)
{
    return bwd_impl(x, dy, coef, dx, dA, dB, Workspace{nullptr, 0, false, alloc, alloc_context}, rows, D, G, 5, 4, GRKAN_BF16, stream, later);
}

} // namespace grkan

extern "C" grkan_status_t grkan_bwd(const void *x, const void *dy, const float *A, const float *B,
                                    void *dx, float *dA, float *dB,
                                    void *workspace, size_t workspace_bytes,
                                    int64_t rows, int32_t D, int32_t G, int32_t m, int32_t n,
                                    grkan_dtype_t io, void *hip_stream)
{
    return bwd_impl(x, dy, coef_rows(A, B, m, false, GRKAN_F32), dx, dA, dB,
                    Workspace{workspace, workspace_bytes, false, nullptr, nullptr}, rows, D, G, m, n, io, hip_stream);
}

extern "C" grkan_status_t grkan_bwd_noalloc(const void *x, const void *dy, const float *A, const float *B,
                                            void *dx, float *dA, float *dB,
                                            int64_t rows, int32_t D, int32_t G, int32_t m, int32_t n,
                                            grkan_dtype_t io, void *hip_stream)
{
    return bwd_impl(x, dy, coef_rows(A, B, m, false, GRKAN_F32), dx, dA, dB, Workspace{nullptr, 0, true, nullptr, nullptr},
                    rows, D, G, m, n, io, hip_stream);
}

extern "C" grkan_status_t grkan_bwd_model(const void *x, const void *dy, const void *A, const void *B,
                                          void *dx, void *dA, void *dB, grkan_alloc_t alloc, void *alloc_context,
                                          int64_t rows, int32_t D, int32_t G, int32_t m, int32_t n,
                                          grkan_dtype_t io, grkan_dtype_t coef_dtype, int32_t shared_numerator,
                                          void *hip_stream)
{
    if (coef_dtype != GRKAN_F32 && !(coef_dtype == GRKAN_BF16 && io == GRKAN_BF16))
        return GRKAN_ERR_DTYPE;
    if (!alloc)
        return GRKAN_ERR_NULL;
    return bwd_impl(x, dy, coef_rows(A, B, m, shared_numerator != 0, coef_dtype), dx, dA, dB,
                    Workspace{nullptr, 0, false, alloc, alloc_context}, rows, D, G, m, n, io, hip_stream);
}
