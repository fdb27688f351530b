// Per-element arithmetic of the group-wise rational function (FlashKAT paper,
// Eq. "pade"), shared by the elementwise kernels and the fused GR-KAN layer
// kernel.  Device code only.
#ifndef GRKAN_ELEM_H_
#define GRKAN_ELEM_H_

#include <hip/hip_runtime.h>

namespace grkan {

// --------------------------------------------------------------------------
// coefficients of one group for numerator degree M and denominator degree N
// (scalar registers when the group is wave-uniform, vector registers in the
// flat walk).  Entries no kernel reads cost nothing: everything is unrolled.
// --------------------------------------------------------------------------
template <int M, int N> struct Coef {
    float a[M + 1];  // a_0 .. a_M
    float b[N];      // b_1 .. b_N  (b[j - 1] = b_j)
    float da[M + 1]; // i * a_i, the coefficients of P'  (da[0] unused)
    float db[N];     // j * b_j, the coefficients of Aden'
    double bd[N];    // b_j in double, for the float32-I/O kernels (see aden_of)
};

// Where the coefficient rows are.  A model that shares one numerator row between the groups has a_stride = 0;
// a bfloat16 model's coefficients are read as they are (widened exactly), so that no conversion kernels run
// in front of every call.  That is a variant of the bfloat16 kernels only (BF16): a branch on the type in front
// of the coefficient loads costs every call 0.2 - 0.3 us.
struct CoefRows {
    const void *A;    // row g at element g * a_stride
    const void *B;    // row g at element g * n
    int32_t a_stride; // m + 1, or 0: one numerator row for all groups
    int32_t bf16;     // 1: bfloat16 rows, 0: float32
};

struct CoefSums {
    const float *partial;
    int32_t rows_per_group;
    CoefRows coef;
    void *dA, *dB;
    int32_t G;
};

// UNIFORM: g is the same in all lanes, and the coefficients stay in scalar registers (there is no scalar load
// of 16 bits; a value loaded by the lanes is moved back).
template <int M, int N, bool UNIFORM, bool BF16> __device__ __forceinline__ Coef<M, N> load_coef(const CoefRows &rows, int g)
{
    auto widen = [](uint16_t v) {
        const uint32_t w = (uint32_t)v << 16;
        return __builtin_bit_cast(float, UNIFORM ? (uint32_t)__builtin_amdgcn_readfirstlane((int)w) : w);
    };
    float a[M + 1], b[N];
    if constexpr (BF16) {
        const uint16_t *pa = static_cast<const uint16_t *>(rows.A) + (size_t)g * rows.a_stride;
        const uint16_t *pb = static_cast<const uint16_t *>(rows.B) + (size_t)g * N;
#pragma unroll
        for (int i = 0; i <= M; ++i)
            a[i] = widen(pa[i]);
#pragma unroll
        for (int j = 0; j < N; ++j)
            b[j] = widen(pb[j]);
    } else {
        const float *pa = static_cast<const float *>(rows.A) + (size_t)g * rows.a_stride;
        const float *pb = static_cast<const float *>(rows.B) + (size_t)g * N;
#pragma unroll
        for (int i = 0; i <= M; ++i)
            a[i] = pa[i];
#pragma unroll
        for (int j = 0; j < N; ++j)
            b[j] = pb[j];
    }
    Coef<M, N> c;
#pragma unroll
    for (int i = 0; i <= M; ++i) {
        c.a[i] = a[i];
        c.da[i] = i >= 2 ? (float)i * a[i] : a[i];
    }
#pragma unroll
    for (int j = 0; j < N; ++j) {
        c.b[j] = b[j];
        c.db[j] = j >= 1 ? (float)(j + 1) * b[j] : b[j];
        c.bd[j] = (double)b[j];
    }
    return c;
}

// --------------------------------------------------------------------------
// per-element arithmetic (float32)
// --------------------------------------------------------------------------

// Aden = x (b_1 + b_2 x + ... + b_N x^(N-1)) by Horner.
//
// WIDE = true (float32 I/O): in double, rounded once to float32.  Q = 1 + |Aden|
// sits in every result as 1/Q or 1/Q^2, and next to a real root of the
// denominator polynomial at |x| of a few units Aden is a small difference of
// large monomials: in float32 its absolute error eps * sum |b_j||x|^j would be a
// relative error of that size in Q ~ 1 and, since those are exactly the
// elements where P/Q^2 is huge, would dominate the error of the summed
// b-gradients whatever the summation order (measured: 100x on their mean
// absolute error with N(0,1) coefficients).  Double FMA issues at the unpacked
// float32 rate on this chip, and the float32-I/O kernels are bound by HBM, so
// this is free there.
// WIDE = false (16-bit I/O): in float32.  That backward kernel is bound by
// the vector ALU (the conversions and double compares cost it 12 %), and its
// outputs are rounded to 8 or 11 significant bits anyway.
template <bool WIDE, int M, int N> __device__ __forceinline__ float aden_of(float x, const Coef<M, N> &c)
{
    if constexpr (WIDE) {
        const double xd = (double)x;
        double h = c.bd[N - 1];
#pragma unroll
        for (int j = N - 2; j >= 0; --j)
            h = fma(h, xd, c.bd[j]);
        return (float)(h * xd);
    } else {
        float h = c.b[N - 1];
#pragma unroll
        for (int j = N - 2; j >= 0; --j)
            h = fmaf(h, x, c.b[j]);
        return h * x;
    }
}

template <int M, int N> __device__ __forceinline__ float numerator_of(float x, const Coef<M, N> &c)
{
    float p = c.a[M];
#pragma unroll
    for (int i = M - 1; i >= 0; --i)
        p = fmaf(p, x, c.a[i]);
    return p;
}

// Q = 1 + |Aden| for the forward pass.  WIDE = false: Aden = x h(x) is not needed by itself there, and
// |x h| = |x| |h|, so the product and the addition are one fused multiply-add (one instruction and
// one rounding fewer).
template <bool WIDE, int M, int N> __device__ __forceinline__ float q_of(float x, const Coef<M, N> &c)
{
    if constexpr (WIDE) {
        return 1.0f + fabsf(aden_of<true>(x, c));
    } else {
        float h = c.b[N - 1];
#pragma unroll
        for (int j = N - 2; j >= 0; --j)
            h = fmaf(h, x, c.b[j]);
        return fmaf(fabsf(h), fabsf(x), 1.0f);
    }
}

// Eq. "pade": P by Horner in float32, Q as above, and one hardware
// reciprocal (1 ulp) instead of a division.
template <bool WIDE, int M, int N> __device__ __forceinline__ float fwd_elem(float x, const Coef<M, N> &c)
{
    const float p = numerator_of(x, c);
    const float q = q_of<WIDE>(x, c);
    return p * __builtin_amdgcn_rcpf(q);
}

// Eq. "grad_x", "grad_a", "grad_b" for one element; returns dx and adds this
// element's M + 1 + N terms to acc (acc[0..M] numerator, acc[M+1..M+N]
// denominator, the latter with the opposite sign until negate_b_sums is
// applied).  P/Q^2 is formed as (P r) r with r = 1/Q, so Q^2 is never computed.
// MASKED: `skip` keeps the element out of the sums (powers and weights become zeros, whatever x is).
template <bool WIDE, int M, int N, bool MASKED = false>
__device__ __forceinline__ float bwd_elem(float x, float d, const Coef<M, N> &c, float (&acc)[M + 1 + N], bool skip = false)
{
    // x^k: squares for even k, one more factor x for odd k
    constexpr int K = M > N ? M : N;
    const float xs = MASKED && skip ? 0.0f : x;
    float pw[K + 1];
    pw[0] = 1.0f;
    pw[1] = xs;
#pragma unroll
    for (int k = 2; k <= K; ++k)
        pw[k] = (k % 2 == 0) ? pw[k / 2] * pw[k / 2] : pw[k - 1] * xs;

    const float p = numerator_of(x, c);

    float dp = c.da[M];
#pragma unroll
    for (int i = M - 1; i >= 1; --i)
        dp = fmaf(dp, x, c.da[i]);

    const float aden = aden_of<WIDE>(x, c);

    float dh = c.db[N - 1];
#pragma unroll
    for (int j = N - 2; j >= 0; --j)
        dh = fmaf(dh, x, c.db[j]);

    const float q = 1.0f + fabsf(aden);
    const float r = __builtin_amdgcn_rcpf(q);

    const float t = d * r; // dy / Q
    const float ts = MASKED && skip ? 0.0f : t;
    acc[0] += ts;
#pragma unroll
    for (int i = 1; i <= M; ++i)
        acc[i] = fmaf(ts, pw[i], acc[i]);

    // s / Q with s = sign(Aden), sign(0) = 0: Aden 2^160, beyond r <= 1 for every Aden but 0 (the smallest is 2^-149), clamped
    // to [-r, r].  Two instructions instead of compare, select and copied sign: 16-bit backward passes, bound by
    // instruction issue, [25216, 3072] bfloat16 94.1 -> 91.7 us, [25216, 1536] float16 (7, 6) 63.7 -> 60.2, bits the same.
    const float sr = __builtin_amdgcn_fmed3f(__builtin_ldexpf(aden, 160), -r, r);
    // acc[M+1..] collect +dy s P x^j / Q^2; the minus sign of Eq. "grad_b" is
    // applied once per lane after the loop (negate_b_sums)
    const float wb = t * (p * sr); // (dy / Q) (P s / Q) = dy s P / Q^2
    const float ws = MASKED && skip ? 0.0f : wb;
#pragma unroll
    for (int j = 1; j <= N; ++j)
        acc[M + j] = fmaf(ws, pw[j], acc[M + j]);

    // dx = dy (P'/Q - s Aden' P/Q^2) = (dy/Q) P' - (dy s P/Q^2) Aden'
    const float dx = fmaf(t, dp, -(wb * dh));
    return dx;
}

template <int M, int N> __device__ __forceinline__ void negate_b_sums(float (&acc)[M + 1 + N])
{
#pragma unroll
    for (int k = M + 1; k < M + 1 + N; ++k)
        acc[k] = -acc[k];
}

// --------------------------------------------------------------------------
// wavefront sum with DPP: quad swaps, half-row and row mirrors, then the two
// row broadcasts; the total of all 64 lanes ends in lane 63.
// --------------------------------------------------------------------------
template <int CTRL, int ROW_MASK> __device__ __forceinline__ float dpp_get(float v)
{
    // lanes whose row is masked off receive 0
    return __builtin_bit_cast(
        float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROW_MASK, 0xf, false));
}

__device__ __forceinline__ float wave_sum(float v)
{
    v += dpp_get<0xB1, 0xf>(v);  // quad_perm [1,0,3,2]
    v += dpp_get<0x4E, 0xf>(v);  // quad_perm [2,3,0,1]
    v += dpp_get<0x141, 0xf>(v); // row_half_mirror
    v += dpp_get<0x140, 0xf>(v); // row_mirror: every lane of a row holds the row's sum
    v += dpp_get<0x142, 0xa>(v); // row_bcast:15 into rows 1 and 3
    v += dpp_get<0x143, 0xc>(v); // row_bcast:31 into rows 2 and 3
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}

} // namespace grkan
#endif // GRKAN_ELEM_H_
