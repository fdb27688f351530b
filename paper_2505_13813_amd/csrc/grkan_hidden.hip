// The hidden activation of a KAT MLP block in training, on gfx950 (MI355X): the product that makes or receives it and the
// second layer's rational function on it, in one kernel each way (FlashKAT paper, Eq. "GR_KAN", "pade", "grad_x",
// "grad_a", "grad_b").
//
//   forward    h = X W^T + bias  (bfloat16, kept for the backward pass),  f = F(h)
//   backward   dF = dY W  (bfloat16, never written),  dh = dF F'(h),  dA, dB
//
// Both products contract over the block's width K (192 .. 768) into the wide hidden dimension N = 4 K: 25,216 tokens of
// 384 -> 1536 are 30 GFLOP, 20 us at the matrix cores' rate, around 77 MB of result, that a product by itself leaves to be read
// again.
//
// A wavefront keeps the weights of its CW hidden channels (all of one coefficient group) for the whole kernel: in vector
// registers, and what does not fit there (K = 384 two steps of 32, 512 two, 640 four, 768 six) in LDS that it alone reads, again
// for every 16 tokens.  Tokens pass by in tiles of TR (32; 16 at K = 768), shared by the workgroup's NW wavefronts (eight; twelve
// at K = 192 and 384) through two LDS buffers, one barrier per tile.  The accumulators of 16 tokens are all
// that is live of the result; which hidden channel a matrix row stands for is chosen so that a lane ends up with
// 16 bytes of consecutive channels, and the rational function, the loads of h and the stores work on the
// accumulators' layout as it is.  Coefficients are wave-uniform (scalar registers) and the coefficient sums stay in
// registers to the end: one workspace row per wavefront and part of the tokens, added by the same second stage as the elementwise backward pass.
#include <hip/hip_runtime.h>

#include <mutex>

#include "grkan_plan.h"
#include "grkan_tile.h"

namespace grkan {
namespace hidden {

using namespace tile;

constexpr int kM = 5, kN = 4, kSums = kM + 1 + kN;

struct Args {
    const char *x;      // bfloat16 [rows, K]: the product's left operand (forward F(x) of the first layer, backward dY)
    const char *W;      // forward [N, K], backward [K, N]
    const char *bias;   // forward: bfloat16 [N] or NULL
    char *h;            // bfloat16 [rows, N]: written by the forward pass, read by the backward pass
    char *out;          // bfloat16 [rows, N]: F(h), or dh
    CoefRows coef;
    float *partial;     // backward: [G][parts * d_g / CW][kSums]
    int64_t rows;
    int32_t N, dg;
    int32_t slabs, parts, tiles;
};

// The shape of a variant.  KS: contraction in steps of 32; KR: of these in registers, the others in LDS; NT: 16-channel
// tiles of a wavefront.
template <int KS, int KR, int NT, int NW, int TR> struct Shape {
    static constexpr int K = 32 * KS, CW = 16 * NT;
    static constexpr int kPieces = K / 8;                                    // 16-byte pieces of a token's row
    // A token's row in LDS.  Up to 384 rows are 16 bytes apart from the next bank: one lane in sixteen of an operand read meets
    // another's bank, which costs the read a second pass, 38 % of the LDS's cycles at 384.  From 512 on, where the weights in LDS take more of
    // them, pieces of 16 bytes are permuted (xor with the row number, in blocks of sixteen) instead, and none meets: us forward,
    // backward at 25,216 rows, padded / permuted 512 72.4 / 69.3, 103.7 / 101.6, 640 109.6 / 106.2, 156.1 / 153.6, 768 168.4 / 164.7,
    // 232.5 / 229.1.  The addresses are more instructions, though, which is what bounds the narrow ones: 192 37.7 / 38.6 backward, 256
    // 26.1 / 27.5, 46.4 / 47.3, 384 44.3 / 46.0, 71.9 / 72.4.
    static constexpr bool kPermuted = K >= 512;
    static constexpr uint32_t kPitch = K * 2 + (kPermuted ? 0 : 16);
    static __device__ uint32_t swizzle(uint32_t row) { return kPermuted ? (row & 15u) * 16u : 0u; } // bytes
    static constexpr uint32_t kXBuf = TR * kPitch;
    static constexpr int kKept = KS - KR > 2 ? KS - KR : 2;                  // steps a wavefront's own LDS holds (two while loading)
    static constexpr uint32_t kOwn = kKept * NT * 1024u;
    static constexpr size_t kLds = 2 * kXBuf + NW * kOwn;
    static_assert(KS % 2 == 0 && NT % 2 == 0 && kLds <= 160 * 1024 && (!kPermuted || K % 128 == 0), "");
};

template <int KS, int KR, int NT, int NW, int TR, bool BWD>
__global__ __launch_bounds__(64 * NW, NW / 4) void hidden_kernel(const Args a)
{
    using S = Shape<KS, KR, NT, NW, TR>;
    constexpr int kTileRows = TR;
    extern __shared__ __align__(256) char smem[];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t i16 = (uint32_t)lane & 15u, g4 = (uint32_t)lane >> 4;

    // workgroup -> (part of the tokens, slab of channels): the slabs of one part run on one XCD, which then fetches the
    // part's tokens once
    const int xcd = (int)blockIdx.x & 7, slot = (int)blockIdx.x >> 3;
    const int slab = __builtin_amdgcn_readfirstlane(slot % a.slabs);
    const int part = __builtin_amdgcn_readfirstlane(slot / a.slabs) * 8 + xcd;
    const int32_t c0 = (slab * NW + wave) * S::CW; // the wavefront's first channel
    const int cg = __builtin_amdgcn_readfirstlane(c0 / a.dg);
    const Coef<kM, kN> c = load_coef<kM, kN, true, true>(a.coef, cg);

    // ---- weights.  Row r = 4 b + j of matrix tile t stands for channel 32 (t / 2) + 8 b + 4 (t % 2) + j of the
    // wavefront's, so that the two tiles of a pair give lane (i, g) the 8 consecutive channels 32 (t / 2) + 8 g .. of
    // token i.  They are loaded in whole rows (all of them in flight at once) and put in the matrix cores' order through the
    // wavefront's own LDS, two steps of 32 k at a time.
    const uint32_t own = lds0 + 2 * S::kXBuf + (uint32_t)wave * S::kOwn;
    bf16x8 w[KR][NT];
    {
        constexpr int kLoads = 2 * NT; // per two steps: 2 NT KB
        u32x4 raw[KS / 2][kLoads];
        uint32_t src[kLoads], dst[kLoads];
        const uint32_t ld = (BWD ? (uint32_t)a.N : (uint32_t)S::K) * 2u; // bytes between rows
#pragma unroll
        for (int u = 0; u < kLoads; ++u) {
            // forward: CW rows (channels) of 128 bytes of k; backward: 64 rows (k) of 2 CW bytes of channels
            constexpr uint32_t per_row = BWD ? 2 * NT : 8;
            const uint32_t v = (uint32_t)(u * 64 + lane), row = v / per_row, piece = v % per_row;
            src[u] = row * ld + piece * 16u;
            dst[u] = BWD ? v * 16u : row * 128u + ((piece ^ ((row >> 1) & 7u)) * 16u);
        }
        const uint64_t base = reinterpret_cast<uint64_t>(a.W) + (BWD ? (uint64_t)(uint32_t)c0 * 2u : (uint64_t)(uint32_t)c0 * ld);
#pragma unroll
        for (int q = 0; q < KS / 2; ++q)
#pragma unroll
            for (int u = 0; u < kLoads; ++u)
                raw[q][u] = gload16(uniform_u64(base + (BWD ? (uint64_t)(q * 64) * ld : (uint64_t)(q * 128))), src[u]);
        u32x4 rest[KS > KR ? KS - KR : 1][NT];
        static_for<0, KS / 2>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
#pragma unroll
            for (int u = 0; u < kLoads; ++u)
                lds_write16(own + dst[u], raw[q][u]);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); // what other lanes wrote
            static_for<0, 2 * NT>([&](auto fc) {
                constexpr int h = decltype(fc)::value / NT, t = decltype(fc)::value % NT, s = 2 * q + h;
                u32x4 v;
                if constexpr (BWD) {
                    const uint32_t at = own + ((uint32_t)(32 * h) + 8u * g4 + (i16 >> 2)) * (2u * S::CW) +
                                        (uint32_t)(32 * (t / 2) + 4 * (t % 2)) * 2u + (i16 & 3u) * 16u;
                    const u32x2 lo = __builtin_bit_cast(u32x2, lds_read_transposed(at));
                    const u32x2 hi = __builtin_bit_cast(u32x2, lds_read_transposed(at + 4u * 2u * S::CW));
                    v = u32x4{lo[0], lo[1], hi[0], hi[1]};
                } else {
                    const uint32_t ch = (uint32_t)(32 * (t / 2) + 4 * (t % 2)) + 8u * (i16 >> 2) + (i16 & 3u);
                    v = lds_read16(own + ch * 128u + (((uint32_t)(4 * h) + g4) ^ ((ch >> 1) & 7u)) * 16u);
                }
                if constexpr (s < KR)
                    w[s][t] = __builtin_bit_cast(bf16x8, v);
                else
                    rest[s - KR][t] = v;
            });
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); // read before it is written again
        });
        if constexpr (KS > KR)
#pragma unroll
            for (int s = 0; s < KS - KR; ++s)
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    lds_write16(own + (uint32_t)(s * NT + t) * 1024u + (uint32_t)lane * 16u, rest[s][t]);
    }

    // ---- tokens: the tile's rows are one run of memory; 16 bytes per lane and load
    constexpr int kPer = (kTileRows * S::kPieces + 64 * NW - 1) / (64 * NW);
    uint32_t t_at[kPer]; // row of the tile in the upper half, byte of the row in the lower
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const uint32_t v = (uint32_t)(tid + j * 64 * NW);
        t_at[j] = (v / (uint32_t)S::kPieces) << 16 | (v % (uint32_t)S::kPieces) * 16u;
    }
    u32x4 xr[kPer];
    auto load_tile = [&](int32_t t) {
        const int64_t row0 = (int64_t)t * kTileRows;
        const int64_t left = a.rows - row0;
        const uint32_t most = left < kTileRows ? (uint32_t)left - 1u : kTileRows - 1u; // rows past the end read the last one
        const uint64_t base = uniform_u64(reinterpret_cast<uint64_t>(a.x) + (uint64_t)row0 * (uint64_t)(S::K * 2));
#pragma unroll
        for (int j = 0; j < kPer; ++j)
            if ((j + 1) * 64 * NW <= kTileRows * S::kPieces || wave * 64 + j * 64 * NW < kTileRows * S::kPieces)
            {
                keep_in_loop(t_at[j]);
                const uint32_t row = t_at[j] >> 16;
                xr[j] = gload16(base, (row < most ? row : most) * (uint32_t)(S::K * 2) + (t_at[j] & 0xffffu));
            }
    };
    auto put_tile = [&](uint32_t buf) {
#pragma unroll
        for (int j = 0; j < kPer; ++j)
            if ((j + 1) * 64 * NW <= kTileRows * S::kPieces || wave * 64 + j * 64 * NW < kTileRows * S::kPieces)
            {
                keep_in_loop(t_at[j]);
                const uint32_t row = t_at[j] >> 16;
                lds_write16(lds0 + buf + row * S::kPitch + ((t_at[j] & 0xffffu) ^ S::swizzle(row)), xr[j]);
            }
    };

    u32x4 bias[NT / 2];
#pragma unroll
    for (int p = 0; p < NT / 2; ++p) {
        bias[p] = u32x4{0u, 0u, 0u, 0u};
        if (!BWD && a.bias)
            bias[p] = *(const u32x4 *)(a.bias + (size_t)(c0 + 32 * p + 8 * (int)g4) * 2u);
    }
    float sums[kSums];
#pragma unroll
    for (int k = 0; k < kSums; ++k)
        sums[k] = 0.0f;

    const int32_t n_it = part < a.tiles ? (a.tiles - part + a.parts - 1) / a.parts : 0;
    const uint32_t ldn = (uint32_t)a.N * 2u;
    uint32_t out_lane = i16 * ldn + g4 * 16u; // from the sub-tile's first token and the wavefront's first channel
    if (n_it > 0) {
        load_tile(part);
        put_tile(0);
        if (n_it > 1)
            load_tile(part + a.parts);
    }
    // backward: h of a sub-tile, loaded one ahead; tokens past the end read the last one
    u32x4 h_next[NT / 2];
    auto load_h = [&](int64_t row) {
        const int64_t last = a.rows - 1;
        const int64_t from = row < last ? row : last;
        const uint32_t most = last - from < 15 ? (uint32_t)(last - from) : 15u;
        const uint64_t base = uniform_u64(reinterpret_cast<uint64_t>(a.h) + (uint64_t)from * ldn + (uint64_t)(uint32_t)c0 * 2u);
        const uint32_t off = (i16 < most ? i16 : most) * ldn + g4 * 16u;
#pragma unroll
        for (int p = 0; p < NT / 2; ++p)
            h_next[p] = gload16(base, off + (uint32_t)(64 * p));
    };
    if (BWD && n_it > 0)
        load_h((int64_t)part * kTileRows);
    uint32_t buf = 0;
    for (int32_t it = 0; it < n_it; ++it) {
        const int32_t t = part + it * a.parts;
        // this tile is in its buffer, and the other one, of the tile before, has been read by all
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (it + 1 < n_it)
            put_tile(S::kXBuf - buf);
        if (it + 2 < n_it)
            load_tile(t + 2 * a.parts);
        const int64_t row0 = (int64_t)t * kTileRows;
        const int64_t left = a.rows - row0;
        const int64_t row1 = row0 + (int64_t)a.parts * kTileRows; // of the next tile
#pragma unroll 1
        for (int st = 0; st < kTileRows / 16; ++st) {
            const uint64_t at = ((uint64_t)row0 + (uint64_t)(16 * st)) * ldn + (uint64_t)(uint32_t)c0 * 2u;
            const bool valid = (int64_t)(16 * st) + (int64_t)i16 < left;
            u32x4 hv[NT / 2];
            keep_in_loop(out_lane);
            if constexpr (BWD) {
#pragma unroll
                for (int p = 0; p < NT / 2; ++p)
                    hv[p] = h_next[p];
                // of the sub-tile after this one
                load_h(st + 1 < kTileRows / 16 ? row0 + 16 * (st + 1) : row1);
            }
            f32x4 acc[NT];
#pragma unroll
            for (int p = 0; p < NT / 2; ++p) {
                acc[2 * p] = f32x4{low(bias[p][0]), high(bias[p][0]), low(bias[p][1]), high(bias[p][1])};
                acc[2 * p + 1] = f32x4{low(bias[p][2]), high(bias[p][2]), low(bias[p][3]), high(bias[p][3])};
            }
            const uint32_t xf_at = lds0 + buf + ((uint32_t)(16 * st) + i16) * S::kPitch + (g4 * 16u ^ S::swizzle(i16));
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const bf16x8 xf = __builtin_bit_cast(bf16x8, lds_read16(S::kPermuted ? (xf_at ^ (uint32_t)(s % 4) * 64u) + (uint32_t)(s / 4) * 256u : xf_at + (uint32_t)s * 64u));
#pragma unroll
                for (int n = 0; n < NT; ++n) {
                    bf16x8 wf;
                    if (s < KR)
                        wf = w[s < KR ? s : 0][n];
                    else
                        wf = __builtin_bit_cast(bf16x8, lds_read16(own + (uint32_t)((s - KR) * NT + n) * 1024u + (uint32_t)lane * 16u));
                    acc[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, xf, acc[n], 0, 0, 0);
                }
            }
            const uint64_t o_at = uniform_u64(reinterpret_cast<uint64_t>(a.out) + at);
            if constexpr (!BWD) {
                const uint64_t h_at = uniform_u64(reinterpret_cast<uint64_t>(a.h) + at);
#pragma unroll
                for (int p = 0; p < NT / 2; ++p) {
                    const f32x4 u = acc[2 * p], v = acc[2 * p + 1];
                    const u32x4 hw = u32x4{pack(u[0], u[1]), pack(u[2], u[3]), pack(v[0], v[1]), pack(v[2], v[3])};
                    const u32x4 f = rational8(hw, c);
                    if (valid) {
                        gstore16(h_at, out_lane + (uint32_t)(64 * p), hw);
                        gstore16(o_at, out_lane + (uint32_t)(64 * p), f);
                    }
                }
            } else {
                if (left < kTileRows) { // tokens past the end add nothing to the sums (a whole tile needs no selects)
#pragma unroll
                    for (int n = 0; n < NT; ++n)
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            acc[n][j] = valid ? acc[n][j] : 0.0f;
#pragma unroll
                    for (int p = 0; p < NT / 2; ++p)
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            hv[p][j] = valid ? hv[p][j] : 0u;
                }
#pragma unroll
                for (int p = 0; p < NT / 2; ++p) {
                    // dF rounded to bfloat16, as the tensor that a product of its own would write
                    const f32x4 u = acc[2 * p], v = acc[2 * p + 1];
                    const u32x4 dw = u32x4{pack(u[0], u[1]), pack(u[2], u[3]), pack(v[0], v[1]), pack(v[2], v[3])};
                    float dx[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const uint32_t word = hv[p][e / 2], d = dw[e / 2];
                        dx[e] = bwd_elem<false, kM, kN>(e % 2 == 0 ? low(word) : high(word), e % 2 == 0 ? low(d) : high(d), c, sums);
                        if (e % 4 == 3)
                            fence_schedule(); // (more elements at a time do not fit the registers)
                    }
                    const u32x4 d = u32x4{pack(dx[0], dx[1]), pack(dx[2], dx[3]), pack(dx[4], dx[5]), pack(dx[6], dx[7])};
                    if (valid)
                        gstore16(o_at, out_lane + (uint32_t)(64 * p), d);
                }
            }
        }
        buf = S::kXBuf - buf;
    }

    if constexpr (BWD) {
        negate_b_sums<kM, kN>(sums);
        const int32_t per_group = a.dg / S::CW; // wavefronts of a part that share the group
        const int64_t row = (int64_t)cg * ((int64_t)a.parts * per_group) + (int64_t)part * per_group + (c0 - cg * a.dg) / S::CW;
#pragma unroll
        for (int k = 0; k < kSums; ++k) {
            const float s = wave_sum(sums[k]);
            if (lane == 0)
                a.partial[row * kSums + k] = s;
        }
    }
}

// --------------------------------------------------------------------------
// host side
// --------------------------------------------------------------------------
using Kernel = void (*)(const Args);

struct Variant {
    int32_t K, CW, waves, tile_rows;
    int32_t fwd_units, bwd_units; // compute units that have to get a workgroup for a large call to be the faster route (pays)
    size_t lds;
    Kernel fwd, bwd;
};

template <int KS, int KR, int NT, int NW, int TR = 32>
static constexpr Variant variant(int32_t fwd_units, int32_t bwd_units)
{
    using S = Shape<KS, KR, NT, NW, TR>;
    return Variant{S::K, S::CW, NW, TR, fwd_units, bwd_units, S::kLds,
                   hidden_kernel<KS, KR, NT, NW, TR, false>, hidden_kernel<KS, KR, NT, NW, TR, true>};
}

// The contractions that are built: the widths 192, 384 and 768 of the model table, and of the other multiples of 64 those that
// are multiples of 128.  (Any even number of steps fits the template; 320, 448, 576 and 704 are neither built nor measured, and
// such a block runs its layers one by one.)
//
// us at 25,216 rows, forward / backward (two 16-channel tiles a wavefront but for the last column; twelve wavefronts are
// three per SIMD of 168 registers each, eight are two of 256):
//   K = 192: 12 wavefronts 20.3 / 37.9   8: 21.9 / 37.6                                 8 of 96 channels 24.2 / 44.5
//   K = 256:  8 wavefronts 26.5 / 46.2  16: 25.7 / 66 (spills)                          8 of 64 channels 27.9 / 46.9
//   K = 384: 12 wavefronts 44.1 / 69.9 (two steps of the weights in LDS)  8: 47.0 / 75.2   8 of 64 channels 44.0 / 78.4
//   K = 512:  8 wavefronts 69 / 102   K = 640: 106 / 154   K = 768: 165 / 229
// (192 - 384 before bwd_elem took the sign by a clamp; backward since: K = 192 0.5 %, 384 2.7 % less.)
static const Variant kVariants[] = {variant<6, 6, 2, 12>(0, 176), variant<8, 8, 2, 8>(0, 192), variant<12, 10, 2, 12>(0, 176),
                                    variant<16, 14, 2, 8>(160, 192), variant<20, 16, 2, 8>(176, 192),
                                    variant<24, 18, 2, 8, 16>(192, 208)};

// The variant of a shape, or NULL: whole slabs of the workgroup's wavefronts, each of these within one coefficient group.
static const Variant *variant_of(int32_t K, int32_t N, int32_t G)
{
    for (const Variant &v : kVariants)
        if (v.K == K && N > 0 && G > 0 && N % (v.waves * v.CW) == 0 && N / (v.waves * v.CW) <= 32 && N % G == 0 && N / G % v.CW == 0)
            return &v;
    return nullptr;
}

// Whether the kernel is the faster route than a product and the rational function's own kernel.
//
// (The table below was measured with a library product, which is up to 1.6 times slower here than grkan_product, and not again: the
// lines lie where the kernels win against the former.  Against grkan_product both still pay in whole blocks of widths 192 - 640, 4 x as wide:
// us with both / neither 192 236 / 264 and 640 1,309 / 1,384 at 50,432 rows, 640 152 / 168 at 3,152.  The forward one at 768 -> 3072
// does not: with it / with neither 447 / 434 at 12,608 rows, 844 / 836 at 25,216, 1,637 / 1,619 at 50,432.)
// Large calls: a number of slabs that does not divide the 32 compute units of an XCD leaves units without a workgroup, and how
// many of these the kernel can do without falls with K: the more of the weights is in LDS, the nearer it is to what it replaces.
// Measured on MI355X in whole training blocks (forward and backward pass, 18 numbers of slabs, 6,304 - 50,432 rows; what the block
// is slower, in per cent of its time, with the two kernels in place of the forward one, and of the backward one):
//   units       240, 256             208 - 224            192 (12, 24 slabs)    176 (11, 22)          160 (20)              136 (17)
//   K = 192     3 .. 16,  5 .. 17    6 .. 11,  6 .. 11    3 .. 9,   2 .. 5      4 .. 10,  3 .. 15     -1 .. 2, -4 .. -1     0 .. 3,   1 .. 7
//   K = 256     3 .. 12,  5 .. 8     3 .. 16,  3 .. 9     4 .. 10,  1 .. 3      6 .. 11, -2 .. 3       3,      -5 .. -2     2 .. 5,  -9 .. -3
//   K = 384     4 .. 15,  6 .. 15    8 .. 16,  5 .. 11    5 .. 9,   2 .. 5      6 .. 13,  1 .. 10      2 .. 3, -2 .. -1     4 .. 5,   0 .. 4
//   K = 512     3 .. 14,  3 .. 9     2 .. 13,  3 .. 7     1 .. 11,  0 .. 6      5 .. 13, -1 .. 1       1 .. 3, -4 .. -3    -3 .. 8,  -8 .. -4
//   K = 640     2 .. 10,  1 .. 12    2 .. 8,   1 .. 7     1 .. 7,   0 .. 5      0 .. 8,  -3 .. 0      -1 .. 0, -4          -1 .. 5,  -8 .. -5
//   K = 768     2 .. 9,   1 .. 11   -1 .. 8,   0 .. 5     0 .. 6,  -1 .. 1     -2 .. 7,  -4 .. -1     -2,      -6 .. -5    -3 .. 2,  -9 .. -5
// 768 -> 3072 is twelve slabs; us of the block with both kernels / the forward one / neither: 9,456 rows 430 / 419 / 421,
// 25,216 1,032 / 1,015 / 1,047, 50,432 1,859 / 1,783 / 1,818.  (Timed by themselves, over the same buffers again and again, the
// two kernels look up to a tenth better than in a block: the one finds in the caches what the other has just written.)
//
// Calls of less than 24 million hidden activations are bound by the host, which has one launch less to make: 768 -> 3072 211 /
// 214 / 229 us at 3,152 rows (by themselves the kernels take 84 us there, the two of each direction 70), 299 / 302 / 321 at 6,304.
static bool pays(const Variant &v, int64_t rows, int32_t N, bool backward)
{
    const int32_t slabs = N / (v.waves * v.CW), units = 8 * (32 / slabs) * slabs;
    return rows * N < 24000000 || units >= (backward ? v.bwd_units : v.fwd_units);
}

static bool allow_lds(const Variant &v)
{
    static std::mutex mu;
    static bool done[64][sizeof(kVariants) / sizeof(kVariants[0])];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64)
        return false;
    std::lock_guard<std::mutex> lock(mu);
    bool &is = done[dev][&v - kVariants];
    if (!is)
        is = hipFuncSetAttribute(reinterpret_cast<const void *>(v.fwd), hipFuncAttributeMaxDynamicSharedMemorySize, (int)v.lds) == hipSuccess &&
             hipFuncSetAttribute(reinterpret_cast<const void *>(v.bwd), hipFuncAttributeMaxDynamicSharedMemorySize, (int)v.lds) == hipSuccess;
    return is;
}

// One workgroup per compute unit; the slabs of a part on one XCD of 32 units, as many parts on each as fit.
static void divide(const Variant &v, int64_t rows, int32_t N, Args *a)
{
    a->slabs = N / (v.waves * v.CW);
    a->tiles = (int32_t)((rows + v.tile_rows - 1) / v.tile_rows);
    const int32_t most = 8 * (32 / a->slabs), few = (a->tiles + 7) / 8 * 8;
    a->parts = few < most ? few : most;
}

static grkan_status_t run(bool backward, const void *x, const void *W, const void *bias, void *h, void *out, const CoefRows &coef,
                          void *dA, void *dB, void *workspace, size_t workspace_bytes, int64_t rows, int32_t K, int32_t N, int32_t G,
                          hipStream_t stream, CoefSums *later = nullptr)
{
    if (rows < 0 || K <= 0 || N <= 0 || G <= 0)
        return GRKAN_ERR_SHAPE;
    const Variant *const v = variant_of(K, N, G);
    if (!v || rows > (int64_t)1 << 30)
        return GRKAN_ERR_UNSUPPORTED;
    if (!W || !coef.A || !coef.B || (rows > 0 && (!x || !h || !out)) || (backward && (!dA || !dB)))
        return GRKAN_ERR_NULL;
    if ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(W) | reinterpret_cast<uintptr_t>(bias) |
         reinterpret_cast<uintptr_t>(h) | reinterpret_cast<uintptr_t>(out) | reinterpret_cast<uintptr_t>(workspace)) % 16 != 0 ||
        (reinterpret_cast<uintptr_t>(coef.A) | reinterpret_cast<uintptr_t>(coef.B) | reinterpret_cast<uintptr_t>(dA) |
         reinterpret_cast<uintptr_t>(dB)) % 2 != 0)
        return GRKAN_ERR_ALIGN;
    if (rows == 0 && !backward)
        return GRKAN_OK;
    Args a;
    a.x = static_cast<const char *>(x);
    a.W = static_cast<const char *>(W);
    a.bias = static_cast<const char *>(bias);
    a.h = static_cast<char *>(h);
    a.out = static_cast<char *>(out);
    a.coef = coef;
    a.partial = static_cast<float *>(workspace);
    a.rows = rows;
    a.N = N;
    a.dg = N / G;
    divide(*v, rows, N, &a);
    const int32_t rows_per_group = a.parts * (a.dg / v->CW);
    if (backward && rows_per_group > 0 &&
        (!workspace || workspace_bytes < (size_t)G * (size_t)rows_per_group * kSums * sizeof(float)))
        return GRKAN_ERR_WORKSPACE;
    if (a.parts > 0) {
        if (!allow_lds(*v))
            return GRKAN_ERR_LAUNCH;
        void *args[] = {&a};
        if (hipLaunchKernel(reinterpret_cast<const void *>(backward ? v->bwd : v->fwd), dim3((unsigned)(a.parts * a.slabs)),
                            dim3(64 * v->waves), args, v->lds, stream) != hipSuccess)
            return GRKAN_ERR_LAUNCH;
    }
    if (later) {
        *later = CoefSums{a.partial, rows_per_group, coef, dA, dB, G};
        return GRKAN_OK;
    }
    return backward ? run_stage2(a.partial, rows_per_group, coef, dA, dB, G, kM, kN, stream) : GRKAN_OK;
}

} // namespace hidden

grkan_status_t hidden_bwd_stage1(const void *dout, const void *W, const void *h, const CoefRows &coef, void *dh, void *dA, void *dB,
                                 grkan_alloc_t alloc, void *alloc_context, int64_t rows, int32_t K, int32_t N, int32_t G, CoefSums *later,
                                 hipStream_t stream)
{
    const size_t need = grkan_hidden_workspace_bytes(rows, K, N, G);
    if (need == 0)
        return GRKAN_ERR_UNSUPPORTED;
    void *const workspace = alloc(need, alloc_context);
    if (!workspace)
        return GRKAN_ERR_WORKSPACE;
    return hidden::run(true, dout, W, nullptr, const_cast<void *>(h), dh, coef, dA, dB, workspace, need, rows, K, N, G, stream, later);
}

} // namespace grkan

using namespace grkan;

extern "C" int32_t grkan_hidden_supported(int32_t K, int32_t N, int32_t G) { return hidden::variant_of(K, N, G) != nullptr; }

extern "C" int32_t grkan_hidden_pays(int64_t rows, int32_t K, int32_t N, int32_t G, int32_t backward)
{
    const hidden::Variant *const v = hidden::variant_of(K, N, G);
    return v != nullptr && hidden::pays(*v, rows, N, backward != 0);
}

extern "C" size_t grkan_hidden_workspace_bytes(int64_t rows, int32_t K, int32_t N, int32_t G)
{
    const hidden::Variant *const v = hidden::variant_of(K, N, G);
    if (!v || rows < 0 || rows > (int64_t)1 << 30)
        return 0;
    hidden::Args a;
    hidden::divide(*v, rows, N, &a);
    const size_t need = (size_t)G * (size_t)a.parts * (size_t)(N / G / v->CW) * hidden::kSums * sizeof(float);
    return need > 0 ? need : 16;
}

extern "C" grkan_status_t grkan_hidden_fwd(const void *y, const void *W, const void *bias, const void *A, const void *B, void *h,
                                           void *f, int64_t rows, int32_t K, int32_t N, int32_t G, int32_t shared_numerator,
                                           void *hip_stream)
{
    const CoefRows coef{A, B, shared_numerator ? 0 : hidden::kM + 1, 1};
    return hidden::run(false, y, W, bias, h, f, coef, nullptr, nullptr, nullptr, 0, rows, K, N, G, static_cast<hipStream_t>(hip_stream));
}

extern "C" grkan_status_t grkan_hidden_bwd(const void *dout, const void *W, const void *h, const void *A, const void *B, void *dh,
                                           void *dA, void *dB, void *workspace, size_t workspace_bytes, int64_t rows, int32_t K,
                                           int32_t N, int32_t G, int32_t shared_numerator, void *hip_stream)
{
    const CoefRows coef{A, B, shared_numerator ? 0 : hidden::kM + 1, 1};
    return hidden::run(true, dout, W, nullptr, const_cast<void *>(h), dh, coef, dA, dB, workspace, workspace_bytes, rows, K, N, G,
                       static_cast<hipStream_t>(hip_stream));
}
