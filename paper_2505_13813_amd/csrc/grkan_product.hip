// The matrix products of a KAT MLP block on gfx950 (MI355X), bfloat16 in and out, float32 sums:
//
//     out = x W^T + bias          (W [N, K], forward)           optionally out = F(x W^T + bias), F the group-wise rational
//     out = x W                   (W [K, N], backward)          function of the next layer on the rounded result
//                                                               dx, and F's coefficient sums, with x W as F's upstream gradient
//
// A workgroup owns a tile of rows x channels and walks K in stages of 64: whole 128-byte lines of both operands come to LDS by
// LDS-direct loads, NBUF stages deep.  16-byte pieces of a row are permuted (xor with the row number), so that operand reads
// hit all banks; where W has the contraction as its slow dimension it comes as it lies and is transposed on the way out of LDS
// (ds_read_b64_tr_b16), its rows numbered so that both operands count k alike.
//
//   * Wavefronts of their own (LD of them) issue the loads: a wavefront that waits to hand a load to a busy memory pipe cannot
//     issue matrix instructions meanwhile.  6,304 x 3072 -> 768 in 160 x 128 tiles 33.3 -> 28.9 us, 25,216 x 1536 -> 384 in 224 x 192
//     33.3 -> 30.1.  (The 320 x 256 tile has no registers for a third wavefront per SIMD, and hides more behind a longer stage.)
//   * The others multiply, with one barrier per stage: it stands behind the first of TM rows of tiles, when every wavefront has the
//     stage's operands in registers.  Behind it the next stage's are read, each row of tiles behind the last use of its registers,
//     W's into a second set.  (With the reads just in front of their use, and the barrier among them, 160 x 128 with two workgroups
//     per unit took 45.6 us for 3,152 x 3072 -> 768, with this order 36.8.)
//   * The result leaves through LDS in whole rows; F is evaluated there, where a lane holds eight channels of one group.
//
// Measured on one MI355X against the library's product, us (by itself, over the same buffers):
//   25,216 x 1536 -> 384  29 against 35 - 38    6,304 x 3072 -> 768  28 against 32 - 36    6,304 x 768 -> 3072  31 against 48 (37 with F)
//   25,216 x 384 -> 1536  37 against 59         25,216 x 3072 -> 768 89 against 146        50,432 x 768 -> 3072 227 - 237 against 227
// It loses where the library's rounds of tiles are full, or its contraction is split over the chip: 12,608 x 640 -> 2560 46 against 42,
// 25,216 x 2048 -> 256 34 against 31, x 6400 -> 256 137 against 95, 50,432 x 768 -> 8192 664 against 559.
// What bounds it: at 6,304 x 3072 -> 768 the loads alone take 24 of the 29 us, the matrix instructions alone 19, the LDS
// reads alone 16 (launch, first loads and result 5 in each); at 25,216 x 3072 -> 768 59, 66 and 33 of the 97 that it took on
// that card, with the clock at 2.2 GHz.
#include <hip/hip_runtime.h>

#include <mutex>

#include "grkan_plan.h"
#include "grkan_tile.h"

namespace grkan {
namespace product {

using namespace tile;

constexpr int kM = 5, kN = 4, kSums = kM + 1 + kN;

struct Args {
    const char *x;    // bfloat16 [M, K]
    const char *W;    // bfloat16 [N, K]; TRANSPOSED: [K, N]
    const char *bias; // bfloat16 [N] or NULL
    char *out;        // bfloat16 [M, N]
    CoefRows coef;    // of F
    const char *fx;   // kBackward: F's input, bfloat16 [M, N]; out is the gradient for it
    float *partial;   // kBackward: [groups][partial_rows][kSums]
    int64_t M;
    int32_t N, K;
    int32_t dg;       // F's channels per group
    int32_t tiles_n, tiles, per_xcd;
    int32_t partial_rows, tile0; // kBackward: rows per group, and row tiles of launches before this one
};

// What becomes of the product: nothing; F on it; F's backward pass with it.
enum Then { kPlain, kRational, kBackward };

// A wavefront's share is TM x TN tiles of 16 x 16, a workgroup WM x WN such wavefronts and LD that load; PER workgroups per
// compute unit.
template <int TM_, int TN_, int WM_, int WN_, int NBUF_, int LD_, int PER_ = 1> struct Shape {
    static constexpr int TM = TM_, TN = TN_, WM = WM_, WN = WN_, NBUF = NBUF_, LD = LD_, PER = PER_;
    static constexpr int BM = 16 * TM * WM, BN = 16 * TN * WN, kWaves = WM * WN, kThreads = 64 * (kWaves + LD);
    static constexpr int kFetchers = LD ? LD : kWaves;      // wavefronts that load
    static constexpr uint32_t kXB = BM * 128u, kWB = BN * 128u, kStage = kXB + kWB;
    static constexpr int kLoads = (BM + BN) / 8;            // of a stage, 1 KB each
    static constexpr int kHi = (kLoads + kFetchers - 1) / kFetchers, kLo = kLoads / kFetchers, kRem = kLoads % kFetchers;
    static constexpr uint32_t kPitch = BN * 2 + 16;         // of the result's rows in LDS
    static constexpr int kParts = (size_t)BM * kPitch > 160 * 1024 ? 2 : 1, kMP = (TM + kParts - 1) / kParts; // it leaves in parts
    static constexpr size_t kMain = (size_t)NBUF * kStage, kRows = (size_t)WM * kMP * 16 * kPitch;
    static constexpr size_t kLds = kMain > kRows ? kMain : kRows;
    // Registers of their own for the last row of tiles' next operand: it can then be read with the others, well in front of the
    // barrier that waits for all reads.  (The largest tile has none left.)
    static constexpr bool kTwoLast = TM * TN < 40;
    static_assert(2 * (TM - 1) >= TN && PER * kLds <= 160 * 1024 && TM >= 2 && (kWaves + LD) % 4 == 0, "");
};

template <class SH, bool TRANSPOSED, Then THEN>
__global__ __launch_bounds__(SH::kThreads, SH::PER *SH::kThreads / 256) void product_kernel(const Args a)
{
    constexpr int TM = SH::TM, TN = SH::TN, NBUF = SH::NBUF, BM = SH::BM, BN = SH::BN;
    constexpr uint32_t NP = BN / 16; // 32-byte column pairs of a row of W, TRANSPOSED
    extern __shared__ __align__(128) char smem[]; // the second half of a row's 64 k is read at the first's address xor 64
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t i16 = (uint32_t)lane & 15u, g4 = (uint32_t)lane >> 4;
    const bool computes = SH::LD == 0 || wave < SH::kWaves, fetches = SH::LD == 0 || wave >= SH::kWaves;

    // workgroups go round-robin over the 8 XCDs; each gets a run of tiles in row order, whose rows of x its L2 fetches once
    const int32_t lin = ((int32_t)blockIdx.x & 7) * a.per_xcd + ((int32_t)blockIdx.x >> 3);
    if (lin >= a.tiles)
        return;
    const int32_t tm = __builtin_amdgcn_readfirstlane(lin / a.tiles_n);
    const int32_t tn = lin - tm * a.tiles_n;
    const int64_t row0 = (int64_t)tm * BM;
    const int32_t col0 = tn * BN;
    const int32_t T = a.K / 64;
    const uint32_t ldk = (uint32_t)a.K * 2u, ldn = (uint32_t)a.N * 2u;

    // ---- loads: load u of a stage fills KB u of its buffer.  x (and W): rows of 128 bytes, 16-byte piece p of row r at slot
    // p xor (r / 2 mod 8).  W transposed: 64 rows of BN channels, slot row r holding k = 8 (r / 4 mod 4) + r mod 4 + 4 (r / 16 mod 2)
    // of its 32, column pairs rotated by the row.  Rows and columns past the end repeat the last (their results are not stored).
    const int fw = SH::LD ? wave - SH::kWaves : wave;
    uint32_t off[SH::kHi];
    {
        const int64_t left = a.M - row0;
        const uint32_t last_x = left < BM ? (uint32_t)left - 1u : (uint32_t)BM - 1u;
        const uint32_t last_w = a.N - col0 < BN ? (uint32_t)(a.N - col0) - 1u : (uint32_t)BN - 1u;
#pragma unroll
        for (int q = 0; q < SH::kHi; ++q) {
            const uint32_t u = (uint32_t)(fw + q * SH::kFetchers);
            const bool isx = u * 8u < (uint32_t)BM;
            if (isx || !TRANSPOSED) {
                const uint32_t row = (isx ? u * 8u : u * 8u - BM) + ((uint32_t)lane >> 3), last = isx ? last_x : last_w;
                const uint32_t piece = ((uint32_t)lane & 7u) ^ ((row >> 1) & 7u);
                off[q] = (row < last ? row : last) * ldk + piece * 16u;
            } else {
                const uint32_t e = (u - BM / 8u) * 64u + (uint32_t)lane;
                const uint32_t r = e / (2u * NP), s = e % (2u * NP);
                const uint32_t rot = BN % 128 == 0 ? (r & 15u) % NP : ((r & 15u) >> 1) % NP;
                const uint32_t k = (r & 32u) + 8u * ((r >> 2) & 3u) + (r & 3u) + ((r >> 4) & 1u) * 4u;
                const uint32_t c = 2u * (((s >> 1) + NP - rot) % NP) + (s & 1u), most = (last_w + 1u) / 8u - 1u;
                off[q] = k * ldn + (c < most ? c : most) * 16u;
            }
        }
    }
    const uint64_t x_base = reinterpret_cast<uint64_t>(a.x) + (uint64_t)row0 * ldk;
    const uint64_t w_base = reinterpret_cast<uint64_t>(a.W) + (TRANSPOSED ? (uint64_t)(uint32_t)col0 * 2u : (uint64_t)(uint32_t)col0 * ldk);
    auto fetch_one = [&](auto qc, int32_t t, uint32_t buf) {
        constexpr int q = decltype(qc)::value;
        const int u = fw + q * SH::kFetchers;
        if ((q + 1) * SH::kFetchers <= SH::kLoads || u < SH::kLoads) {
            const uint64_t base = u * 8 < BM ? x_base + (uint64_t)t * 128u : w_base + (uint64_t)t * (TRANSPOSED ? (uint64_t)ldn * 64u : 128u);
            load_to_lds(uniform_u64(base), off[q], lds0 + buf + (uint32_t)u * 1024u);
        }
    };
    auto wait_for = [&](auto ahead, bool more) { // all but the last `ahead` stages' loads, then for everyone
        constexpr int kAhead = decltype(ahead)::value;
        if (!more)
            wait_loads<0>();
        else if (SH::kRem == 0 || fw < SH::kRem)
            wait_loads<kAhead * SH::kHi>();
        else
            wait_loads<kAhead * SH::kLo>();
        asm volatile("s_barrier" ::: "memory");
    };

    // ---- operand reads: 16 rows (x) or 16 channels (W) x 32 k, lane (i, g) row or channel i, k = 8 g ..
    const int wm = wave / SH::WN, wn = wave % SH::WN;
    const uint32_t piece0 = g4 ^ ((i16 >> 1) & 7u);
    const uint32_t x_at = lds0 + ((uint32_t)(wm * TM * 16) + i16) * 128u + piece0 * 16u; // second half of 64 k: xor 64
    const uint32_t w_at = lds0 + SH::kXB + ((uint32_t)(wn * TN * 16) + i16) * 128u + piece0 * 16u;
    uint32_t wt_at[TN];
    if constexpr (TRANSPOSED) {
        const uint32_t r15 = g4 * 4u + (i16 >> 2), rot = BN % 128 == 0 ? r15 % NP : (r15 >> 1) % NP;
#pragma unroll
        for (int n = 0; n < TN; ++n)
            wt_at[n] = lds0 + SH::kXB + r15 * (BN * 2u) + (((uint32_t)(wn * TN + n) + rot) % NP) * 32u + (i16 & 3u) * 8u;
    }
    auto read_x = [&](uint32_t buf, int h, int m) { return lds_read16(((x_at + buf) ^ (uint32_t)(h * 64)) + (uint32_t)m * 2048u); };
    auto read_w = [&](uint32_t buf, int h, int n) {
        if constexpr (TRANSPOSED) {
            const uint32_t at = wt_at[n] + buf + (uint32_t)(h * 32) * (BN * 2u);
            const u32x2 lo = __builtin_bit_cast(u32x2, lds_read_transposed(at));
            const u32x2 hi = __builtin_bit_cast(u32x2, lds_read_transposed(at + 16u * (BN * 2u)));
            return u32x4{lo[0], lo[1], hi[0], hi[1]};
        } else {
            return lds_read16(((w_at + buf) ^ (uint32_t)(h * 64)) + (uint32_t)n * 2048u);
        }
    };

    f32x4 acc[TM][TN];
#pragma unroll
    for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int n = 0; n < TN; ++n)
            acc[m][n] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

    // One step of 32 k, half h of stage t: multiplies with x and wc while the next step's operands are read into x, each row of
    // tiles behind its own last use, and wn_.  In the second half, behind the first row of tiles, the barrier: every
    // wavefront has its operands of this stage, so that its buffer is free for stage t + NBUF, and stage t + 1 has landed.
    // (Behind the last stage the next buffer is read too, and not used.)
    auto step = [&](auto hc, int32_t t, uint32_t buf, uint32_t buf_next, u32x4(&x)[TM - 1], u32x4(&last)[2], u32x4(&wc)[TN], u32x4(&wn_)[TN]) {
        constexpr int h = decltype(hc)::value;
        const uint32_t from = h == 1 ? buf_next : buf;
        const bool more = t + NBUF < T;
        static_for<0, TM>([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            if constexpr (h == 1 && m == 1 && SH::LD > 0)
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            if constexpr (h == 1 && m == 1 && SH::LD == 0)
                wait_for(std::integral_constant<int, NBUF - 2>{}, t + NBUF - 1 < T);
            // reads (and loads) between the matrix instructions: one after the other they would wait for the LDS with the matrix
            // core idle
            constexpr int n0 = m > 0 ? (2 * m - 2 < TN ? 2 * m - 2 : TN) : 0, n1 = 2 * m < TN ? 2 * m : TN; // W's of this group
            constexpr int kX = m > 0 ? 1 : 0, kLast = m == (SH::kTwoLast ? TM - 1 : 0) ? 1 : 0;
            constexpr bool loads = h == 1 && m >= 1 && SH::LD == 0;
            constexpr int q0 = loads ? (m - 1) * SH::kHi / (TM - 1) : 0, q1 = loads ? m * SH::kHi / (TM - 1) : 0;
            constexpr int kOps = kX + (n1 - n0) + kLast + (q1 - q0);
            static_for<0, TN>([&](auto nc) {
                constexpr int n = decltype(nc)::value;
                static_for<0, kOps>([&](auto oc) {
                    constexpr int o = decltype(oc)::value;
                    if constexpr (o * TN / kOps == n) {
                        if constexpr (o < kX)
                            x[m - 1] = read_x(from, 1 - h, m - 1);
                        else if constexpr (o < kX + n1 - n0)
                            wn_[n0 + o - kX] = read_w(from, 1 - h, n0 + o - kX);
                        else if constexpr (o < kX + n1 - n0 + kLast)
                            last[SH::kTwoLast ? 1 - h : 0] = SH::kTwoLast ? read_x(from, 1 - h, TM - 1) : read_x(buf, h, TM - 1);
                        else if (more)
                            fetch_one(std::integral_constant<int, q0 + o - kX - kLast - (n1 - n0)>{}, t + NBUF, buf);
                    }
                });
                fence_schedule();
                acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wc[n]), __builtin_bit_cast(bf16x8, m < TM - 1 ? x[m < TM - 1 ? m : 0] : last[SH::kTwoLast ? h : 0]),
                                                                    acc[m][n], 0, 0, 0);
                fence_schedule();
            });
        });
    };
    auto advance = [&](uint32_t b) { return b + SH::kStage == NBUF * SH::kStage ? 0u : b + SH::kStage; };

    // every wavefront passes T + 1 barriers here
    if (fetches) {
        static_for<0, NBUF>([&](auto sc) {
            constexpr int s = decltype(sc)::value;
            if (s < T)
                static_for<0, SH::kHi>([&](auto qc) { fetch_one(qc, s, (uint32_t)s * SH::kStage); });
        });
        wait_for(std::integral_constant<int, NBUF - 1>{}, NBUF <= T);
    } else {
        asm volatile("s_barrier" ::: "memory");
    }
    if (!computes) {
        uint32_t buf = 0;
        for (int32_t t = 0; t < T; ++t) {
            wait_for(std::integral_constant<int, NBUF - 2>{}, t + NBUF - 1 < T);
            if (t + NBUF < T)
                static_for<0, SH::kHi>([&](auto qc) { fetch_one(qc, t + NBUF, buf); });
            buf = advance(buf);
        }
    } else {
        u32x4 x[TM - 1], last[2], wa[TN], wb[TN]; // (as words: carried around the loop as bfloat16 the compiler takes them apart)
#pragma unroll
        for (int n = 0; n < TN; ++n)
            wa[n] = read_w(0, 0, n);
#pragma unroll
        for (int m = 0; m < TM - 1; ++m)
            x[m] = read_x(0, 0, m);
        if (SH::kTwoLast)
            last[0] = read_x(0, 0, TM - 1);
        uint32_t buf = 0;
        for (int32_t t = 0; t < T; ++t) {
            const uint32_t next = advance(buf);
            step(std::integral_constant<int, 0>{}, t, buf, next, x, last, wa, wb);
            step(std::integral_constant<int, 1>{}, t, buf, next, x, last, wb, wa);
            buf = next;
        }
    }

    // ---- result: bias, bfloat16, to LDS; from there in whole rows, eight channels a lane, through F
    __syncthreads();
    u32x2 bias[TN];
#pragma unroll
    for (int n = 0; n < TN; ++n) {
        const int32_t c = col0 + (wn * TN + n) * 16 + (int32_t)g4 * 4;
        bias[n] = computes && a.bias && c < a.N ? *(const u32x2 *)(a.bias + (size_t)c * 2u) : u32x2{0u, 0u};
    }
    constexpr int LR = BN / 8, RP = SH::kThreads / LR, MP = SH::kMP; // lanes per row, rows at a time
    const int32_t c = col0 + (tid % LR) * 8;
    const bool in = tid < RP * LR && c < a.N;
    Coef<kM, kN> co;
    if constexpr (THEN != kPlain)
        if (in)
            co = load_coef<kM, kN, false, true>(a.coef, c / a.dg);
    const int64_t left = a.M - row0;
    const int rows = left < BM ? (int)left : BM;
    const size_t at_c = ((size_t)row0 * (size_t)a.N + (size_t)c) * 2u;
    char *const to = a.out + at_c;
    // kBackward: F's input, on its way while the product goes through LDS
    constexpr int kPass = THEN == kBackward ? (BM + RP - 1) / RP : 1;
    u32x4 fx[kPass];
    if constexpr (THEN == kBackward) {
        static_assert(SH::kParts == 1, "rows of the tile are rows of the result in LDS");
#pragma unroll
        for (int j = 0; j < kPass; ++j) {
            const int r = tid / LR + j * RP;
            fx[j] = in && r < rows ? *(const u32x4 *)(a.fx + at_c + (size_t)r * ldn) : u32x4{0u, 0u, 0u, 0u};
        }
    }
    static_for<0, SH::kParts>([&](auto pc) {
        constexpr int m0 = decltype(pc)::value * MP, m1 = m0 + MP < TM ? m0 + MP : TM; // rows of tiles in this part
        if (m0 > 0)
            __syncthreads();
        if (computes) {
#pragma unroll
            for (int m = m0; m < m1; ++m) {
                const uint32_t at = lds0 + ((uint32_t)(wm * MP + m - m0) * 16u + i16) * SH::kPitch + (uint32_t)(wn * TN * 32) + g4 * 8u;
#pragma unroll
                for (int n = 0; n < TN; ++n) {
                    const f32x4 v = acc[m][n];
                    *(__attribute__((address_space(3))) u32x2 *)(uintptr_t)(at + (uint32_t)n * 32u) =
                        u32x2{pack(v[0] + low(bias[n][0]), v[1] + high(bias[n][0])), pack(v[2] + low(bias[n][1]), v[3] + high(bias[n][1]))};
                }
            }
        }
        __syncthreads();
        if (THEN != kBackward && in) {
#pragma unroll 2
            for (int l = tid / LR; l < SH::WM * MP * 16; l += RP) {
                const int m = m0 + l / 16 % MP, r = (l / (MP * 16) * TM + m) * 16 + l % 16;
                if (m >= m1 || r >= rows)
                    continue;
                u32x4 v = lds_read16(lds0 + (uint32_t)l * SH::kPitch + (uint32_t)(tid % LR) * 16u);
                if constexpr (THEN == kRational)
                    v = rational8(v, co);
                *(u32x4 *)(to + (size_t)r * ldn) = v;
            }
        }
    });
    if constexpr (THEN == kBackward) {
        // dx of the lane's eight channels, row by row, and the sums over them; a workspace row for every eight channels of the tile
        float sums[kSums];
#pragma unroll
        for (int k = 0; k < kSums; ++k)
            sums[k] = 0.0f;
#pragma unroll
        for (int j = 0; j < kPass; ++j) {
            const int r = tid / LR + j * RP;
            if (in && r < rows) {
                const u32x4 v = lds_read16(lds0 + (uint32_t)r * SH::kPitch + (uint32_t)(tid % LR) * 16u);
                float dx[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const uint32_t word = fx[j][e / 2], d = v[e / 2];
                    dx[e] = bwd_elem<false, kM, kN>(e % 2 == 0 ? low(word) : high(word), e % 2 == 0 ? low(d) : high(d), co, sums);
                }
                *(u32x4 *)(to + (size_t)r * ldn) = u32x4{pack(dx[0], dx[1]), pack(dx[2], dx[3]), pack(dx[4], dx[5]), pack(dx[6], dx[7])};
            }
        }
        negate_b_sums<kM, kN>(sums);
        static_assert((size_t)kSums * SH::kThreads * 4 <= SH::kLds, "");
        __syncthreads(); // the product has been read
#pragma unroll
        for (int k = 0; k < kSums; ++k)
            *(__attribute__((address_space(3))) float *)(uintptr_t)(lds0 + (uint32_t)(k * SH::kThreads + tid) * 4u) = sums[k];
        __syncthreads();
        for (int t = tid; t < LR * kSums; t += SH::kThreads) {
            const int k = t / LR, o = t % LR, oc = col0 + o * 8;
            if (oc < a.N) {
                float v = 0.0f;
                for (int i = 0; i < RP; ++i)
                    v += *(const __attribute__((address_space(3))) float *)(uintptr_t)(lds0 + (uint32_t)(k * SH::kThreads + i * LR + o) * 4u);
                const int32_t g = oc / a.dg;
                const int64_t row = (int64_t)g * a.partial_rows + (int64_t)(a.tile0 + tm) * (a.dg / 8) + (oc - g * a.dg) / 8;
                a.partial[row * kSums + k] = v;
            }
        }
    }
}

// --------------------------------------------------------------------------
// host side
// --------------------------------------------------------------------------
using Kernel = void (*)(const Args);

// us of a call: once + rounds (round + T (stage + fill share)), T = K / 64 and share of the compute units that a round gives a tile
// on average (the more do, the slower the loads and the clock).  Two workgroups on a unit: a round of one each and one of two.
struct Variant {
    int32_t BM, BN, threads, per_cu;
    size_t lds;
    Kernel kernel[4]; // W [N, K]; with F; W [K, N]; with F's backward pass or NULL
    double once, round, stage, fill, round2, stage2;
};

template <class SH> static constexpr Kernel backward_kernel()
{
    // not the two largest tiles: one leaves in parts, and the other was never the estimate's choice at a size of a block that
    // product_backward_pays takes
    if constexpr (SH::kParts == 1 && SH::TM * SH::TN < 32)
        return product_kernel<SH, true, kBackward>;
    else
        return nullptr;
}

template <class SH> static constexpr Variant variant(double once, double round, double stage, double fill, double round2 = 0, double stage2 = 0)
{
    return Variant{SH::BM, SH::BN, SH::kThreads, SH::PER, SH::kLds,
                   {product_kernel<SH, false, kPlain>, product_kernel<SH, false, kRational>, product_kernel<SH, true, kPlain>,
                    backward_kernel<SH>()},
                   once, round, stage, fill, round2, stage2};
}

// Of fourteen tiles these eight together lose 1 % in the mean to the best of all at 154 measured sizes (fourteen pairs N, K of 192 ..
// 3072 and 256 .. 3072, 197 - 50,432 rows).  The figures are least squares over the same sizes (residuals 4 - 8 %); the tile that the
// estimate takes is 1.7 % slower than the best of all fourteen in the mean, 18 % at most.  Large tiles move less through the L2 and
// LDS for each product, small ones fill the chip:
//   320 x 256 / 256 x 256 / 224 x 192 / 160 x 192 / 160 x 128 / two of 160 x 128 / 96 x 128 / 64 x 64, us
//   25,216 x  384 -> 1536  42 / 50 / 57 / 50 / 53 / 43 / 60 / 68
//   25,216 x 1536 ->  384  44 / 37 / 33 / 40 / 37 / 32 / 47 / 49
//    9,456 x  768 -> 3072  54 / 48 / 59 / 64 / 72 / 54 / 84 / 88
//    6,304 x 3072 ->  768  71 / 59 / 40 / 32 / 30 / 42 / 41 / 48
//    3,152 x 3072 ->  768  70 / 58 / 38 / 30 / 24 / 37 / 20 / 30
//      788 x 1536 ->  384  38 / 31 / 21 / 17 / 12 / 18 / 9 / 7
static const Variant kVariants[] = {
    variant<Shape<10, 4, 2, 4, 2, 0>>(0.22, 8.07, 1.183, 0.679), variant<Shape<8, 4, 2, 4, 2, 0>>(-0.39, 7.27, 0.959, 0.567),
    variant<Shape<7, 3, 2, 4, 3, 4>>(0.45, 6.37, 0.558, 0.438), variant<Shape<5, 3, 2, 4, 3, 4>>(0.75, 5.09, 0.418, 0.333),
    variant<Shape<5, 2, 2, 4, 4, 4>>(1.01, 3.72, 0.297, 0.281), variant<Shape<5, 4, 2, 2, 2, 0, 2>>(1.89, 2.36, 0.612, 0, 4.15, 1.067),
    variant<Shape<3, 2, 2, 4, 4, 4>>(1.74, 2.34, 0.211, 0.199), variant<Shape<2, 2, 2, 2, 4, 4>>(2.95, 0.66, 0.129, 0.047)};

static int64_t tiles_of(const Variant &v, int64_t rows, int32_t N) { return (rows + v.BM - 1) / v.BM * ((N + v.BN - 1) / v.BN); }

static double estimate_us(const Variant &v, int64_t rows, int32_t K, int32_t N, Then then)
{
    // F of a tile: 6 us at 320 x 256, its backward pass 17.5
    const double T = K / 64, f = (then == kRational ? 6.0 : then == kBackward ? 17.5 : 0.0) * v.BM * v.BN / 81920;
    const int64_t tiles = tiles_of(v, rows, N), per_xcd = (tiles + 7) / 8, rounds = (per_xcd + 31) / 32;
    if (v.per_cu == 2)
        return v.once + (double)(rounds % 2) * (v.round + v.stage * T + f) + (double)(rounds / 2) * (v.round2 + v.stage2 * T + f);
    return v.once + (double)rounds * (v.round + T * (v.stage + v.fill * ((double)tiles / ((double)rounds * 256))) + f);
}

static const Variant *best_tile(int64_t rows, int32_t K, int32_t N, Then then, double *us)
{
    const Variant *best = nullptr;
    for (const Variant &v : kVariants) {
        if (then == kBackward && !v.kernel[3])
            continue;
        const double t = estimate_us(v, rows, K, N, then);
        if (!best || t < *us) {
            best = &v;
            *us = t;
        }
    }
    return best;
}

// The launches of a call: all rows in one tile, or, where a last round would be nearly empty, whole rounds of one and the rows that are
// left in another (12,593 x 2048 -> 2048: 105 us in one tile, 92 as 10,240 rows in 320 x 256
// and 2,353 in a small one; 30,000 x 384 -> 1536 48.8 and 40.2; 9,456 x 768 -> 3072 54 and 49).
struct Plan {
    const Variant *first, *second;
    int64_t first_rows; // all where there is no second
    double us;
};

static Plan make_plan(int64_t rows, int32_t K, int32_t N, Then then)
{
    Plan best{nullptr, nullptr, rows, 0};
    best.first = best_tile(rows, K, N, then, &best.us);
    for (const Variant &v : kVariants) {
        if (then == kBackward && !v.kernel[3])
            continue;
        const int64_t tiles_n = (N + v.BN - 1) / v.BN, blocks = (rows + v.BM - 1) / v.BM, at_once = 256 * (int64_t)v.per_cu;
        const int64_t rounds = blocks * tiles_n / at_once; // whole ones
        const int64_t take = rounds * at_once / tiles_n;   // row blocks in them
        if (rounds == 0 || take == 0 || take >= blocks)
            continue;
        Plan p{&v, nullptr, take * v.BM, 0};
        p.second = best_tile(rows - p.first_rows, K, N, then, &p.us);
        p.us += estimate_us(v, p.first_rows, K, N, then) + 1.0;
        if (p.us < best.us)
            best = p;
    }
    return best;
}

// 16-byte pieces of rows, lane offsets of 32 bits, tiles counted in 31.
static bool supported(int64_t rows, int32_t K, int32_t N)
{
    return rows >= 0 && rows <= (int64_t)1 << 30 && K > 0 && K % 64 == 0 && K <= 1 << 20 && N > 0 && N % 8 == 0 && N <= 1 << 20 &&
           (rows + 63) / 64 * ((N + 63) / 64) < INT32_MAX / 16;
}

static bool allow_lds(const Variant &v, int which)
{
    static std::mutex mu;
    static bool done[64][sizeof(kVariants) / sizeof(kVariants[0])][4];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64)
        return false;
    std::lock_guard<std::mutex> lock(mu);
    bool &is = done[dev][&v - kVariants][which];
    if (!is)
        is = hipFuncSetAttribute(reinterpret_cast<const void *>(v.kernel[which]), hipFuncAttributeMaxDynamicSharedMemorySize,
                                 (int)v.lds) == hipSuccess;
    return is;
}

static int32_t row_tiles(const Plan &plan, int64_t rows)
{
    const int64_t one = (plan.first_rows + plan.first->BM - 1) / plan.first->BM;
    return (int32_t)(plan.second ? one + (rows - plan.first_rows + plan.second->BM - 1) / plan.second->BM : one);
}

static grkan_status_t launch(const Plan &plan, Args a, int64_t rows, bool transposed, Then then, hipStream_t stream)
{
    const int which = then == kBackward ? 3 : transposed ? 2 : then == kRational ? 1 : 0;
    const Args all = a;
    for (int part = 0; part < (plan.second ? 2 : 1); ++part) {
        const Variant &v = part ? *plan.second : *plan.first;
        const size_t row0 = part ? (size_t)plan.first_rows : 0;
        a.x = all.x + row0 * (size_t)a.K * 2u;
        a.out = all.out + row0 * (size_t)a.N * 2u;
        a.fx = all.fx ? all.fx + row0 * (size_t)a.N * 2u : nullptr;
        a.tile0 = part ? (int32_t)((plan.first_rows + plan.first->BM - 1) / plan.first->BM) : 0;
        a.M = part ? rows - plan.first_rows : plan.first_rows;
        a.tiles_n = (a.N + v.BN - 1) / v.BN;
        a.tiles = (int32_t)tiles_of(v, a.M, a.N);
        a.per_xcd = (a.tiles + 7) / 8;
        if (!allow_lds(v, which))
            return GRKAN_ERR_LAUNCH;
        void *args[] = {&a};
        if (hipLaunchKernel(reinterpret_cast<const void *>(v.kernel[which]), dim3((unsigned)a.per_xcd * 8u), dim3((unsigned)v.threads), args,
                            v.lds, stream) != hipSuccess)
            return GRKAN_ERR_LAUNCH;
    }
    return GRKAN_OK;
}

} // namespace product

// Whether the backward pass of F runs in the product that makes its upstream gradient: that is then not written and read again,
// and a launch less, but the multiplying wavefronts wait for it.  Whole training blocks, us with F in a launch of its own / here, by
// elements of dx (rows x N):
//   0.6 - 3 M  192 138 / 136, 384 140 / 134, 512 162.5 / 158, 768 179 / 175     4.8 M  192 147 / 143.5, 384 175.5 / 171.5, 768 269 / 264
//   8 - 10 M   192 239 / 236, 384 290.5 / 290.5, 640 350 / 345, 768 446 / 439.5  13 - 19 M  384 546 / 551, 512 443 / 462, 640 656 / 647, 768 841 / 859
// These are four times as wide inside as out.  At 1 - 25 times (78 blocks up to the limit) inside is 0 - 5 % less, but for 256 -> 2048 .. 6400
// at 25,216 rows, 1 - 3 % more.
bool product_backward_pays(int64_t rows, int32_t K, int32_t N, int32_t G)
{
    return product::supported(rows, K, N) && G > 0 && N % G == 0 && N / G % 8 == 0 && rows * N <= 10000000;
}

grkan_status_t product_backward(const void *dh, const void *W, const void *x, const CoefRows &coef, void *dx, void *dA, void *dB,
                                grkan_alloc_t alloc, void *alloc_context, int64_t rows, int32_t K, int32_t N, int32_t G, CoefSums *later,
                                hipStream_t stream)
{
    if (!product::supported(rows, K, N) || rows == 0 || G <= 0 || N % G != 0 || N / G % 8 != 0)
        return GRKAN_ERR_UNSUPPORTED;
    if (!dh || !W || !x || !dx || !coef.A || !coef.B || !dA || !dB)
        return GRKAN_ERR_NULL;
    auto address = [](const void *p) { return reinterpret_cast<uintptr_t>(p); };
    if ((address(dh) | address(W) | address(x) | address(dx)) % 16 != 0 ||
        (address(coef.A) | address(coef.B) | address(dA) | address(dB)) % 2 != 0)
        return GRKAN_ERR_ALIGN;
    const product::Plan plan = product::make_plan(rows, K, N, product::kBackward);
    product::Args a = {};
    a.x = static_cast<const char *>(dh);
    a.W = static_cast<const char *>(W);
    a.out = static_cast<char *>(dx);
    a.coef = coef;
    a.fx = static_cast<const char *>(x);
    a.N = N;
    a.K = K;
    a.dg = N / G;
    const int64_t per_group = (int64_t)product::row_tiles(plan, rows) * (a.dg / 8);
    if (per_group > INT32_MAX)
        return GRKAN_ERR_UNSUPPORTED;
    a.partial_rows = (int32_t)per_group;
    a.partial = static_cast<float *>(alloc((size_t)G * (size_t)per_group * product::kSums * sizeof(float), alloc_context));
    if (!a.partial)
        return GRKAN_ERR_WORKSPACE;
    *later = CoefSums{a.partial, a.partial_rows, coef, dA, dB, G};
    return product::launch(plan, a, rows, true, product::kBackward, stream);
}

} // namespace grkan

using namespace grkan;

extern "C" int32_t grkan_product_supported(int64_t rows, int32_t K, int32_t N) { return product::supported(rows, K, N); }

extern "C" double grkan_product_estimate_us(int64_t rows, int32_t K, int32_t N, int32_t rational)
{
    if (rows <= 0 || !product::supported(rows, K, N))
        return 0;
    return product::make_plan(rows, K, N, rational ? product::kRational : product::kPlain).us;
}

extern "C" grkan_status_t grkan_product_tile(int64_t rows, int32_t K, int32_t N, int32_t rational, int32_t *tile_rows, int32_t *tile_channels,
                                             int32_t *per_unit, int64_t *rows_in_it)
{
    if (!tile_rows || !tile_channels || !per_unit || !rows_in_it)
        return GRKAN_ERR_NULL;
    if (rows <= 0 || !product::supported(rows, K, N))
        return GRKAN_ERR_UNSUPPORTED;
    const product::Plan plan =
        product::make_plan(rows, K, N, rational == 2 ? product::kBackward : rational ? product::kRational : product::kPlain);
    *tile_rows = plan.first->BM;
    *tile_channels = plan.first->BN;
    *per_unit = plan.first->per_cu;
    *rows_in_it = plan.first_rows;
    return GRKAN_OK;
}

extern "C" grkan_status_t grkan_product(const void *x, const void *W, const void *bias, void *out, int64_t rows, int32_t K, int32_t N,
                                        int32_t transposed, const void *A, const void *B, int32_t G, int32_t shared_numerator,
                                        void *hip_stream)
{
    if (rows < 0 || K <= 0 || N <= 0)
        return GRKAN_ERR_SHAPE;
    const bool rational = A != nullptr || B != nullptr;
    if (rational && (G <= 0 || N % G != 0))
        return GRKAN_ERR_SHAPE;
    if (!product::supported(rows, K, N) || (rational && (transposed || N / G % 8 != 0)))
        return GRKAN_ERR_UNSUPPORTED;
    if ((rows > 0 && (!x || !W || !out)) || (rational && (!A || !B)))
        return GRKAN_ERR_NULL;
    auto address = [](const void *p) { return reinterpret_cast<uintptr_t>(p); };
    if ((address(x) | address(W) | address(out)) % 16 != 0 || address(bias) % 8 != 0 || (address(A) | address(B)) % 2 != 0)
        return GRKAN_ERR_ALIGN;
    if (rows == 0)
        return GRKAN_OK;
    const product::Then then = rational ? product::kRational : product::kPlain;
    product::Args a = {};
    a.x = static_cast<const char *>(x);
    a.W = static_cast<const char *>(W);
    a.bias = static_cast<const char *>(bias);
    a.out = static_cast<char *>(out);
    a.coef = CoefRows{A, B, shared_numerator ? 0 : product::kM + 1, 1};
    a.N = N;
    a.K = K;
    a.dg = rational ? N / G : N;
    return product::launch(product::make_plan(rows, K, N, then), a, rows, transposed != 0, then, static_cast<hipStream_t>(hip_stream));
}
