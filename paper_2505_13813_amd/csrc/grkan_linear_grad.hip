// Weight and bias gradient of the GR-KAN layer's product on gfx950 (MI355X):
//
//     dW[o, i] = sum_r dOut[r, o] Y[r, i]        dbias[o] = sum_r dOut[r, o]
//
// with Y = F(x) (FlashKAT paper, Eq. "GR_KAN"), bfloat16 in, float32 sums, bfloat16 out.
//
// The contraction runs over the rows (25,216 tokens at the paper's per-GPU batch) while the result is
// small (384 x 1536 for KAT-S), so the work is split over the rows: a workgroup owns a 192 x 192 tile of dW
// and one range of rows, and writes a float32 partial tile; a second kernel adds the partials in range
// order.  Nothing is atomic and every order is fixed by the sizes, so results are the same from run to run.
// A block's two products share one launch where both together still fill the chip (make_plan): the partial tiles that do are 38 MB in
// all, whatever the sizes, written and read once instead of twice.
//
//   * Both operands have the contraction as their slow dimension.  Stages of 32 rows come to LDS as they lie
//     in memory (LDS-direct loads of whole 384-byte row pieces, six buffers) and are transposed on the way into the matrix
//     cores by ds_read_b64_tr_b16, which hands lane (i, g) of a wavefront the rows 4 g .. 4 g + 3 of column i.  The rows of a
//     stage are numbered alike for both operands, which is all a contraction needs.
//   * 32-byte column pairs of a row are rotated by half the row number, so that the 16 rows a transposing
//     read touches fall into different banks (rows are 384 bytes = 1.5 bank sweeps apart).
//   * Eight wavefronts multiply, two per SIMD, 96 x 48 each.  (Four of 96 x 96 read a third less, but one per SIMD does
//     not issue its reads beside its own matrix instructions: 0.76 - 0.82 us per 64 rows against 0.71 without loads.)  One barrier
//     per stage, behind the first row of tiles; the next stage's operands are read between the matrix instructions, each
//     behind the last use of the registers it goes to.
//   * Four wavefronts load.  The column sums for dbias are matrix products with ones that they make meanwhile; tiles that see
//     the same columns of dOut take turns by the stage.  (Added up lane by lane they cost the whole kernel a tenth of its time.)
//
// Measured on one MI355X, both gradients of one product, 25,216 rows, against the library's product + column sum (us):
//   384 x 1536: 41 against 171     192 x 768: 27 against 189     768 x 3072: 108 against 270
// and of a block's two products, in two launches of eight wavefronts that loaded, read and multiplied in turn / in one of this:
//   384: 90 / 65     192: 57 / 33     512: 154 / 122     768: 266 / 220     768 at 3,152 rows: 67 / 42
// What bounds it: at 384 (50 times 64 rows for each workgroup) 64 rows take 0.53 - 0.59 us of matrix instructions (0.48 at 2.4
// GHz), 0.71 with the transposing reads, 0.82 with loads that hit the L2 and 0.9 - 1.0 with the rows from memory, where the
// loads alone take 0.55; the loads move 4 TB/s where they miss the last-level cache (row pieces of 384 bytes, which eight workgroups
// fetch next to each other).  The second kernel, which reads the partial tiles, takes 7 - 8 us, writing them about as much.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>

#include "grkan_plan.h"
#include "grkan_stage2.h"
#include "grkan_tile.h"

namespace grkan {
namespace wgrad {

using namespace tile;

constexpr int kTile = 192;                       // rows and columns of a tile of dW
constexpr int kRows = 32;                        // rows of dOut and Y per stage
constexpr int kPairs = kTile / 16;               // 32-byte column pairs per row
constexpr uint32_t kRowB = kTile * 2;            // bytes of a row piece
constexpr uint32_t kOperand = kRows * kRowB;     // 12288: one operand of one stage
constexpr uint32_t kStage = 2 * kOperand;
constexpr int kBuffers = 6;
constexpr uint32_t kLds = kBuffers * kStage;     // 147456
constexpr int kMul = 8, kLoaders = 4;            // wavefronts
constexpr int kThreads = 64 * (kMul + kLoaders);
constexpr int kLoads = (int)(kStage / 1024 / kLoaders); // LDS-direct loads per loading wavefront and stage: 6
constexpr int kO = 6, kI = 3;                    // 16 x 16 tiles of a wavefront: columns of dOut, of Y

struct Problem {
    const char *dout; // bfloat16 [rows, Do]
    const char *y;    // bfloat16 [rows, Di]
    float *part;      // [splits][Do][Di]
    float *bpart;     // [splits][tiles_i][Do] or NULL
    int32_t Do, Di;
    int32_t tiles_i;  // ceil(Di / 192)
    int32_t tiles;    // ceil(Do / 192) * tiles_i
};

struct Args {
    Problem p[2]; // one or two products over the same rows
    int64_t rows;
    int32_t tiles; // of both
    int32_t splits;
    int32_t per_xcd; // ceil(tiles * splits / 8)
};

// 16 columns x 32 rows of an operand: lane (i, g) gets column i, rows 4 g .. 4 g + 3 and 16 + 4 g .. 16 + 4 g + 3
__device__ __forceinline__ u32x4 fragment(uint32_t addr)
{
    const u32x2 lo = __builtin_bit_cast(u32x2, lds_read_transposed(addr));
    const u32x2 hi = __builtin_bit_cast(u32x2, lds_read_transposed(addr + 16u * kRowB));
    return u32x4{lo[0], lo[1], hi[0], hi[1]};
}

__global__ __launch_bounds__(kThreads, kThreads / 256) void grkan_linear_wgrad_kernel(const Args a)
{
    extern __shared__ __align__(16) char smem[];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);

    // workgroup -> (row range, tile): workgroups go round-robin over the 8 XCDs; each XCD takes a run of
    // consecutive (range, tile) pairs, so that the tiles of one range share its L2 copy of the rows
    const int32_t lin = ((int32_t)blockIdx.x & 7) * a.per_xcd + ((int32_t)blockIdx.x >> 3);
    if (lin >= a.tiles * a.splits)
        return;
    const int32_t split = __builtin_amdgcn_readfirstlane(lin / a.tiles);
    const int32_t both = lin - split * a.tiles;
    const bool second = both >= a.p[0].tiles;
    const Problem p = a.p[second ? 1 : 0];
    const int32_t tile = both - (second ? a.p[0].tiles : 0);
    const int32_t to = __builtin_amdgcn_readfirstlane(tile / p.tiles_i);
    const int32_t ti = tile - to * p.tiles_i;
    const int64_t n_stages = (a.rows + kRows - 1) / kRows;
    const int64_t s0 = n_stages * split / a.splits;
    const int32_t T = (int32_t)(n_stages * (split + 1) / a.splits - s0);
    auto advance = [&](uint32_t b) { return b + kStage == kBuffers * kStage ? 0u : b + kStage; };

    const uint32_t r15 = (uint32_t)(lane >> 4) * 4u + (uint32_t)(lane & 15) / 4u; // row (mod 16) a lane addresses
    const uint32_t lane_at = lds0 + r15 * kRowB + (uint32_t)(lane & 3) * 8u;

    // every wavefront passes T + 1 barriers in the branches
    if (wave >= kMul) {
        // ---- loads: 16-byte piece e of an operand's stage sits at LDS byte 16 e: row e / 24, slot e % 24, which holds column
        // pair (slot / 2 - (row % 16) / 2) mod 12 of the row.  Pieces past the end of a row repeat its last one (their
        // products are not stored).
        const int fw = wave - kMul;
        const uint32_t ldo = (uint32_t)p.Do * 2u, ldi = (uint32_t)p.Di * 2u;
        uint32_t off[kLoads];
#pragma unroll
        for (int q = 0; q < kLoads; ++q) {
            const int u = fw + q * kLoaders; // KB of the stage: below 24 dOut's, the others Y's (the same for all lanes and q)
            const bool iso = u < (int)(kOperand / 1024);
            const uint32_t e = (uint32_t)(iso ? u : u - (int)(kOperand / 1024)) * 64u + (uint32_t)lane;
            const uint32_t row = e / (uint32_t)(2 * kPairs), s = e - row * (uint32_t)(2 * kPairs);
            const uint32_t pair = ((s >> 1) + (uint32_t)kPairs - ((row & 15u) >> 1)) % (uint32_t)kPairs;
            const uint32_t ld = iso ? ldo : ldi, col = (uint32_t)(iso ? to : ti) * kRowB + (2u * pair + (s & 1u)) * 16u;
            off[q] = row * ld + (col < ld ? col : ld - 16u);
        }
        auto fetch = [&](int32_t t, uint32_t buf) {
            const uint64_t r0 = (uint64_t)(s0 + t) * kRows;
            const uint64_t po = uniform_u64(reinterpret_cast<uint64_t>(p.dout) + r0 * ldo);
            const uint64_t pi = uniform_u64(reinterpret_cast<uint64_t>(p.y) + r0 * ldi);
            if (r0 + kRows <= (uint64_t)a.rows) {
#pragma unroll
                for (int q = 0; q < kLoads; ++q) {
                    const uint32_t u = (uint32_t)(fw + q * kLoaders);
                    load_to_lds(q < kLoads / 2 ? po : pi, off[q], lds0 + buf + u * 1024u);
                }
            } else {
                // the last, partial stage goes through registers: rows past the end are zeros in both operands
                const uint32_t valid = (uint32_t)(a.rows - (int64_t)r0);
#pragma unroll
                for (int q = 0; q < kLoads; ++q) {
                    const uint32_t u = (uint32_t)(fw + q * kLoaders);
                    const uint32_t row = ((u % (kOperand / 1024u)) * 64u + (uint32_t)lane) / (uint32_t)(2 * kPairs);
                    u32x4 v = u32x4{0u, 0u, 0u, 0u};
                    if (row < valid)
                        v = gload16(q < kLoads / 2 ? po : pi, off[q]);
                    lds_write16(lds0 + buf + u * 1024u + (uint32_t)lane * 16u, v);
                }
            }
        };
        static_assert(kLoads % 2 == 0 && kOperand / 1024 % kLoaders == 0, "");

        // ---- column sums for dbias: products with ones, of three sub-tiles of 16 columns for each loading wavefront, in every stage that
        // is this tile's turn (the tiles that see the same columns of dOut take turns)
        uint32_t at_sum[3];
        f32x4 sums[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            at_sum[k] = lane_at + (((uint32_t)(fw * 3 + k) + (r15 >> 1)) % (uint32_t)kPairs) * 32u;
            sums[k] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        }
        const u32x4 ones = u32x4{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};

        static_for<0, kBuffers>([&](auto sc) {
            constexpr int s = decltype(sc)::value;
            if (s < T)
                fetch(s, (uint32_t)s * kStage);
        });
        // all but the last stages' loads have landed (near the end all: the last stage may have gone through registers)
        if (kBuffers < T)
            wait_loads<(kBuffers - 1) * kLoads>();
        else
            wait_loads<0>();
        asm volatile("s_barrier" ::: "memory");
        uint32_t buf = 0;
        int32_t turn = (int32_t)(s0 % p.tiles_i);
        for (int32_t t = 0; t < T; ++t) {
            if (p.bpart && turn == ti)
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    sums[k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ones),
                                                                      __builtin_bit_cast(bf16x8, fragment(at_sum[k] + buf)), sums[k], 0, 0, 0);
            turn = turn + 1 == p.tiles_i ? 0 : turn + 1;
            if (t + kBuffers < T)
                wait_loads<(kBuffers - 2) * kLoads>();
            else
                wait_loads<0>();
            asm volatile("s_barrier" ::: "memory");
            if (t + kBuffers < T)
                fetch(t + kBuffers, buf); // every wavefront has left it
            buf = advance(buf);
        }
        if (p.bpart && lane < 16)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const int32_t o = to * kTile + (fw * 3 + k) * 16 + lane;
                if (o < p.Do)
                    p.bpart[((int64_t)split * p.tiles_i + ti) * p.Do + o] = sums[k][0];
            }
        return;
    }

    // ---- multiplying wavefront: half oh of the tile's columns of dOut, quarter iq of Y's.  Y is the row operand of the matrix
    // instruction, so that a lane ends up with four consecutive i of one o.
    const int oh = wave >> 2, iq = wave & 3;
    uint32_t at_i[kI], at_o[kO];
#pragma unroll
    for (int k = 0; k < kI; ++k)
        at_i[k] = lane_at + kOperand + (((uint32_t)(iq * kI + k) + (r15 >> 1)) % (uint32_t)kPairs) * 32u;
#pragma unroll
    for (int k = 0; k < kO; ++k)
        at_o[k] = lane_at + (((uint32_t)(oh * kO + k) + (r15 >> 1)) % (uint32_t)kPairs) * 32u;
    f32x4 acc[kO][kI];
#pragma unroll
    for (int m = 0; m < kO; ++m)
#pragma unroll
        for (int n = 0; n < kI; ++n)
            acc[m][n] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

    // One stage: multiplies with x and wc while the next one's operands are read into x, each behind its own last use, and wn.
    // Behind the first row of tiles the barrier: every wavefront has its operands of this stage, and the next one has landed.
    // (Behind the last stage the next buffer is read too, and not used.)
    auto step = [&](auto hc, uint32_t from, u32x4(&x)[kO - 1], u32x4(&last)[2], u32x4(&wc)[kI], u32x4(&wn)[kI]) {
        constexpr int h = decltype(hc)::value; // which of `last`
        static_for<0, kO>([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            if constexpr (m == 1)
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            // reads between the matrix instructions: one after the other they would wait for the LDS with the matrix core idle
            // (wn's first, long before they are used; `last` has two sets of registers, so that it is read with the others)
            constexpr int n0 = m > 0 ? (2 * m - 2 < kI ? 2 * m - 2 : kI) : 0, n1 = 2 * m < kI ? 2 * m : kI;
            constexpr int kX = m > 0 ? 1 : 0, kOps = kX + (n1 - n0) + (m == kO - 1 ? 1 : 0);
            static_for<0, kI>([&](auto nc) {
                constexpr int n = decltype(nc)::value;
                static_for<0, kOps>([&](auto oc) {
                    constexpr int o = decltype(oc)::value;
                    if constexpr (o * kI / kOps == n) {
                        if constexpr (o < kX)
                            x[m - 1] = fragment(at_o[m - 1] + from);
                        else if constexpr (o < kX + n1 - n0)
                            wn[n0 + o - kX] = fragment(at_i[n0 + o - kX] + from);
                        else
                            last[1 - h] = fragment(at_o[kO - 1] + from);
                    }
                });
                fence_schedule();
                acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wc[n]), __builtin_bit_cast(bf16x8, m < kO - 1 ? x[m < kO - 1 ? m : 0] : last[h]),
                                                                    acc[m][n], 0, 0, 0);
                fence_schedule();
            });
        });
    };
    asm volatile("s_barrier" ::: "memory");
    {
        u32x4 x[kO - 1], last[2], wa[kI], wb[kI];
#pragma unroll
        for (int k = 0; k < kI; ++k)
            wa[k] = fragment(at_i[k]);
#pragma unroll
        for (int k = 0; k < kO - 1; ++k)
            x[k] = fragment(at_o[k]);
        last[0] = fragment(at_o[kO - 1]);
        uint32_t buf = 0;
        int32_t t = 0;
        for (; t + 1 < T; t += 2) {
            const uint32_t next = advance(buf), after = advance(next);
            step(std::integral_constant<int, 0>{}, next, x, last, wa, wb);
            step(std::integral_constant<int, 1>{}, after, x, last, wb, wa);
            buf = after;
        }
        if (t < T)
            step(std::integral_constant<int, 0>{}, advance(buf), x, last, wa, wb);
    }

    // ---- the partial tile goes to memory
    const int32_t o_lane = to * kTile + oh * 96 + (lane & 15);
    const int32_t i_lane = ti * kTile + iq * 48 + (lane >> 4) * 4;
#pragma unroll
    for (int m = 0; m < kO; ++m) {
        const int32_t o = o_lane + m * 16;
        if (o >= p.Do)
            continue;
        float *const row = p.part + ((int64_t)split * p.Do + o) * p.Di;
#pragma unroll
        for (int n = 0; n < kI; ++n) {
            const int32_t i = i_lane + n * 16;
            if (i < p.Di)
                *(f32x4 *)(row + i) = acc[m][n];
        }
    }
}

// Adds the partials in range order.  For each product first workgroups of four consecutive elements of dW per lane, then
// workgroups of 16 columns of dbias, 16 lanes per column that add every 16th row, then in lane order.  An MLP block's pass ends
// with it: the second stages of both rational functions' coefficient sums are workgroups of it too (COEF).
struct Sum {
    const float *part, *bpart;
    char *dW, *dbias;
    int64_t elems;
    int32_t Do, brows, splits;
    int32_t main_blocks, blocks;
};
struct SumArgs {
    Sum s[2];
    int32_t coef_blocks[2]; // COEF: in front of the others (their chains of sums are the longest)
    CoefSums coef[2];
};

template <bool COEF> __global__ __launch_bounds__(256) void grkan_linear_wgrad_sum_kernel(SumArgs a)
{
    const int tid = threadIdx.x;
    int32_t id = (int32_t)blockIdx.x;
    if constexpr (COEF) {
        if (id < a.coef_blocks[0] + a.coef_blocks[1]) {
            const bool last = id >= a.coef_blocks[0];
            const CoefSums c = a.coef[last ? 1 : 0];
            stage2_block<5, 4>(c.partial, c.rows_per_group, c.dA, c.dB, c.coef.a_stride == 0 ? c.G : 0, 1, id - (last ? a.coef_blocks[0] : 0));
            return;
        }
        id -= a.coef_blocks[0] + a.coef_blocks[1];
    }
    const bool second = id >= a.s[0].blocks;
    const Sum s = a.s[second ? 1 : 0];
    const int32_t block = id - (second ? a.s[0].blocks : 0);
    if (block < s.main_blocks) {
        const int64_t e = ((int64_t)block * 256 + tid) * 4;
        if (e >= s.elems)
            return;
        f32x4 v = *(const f32x4 *)(s.part + e);
#pragma unroll 8
        for (int32_t k = 1; k < s.splits; ++k)
            v += *(const f32x4 *)(s.part + (int64_t)k * s.elems + e);
        *(u32x2 *)(s.dW + e * 2) = u32x2{pack(v[0], v[1]), pack(v[2], v[3])};
    } else {
        __shared__ float part_sum[16][17];
        const int c = tid & 15, l = tid >> 4;
        const int32_t o = (block - s.main_blocks) * 16 + c;
        float v = 0.0f;
        if (o < s.Do) {
#pragma unroll 4
            for (int32_t r = l; r < s.brows; r += 16)
                v += s.bpart[(int64_t)r * s.Do + o];
        }
        part_sum[l][c] = v;
        __syncthreads();
        if (tid < 16 && o < s.Do) {
            float t = 0.0f;
            for (int k = 0; k < 16; ++k)
                t += part_sum[k][tid];
            *(uint16_t *)(s.dbias + (int64_t)o * 2) = __builtin_bit_cast(uint16_t, static_cast<__bf16>(t));
        }
    }
}

// --------------------------------------------------------------------------
// host side
// --------------------------------------------------------------------------
struct Size {
    int32_t D_in, D_out;
};

struct Plan {
    int32_t tiles_i[2], tiles[2], splits[2];
    bool together; // both products in one launch
    size_t part_bytes[2], bias_bytes[2];
    size_t bytes() const { return part_bytes[0] + bias_bytes[0] + part_bytes[1] + bias_bytes[1]; }
};

// n products (one or two) over the same rows.
static grkan_status_t make_plan(int64_t rows, const Size *size, int n, Plan *pl)
{
    *pl = Plan{};
    int64_t tiles = 0;
    for (int k = 0; k < n; ++k) {
        const int32_t D_in = size[k].D_in, D_out = size[k].D_out;
        if (rows < 0 || D_in <= 0 || D_out <= 0)
            return GRKAN_ERR_SHAPE;
        // 16-byte pieces of rows; 32-bit lane offsets of 32 rows
        if (D_in % 8 != 0 || D_out % 8 != 0 || D_in > (1 << 24) || D_out > (1 << 24) || rows > ((int64_t)1 << 36))
            return GRKAN_ERR_UNSUPPORTED;
        const int64_t tiles_i = (D_in + kTile - 1) / kTile, mine = (D_out + kTile - 1) / kTile * tiles_i;
        if (mine > INT32_MAX / 32)
            return GRKAN_ERR_UNSUPPORTED;
        pl->tiles_i[k] = (int32_t)tiles_i;
        pl->tiles[k] = (int32_t)mine;
        tiles += mine;
    }
    const int64_t stages = (rows + kRows - 1) / kRows;
    // as many row ranges as fill the 256 compute units once (one workgroup each: 144 KB of LDS), each of eight
    // stages at least: a shorter one would mostly fill and drain its pipeline and write its partial tile
    auto ranges = [&](int64_t of) { return std::max<int64_t>(1, std::min(256 / of, stages / 8)); };
    if (tiles * ranges(tiles) > INT32_MAX / 16)
        return GRKAN_ERR_UNSUPPORTED;
    // Two products: in one launch unless its workgroups walk kLaunch stages more than those of two launches one after the other: what
    // twice as many partial tiles, and filling the pipeline again, cost.  (256 / tiles rounds down: with 65 - 85 tiles for each product one
    // launch leaves up to 126 units without a workgroup that two launches of three ranges use; with 43 - 51 it has two ranges for both
    // against five for each.  MI355X, us of both gradients together / apart: 768, 3840 (80 tiles) at 6,304 rows 89 / 94, at 12,608 159 /
    // 160, at 25,216 350 / 290; 512, 4096 (66) 82 / 84, 150 / 141, 319 / 262; 768, 2048 (44) at 25,216 180 / 176, at 50,432 352 / 328; 512,
    // 2048 (33) 127 / 133, 254 / 245; 768, 3072 (64, as many stages in a row either way) 414 / 424.  Whole blocks at the line: 256, 6400
    // at 6,304 rows, 66 stages, 311 / 323, at 12,608, 131 stages, 595 / 565.)
    constexpr double kLaunch = 96;
    const double alone = (double)stages / (double)ranges(pl->tiles[0]) + (n == 2 ? (double)stages / (double)ranges(pl->tiles[1]) : 0);
    pl->together = n == 1 || (double)stages / (double)ranges(tiles) <= alone + kLaunch;
    for (int k = 0; k < n; ++k)
        pl->splits[k] = (int32_t)ranges(pl->together ? tiles : pl->tiles[k]);
    for (int k = 0; k < n; ++k)
        if (stages / pl->splits[k] >= INT32_MAX) // a range's stages are counted in 31 bits
            return GRKAN_ERR_UNSUPPORTED;
    for (int k = 0; k < n; ++k) {
        pl->part_bytes[k] = (size_t)pl->splits[k] * (size_t)size[k].D_out * (size_t)size[k].D_in * 4;
        pl->bias_bytes[k] = ((size_t)pl->splits[k] * (size_t)pl->tiles_i[k] * (size_t)size[k].D_out * 4 + 15) / 16 * 16;
    }
    return GRKAN_OK;
}

static bool allow_lds()
{
    static std::mutex mu;
    static bool done[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64)
        return false;
    std::lock_guard<std::mutex> lock(mu);
    if (!done[dev]) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(grkan_linear_wgrad_kernel),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLds) != hipSuccess)
            return false;
        done[dev] = true;
    }
    return true;
}

struct Operands {
    const void *dout, *y;
    void *dW, *dbias;
};

static grkan_status_t run(int64_t rows, const Size *size, const Operands *op, int n, void *workspace, size_t workspace_bytes,
                          hipStream_t stream, const CoefSums *coef = nullptr)
{
    Plan pl;
    const grkan_status_t st = make_plan(rows, size, n, &pl);
    if (st != GRKAN_OK)
        return st;
    auto address = [](const void *q) { return reinterpret_cast<uintptr_t>(q); };
    for (int k = 0; k < n; ++k)
        if (!op[k].dW || (rows > 0 && (!op[k].dout || !op[k].y)))
            return GRKAN_ERR_NULL;
    for (int k = 0; k < n; ++k)
        if ((address(op[k].dout) | address(op[k].y) | address(op[k].dW)) % 16 != 0 || address(op[k].dbias) % 2 != 0)
            return GRKAN_ERR_ALIGN;
    if (!workspace || workspace_bytes < pl.bytes() || address(workspace) % 16 != 0)
        return GRKAN_ERR_WORKSPACE;
    if (!allow_lds())
        return GRKAN_ERR_LAUNCH;
    Args a = {};
    SumArgs sum = {};
    a.rows = rows;
    a.splits = pl.splits[0];
    char *at = static_cast<char *>(workspace);
    int64_t blocks = 0;
    for (int k = 0; k < n; ++k) {
        Problem &p = a.p[k];
        p.dout = static_cast<const char *>(op[k].dout);
        p.y = static_cast<const char *>(op[k].y);
        p.part = reinterpret_cast<float *>(at);
        p.bpart = op[k].dbias ? reinterpret_cast<float *>(at + pl.part_bytes[k]) : nullptr;
        at += pl.part_bytes[k] + pl.bias_bytes[k];
        p.Do = size[k].D_out;
        p.Di = size[k].D_in;
        p.tiles_i = pl.tiles_i[k];
        p.tiles = pl.tiles[k];
        a.tiles += p.tiles;
        Sum &s = sum.s[k];
        s.part = p.part;
        s.bpart = p.bpart;
        s.dW = static_cast<char *>(op[k].dW);
        s.dbias = static_cast<char *>(op[k].dbias);
        s.elems = (int64_t)p.Do * p.Di;
        s.Do = p.Do;
        s.splits = pl.splits[k];
        s.brows = pl.splits[k] * p.tiles_i;
        const int64_t main_blocks = (s.elems / 4 + 255) / 256, mine = main_blocks + (s.dbias ? (p.Do + 15) / 16 : 0);
        blocks += mine;
        if (blocks > INT32_MAX)
            return GRKAN_ERR_UNSUPPORTED;
        s.main_blocks = (int32_t)main_blocks;
        s.blocks = (int32_t)mine;
    }
    for (int k = 0; k < (pl.together ? 1 : n); ++k) {
        Args of = a;
        if (!pl.together) {
            of.p[0] = a.p[k];
            of.p[1] = Problem{};
            of.tiles = of.p[0].tiles;
            of.splits = pl.splits[k];
        }
        of.per_xcd = (of.tiles * of.splits + 7) / 8;
        void *args[] = {&of};
        if (hipLaunchKernel(reinterpret_cast<const void *>(grkan_linear_wgrad_kernel), dim3((unsigned)of.per_xcd * 8u), dim3(kThreads),
                            args, kLds, stream) != hipSuccess)
            return GRKAN_ERR_LAUNCH;
    }
    void *args2[] = {&sum};
    if (coef)
        for (int k = 0; k < 2; ++k) {
            sum.coef[k] = coef[k];
            sum.coef_blocks[k] = coef[k].G + (coef[k].coef.a_stride == 0 ? 6 : 0);
            blocks += sum.coef_blocks[k];
        }
    const void *const kernel = coef ? reinterpret_cast<const void *>(grkan_linear_wgrad_sum_kernel<true>)
                                    : reinterpret_cast<const void *>(grkan_linear_wgrad_sum_kernel<false>);
    const hipError_t e = hipLaunchKernel(kernel, dim3((unsigned)blocks), dim3(256), args2, 0, stream);
    return e == hipSuccess ? GRKAN_OK : GRKAN_ERR_LAUNCH;
}

} // namespace wgrad

grkan_status_t wgrad_pair_and_sums(const grkan_block_bwd_t &b, grkan_alloc_t alloc, void *alloc_context, const CoefSums (&sums)[2],
                                   hipStream_t stream)
{
    const wgrad::Size size[2] = {{b.D, b.hidden}, {b.hidden, b.D}};
    const wgrad::Operands op[2] = {{b.dh, b.f1, b.dW1, b.db1}, {b.dout, b.f2, b.dW2, b.db2}};
    wgrad::Plan pl;
    const grkan_status_t st = wgrad::make_plan(b.rows, size, 2, &pl);
    if (st != GRKAN_OK)
        return st;
    void *const workspace = alloc(pl.bytes(), alloc_context);
    return wgrad::run(b.rows, size, op, 2, workspace, pl.bytes(), stream, sums);
}

} // namespace grkan

using namespace grkan::wgrad;

extern "C" size_t grkan_linear_wgrad_workspace_bytes(int64_t rows, int32_t D_in, int32_t D_out)
{
    const Size size{D_in, D_out};
    Plan pl;
    return make_plan(rows, &size, 1, &pl) == GRKAN_OK ? pl.bytes() : 0;
}

extern "C" grkan_status_t grkan_linear_wgrad(const void *dout, const void *y, void *dW, void *dbias, void *workspace,
                                             size_t workspace_bytes, int64_t rows, int32_t D_in, int32_t D_out,
                                             grkan_dtype_t io, void *hip_stream)
{
    if (io != GRKAN_BF16)
        return GRKAN_ERR_DTYPE;
    const Size size{D_in, D_out};
    const Operands op{dout, y, dW, dbias};
    return run(rows, &size, &op, 1, workspace, workspace_bytes, static_cast<hipStream_t>(hip_stream));
}

extern "C" size_t grkan_linear_wgrad_pair_workspace_bytes(int64_t rows, int32_t D_in1, int32_t D_out1, int32_t D_in2, int32_t D_out2)
{
    const Size size[2] = {{D_in1, D_out1}, {D_in2, D_out2}};
    Plan pl;
    return make_plan(rows, size, 2, &pl) == GRKAN_OK ? pl.bytes() : 0;
}

extern "C" grkan_status_t grkan_linear_wgrad_pair(const void *dout1, const void *y1, void *dW1, void *dbias1, int32_t D_in1, int32_t D_out1,
                                                  const void *dout2, const void *y2, void *dW2, void *dbias2, int32_t D_in2, int32_t D_out2,
                                                  void *workspace, size_t workspace_bytes, int64_t rows, void *hip_stream)
{
    const Size size[2] = {{D_in1, D_out1}, {D_in2, D_out2}};
    const Operands op[2] = {{dout1, y1, dW1, dbias1}, {dout2, y2, dW2, dbias2}};
    return run(rows, size, op, 2, workspace, workspace_bytes, static_cast<hipStream_t>(hip_stream));
}
