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
//
//   * Both operands have the contraction as their slow dimension.  Stages of 64 rows come to LDS as they lie
//     in memory (LDS-direct loads of whole 384-byte row pieces, three buffers, two stages ahead, one
//     barrier per stage) and are transposed on the way into the matrix cores by ds_read_b64_tr_b16, which
//     hands lane (i, g) of a wavefront the rows 4 g .. 4 g + 3 of column i.  The rows of a 32-row step are
//     numbered alike for both operands, which is all a contraction needs.
//   * 32-byte column pairs of a row are rotated by half the row number, so that the 16 rows a transposing
//     read touches fall into different banks (rows are 384 bytes = 1.5 bank sweeps apart).
//   * Eight wavefronts, two per SIMD: two halves of the 64 rows x four 96 x 96 quadrants.  With 96 x 96 a
//     wavefront reads 12 KB for 36 matrix instructions; transposing reads run at about 110 B per clock
//     and CU, so that a 96 x 48 share of the tile would be bound by them.
//   * The column sums for dbias ride along as matrix products with a constant fragment of ones, shared out
//     over the workgroups and wavefronts that see the same columns of dOut: 1 % more matrix instructions
//     in place of a pass over dOut.
//
// Measured on one MI355X, both gradients, 25,216 rows, against the library's product + column sum (us):
//   384 x 1536: 46 against 171     192 x 768: 28 against 189     768 x 3072: 124 against 270     3072 x 768: 125 against 305
// What bounds it: at 384 x 1536 (25 stages for each workgroup) the matrix cores are busy 37 %
// of the time and the wavefronts wait 40 % of theirs: the transposing reads (98 KB per stage at 109 B per clock and CU:
// 900 of the stage's 1152 matrix-instruction clocks) and the loads into LDS (49 KB per stage at about 53) go on beside
// the matrix instructions, filling the pipeline and the partial tile's way out do not; 7 - 9 of the 46 us are the second
// kernel, which reads the 37 MB of partial tiles.  No bank conflicts, and both operands are read from memory once.
#include <hip/hip_runtime.h>

#include <mutex>

#include "../../include/grkan.h"

namespace grkan {
namespace wgrad {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef const __attribute__((address_space(1))) char *gcptr_t;
typedef __attribute__((address_space(3))) char *lptr_t;

constexpr int kTile = 192;                       // rows and columns of a tile of dW
constexpr int kRows = 64;                        // rows of dOut and Y per stage
constexpr int kPairs = kTile / 16;               // 32-byte column pairs per row
constexpr int kRowB = kTile * 2;                 // bytes of a row piece
constexpr uint32_t kOperand = kRows * kRowB;     // 24576: one operand of one stage
constexpr uint32_t kStage = 2 * kOperand;
constexpr int kBuffers = 3;
constexpr uint32_t kLds = kBuffers * kStage;     // 147456
constexpr int kLoads = (int)(kOperand / 1024 / 8); // LDS-direct loads per wavefront, operand and stage: 3

struct Args {
    const char *dout; // bfloat16 [rows, Do]
    const char *y;    // bfloat16 [rows, Di]
    float *part;      // [splits][Do][Di]
    float *bpart;     // [splits][shares][2][Do] or NULL
    int64_t rows;
    int32_t Do, Di;
    int32_t tiles_i;  // ceil(Di / 192)
    int32_t tiles;    // ceil(Do / 192) * tiles_i
    int32_t splits;
    int32_t per_xcd;  // ceil(tiles * splits / 8)
};

__device__ __forceinline__ uint64_t uniform_u64(uint64_t v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// LDS-direct load: 16 bytes per lane from "uniform base + lane offset" to LDS bytes lds_at + 16 lane ..
// In assembly because the compiler, seeing such a load in flight, waits for all of them in front of every
// transposing LDS read (the two would be 1,500 clocks of memory latency per stage); they are waited for by
// count before the stage's barrier instead.  The instruction writes no registers.  s_nop: m0 and a base
// formed by a vector instruction need up to five wait states.
__device__ __forceinline__ void load_to_lds(uint64_t base, uint32_t lane_off, uint32_t lds_at)
{
    asm volatile("s_nop 4\n\tglobal_load_lds_dwordx4 %1, %2" : : "{m0}"(lds_at), "v"(lane_off), "s"(base) : "memory");
}

__device__ __forceinline__ s16x4 read_transposed(uint32_t addr)
{
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(uintptr_t)addr);
}

// 16 columns x 32 rows of an operand: lane (i, g) gets column i, rows 4 g .. 4 g + 3 and 16 + 4 g .. 16 + 4 g + 3
__device__ __forceinline__ bf16x8 fragment(uint32_t addr)
{
    const s16x4 lo = read_transposed(addr);
    const s16x4 hi = read_transposed(addr + 16u * kRowB);
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

__global__ __launch_bounds__(512, 1) void grkan_linear_wgrad_kernel(const Args a)
{
    extern __shared__ __align__(16) char smem[];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lptr_t)smem;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);

    // workgroup -> (row range, tile): workgroups go round-robin over the 8 XCDs; each XCD takes a run of
    // consecutive (range, tile) pairs, so that the tiles of one range share its L2 copy of the rows
    const int32_t slot = (int32_t)blockIdx.x >> 3;
    const int32_t lin = ((int32_t)blockIdx.x & 7) * a.per_xcd + slot;
    if (lin >= a.tiles * a.splits)
        return;
    const int32_t split = __builtin_amdgcn_readfirstlane(lin / a.tiles);
    const int32_t tile = lin - split * a.tiles;
    const int32_t to = __builtin_amdgcn_readfirstlane(tile / a.tiles_i);
    const int32_t ti = tile - to * a.tiles_i;
    const int64_t n_stages = (a.rows + kRows - 1) / kRows;
    const int64_t s0 = n_stages * split / a.splits;
    const int32_t mine = (int32_t)(n_stages * (split + 1) / a.splits - s0);

    // ---- loader: 16-byte piece e = (3 wave + q) 64 + lane of an operand's stage sits at LDS byte 16 e: row e / 24,
    // slot e % 24, which holds column pair (slot / 2 - (row % 16) / 2) mod 12 of the row.  Pieces past the end of
    // a row repeat its last one (their products are not stored).
    const uint32_t ldo = (uint32_t)a.Do * 2u, ldi = (uint32_t)a.Di * 2u;
    uint32_t off_o[kLoads], off_i[kLoads];
    int row_of[kLoads];
#pragma unroll
    for (int q = 0; q < kLoads; ++q) {
        const uint32_t e = (uint32_t)(wave * kLoads + q) * 64u + (uint32_t)lane;
        const uint32_t row = e / (uint32_t)(2 * kPairs);
        const uint32_t s = e - row * (uint32_t)(2 * kPairs);
        const uint32_t p = ((s >> 1) + (uint32_t)kPairs - ((row & 15u) >> 1)) % (uint32_t)kPairs;
        const uint32_t col = (2u * p + (s & 1u)) * 16u;
        const uint32_t co = (uint32_t)to * kRowB + col, ci = (uint32_t)ti * kRowB + col;
        row_of[q] = (int)row;
        off_o[q] = row * ldo + (co < ldo ? co : ldo - 16u);
        off_i[q] = row * ldi + (ci < ldi ? ci : ldi - 16u);
    }
    auto fetch = [&](int32_t t) {
        const uint64_t r0 = (uint64_t)(s0 + t) * kRows;
        const uint64_t po = uniform_u64(reinterpret_cast<uint64_t>(a.dout) + r0 * ldo);
        const uint64_t pi = uniform_u64(reinterpret_cast<uint64_t>(a.y) + r0 * ldi);
        const uint32_t buf = (uint32_t)(t % kBuffers) * kStage + (uint32_t)(wave * kLoads) * 1024u;
        if (r0 + kRows <= (uint64_t)a.rows) {
#pragma unroll
            for (int q = 0; q < kLoads; ++q) {
                load_to_lds(po, off_o[q], lds0 + buf + q * 1024u);
                load_to_lds(pi, off_i[q], lds0 + buf + kOperand + q * 1024u);
            }
        } else {
            // the last, partial stage goes through registers: rows past the end are zeros in both operands
            const int valid = (int)(a.rows - (int64_t)r0);
#pragma unroll
            for (int q = 0; q < kLoads; ++q) {
                u32x4 vo = u32x4{0u, 0u, 0u, 0u}, vi = vo;
                if (row_of[q] < valid) {
                    vo = *(const __attribute__((address_space(1))) u32x4 *)((gcptr_t)po + off_o[q]);
                    vi = *(const __attribute__((address_space(1))) u32x4 *)((gcptr_t)pi + off_i[q]);
                }
                const uint32_t at = lds0 + buf + q * 1024u + (uint32_t)lane * 16u;
                *(__attribute__((address_space(3))) u32x4 *)(uintptr_t)at = vo;
                *(__attribute__((address_space(3))) u32x4 *)(uintptr_t)(at + kOperand) = vi;
            }
        }
    };

    // ---- wavefront: rows 32 kh .. of a stage, quadrant (o half oh, i half ih).  Y is the row operand of the
    // matrix instruction, so that a lane ends up with four consecutive i of one o.
    const int kh = wave >> 2, oh = (wave >> 1) & 1, ih = wave & 1;
    const uint32_t r15 = (uint32_t)(lane >> 4) * 4u + (uint32_t)(lane & 15) / 4u; // row (mod 16) a lane addresses
    const uint32_t lane_at = lds0 + ((uint32_t)kh * 32u + r15) * kRowB + (uint32_t)(lane & 3) * 8u;
    uint32_t at_i[6], at_o[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        at_i[k] = lane_at + kOperand + (((uint32_t)(ih * 6 + k) + (r15 >> 1)) % (uint32_t)kPairs) * 32u;
        at_o[k] = lane_at + (((uint32_t)(oh * 6 + k) + (r15 >> 1)) % (uint32_t)kPairs) * 32u;
    }

    f32x4 acc[6][6], bacc[6]; // [i sub-tile][o sub-tile]
#pragma unroll
    for (int n = 0; n < 6; ++n) {
        bacc[n] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int m = 0; m < 6; ++m)
            acc[m][n] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
    const short one = 0x3f80;
    const bf16x8 ones = __builtin_bit_cast(bf16x8, s16x8{one, one, one, one, one, one, one, one});
    const int32_t shares = 2 * a.tiles_i;
    const int32_t share = 2 * ti + ih;
    int32_t turn = (int32_t)(s0 % shares); // of the stage

    if (mine > 0)
        fetch(0);
    if (mine > 1)
        fetch(1);
    for (int32_t t = 0; t < mine; ++t) {
        // this wavefront's part of stage t has landed (the loads of stage t + 1 may be in flight; the stage
        // before the last waits for everything, because the last may have gone through registers), and so have its
        // reads of the buffer that is refilled next, wherever the compiler put the instructions that use them
        if (t + 2 < mine)
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(2 * kLoads) : "memory");
        else
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (t + 2 < mine)
            fetch(t + 2); // into the buffer read in step t - 1, which every wavefront has left
        const uint32_t buf = (uint32_t)(t % kBuffers) * kStage;
        bf16x8 fo[6], fi[6];
#pragma unroll
        for (int k = 0; k < 6; ++k)
            fo[k] = fragment(at_o[k] + buf);
#pragma unroll
        for (int k = 0; k < 6; ++k)
            fi[k] = fragment(at_i[k] + buf);
#pragma unroll
        for (int m = 0; m < 6; ++m)
#pragma unroll
            for (int n = 0; n < 6; ++n)
                acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fi[m], fo[n], acc[m][n], 0, 0, 0);
        const bool my_turn = turn == share;
        turn = turn + 1 == shares ? 0 : turn + 1;
        if (a.bpart && my_turn) {
#pragma unroll
            for (int n = 0; n < 6; ++n)
                bacc[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, fo[n], bacc[n], 0, 0, 0);
        }
    }

    // ---- the two row halves are added through LDS, then the partial tile goes to memory
    __syncthreads();
    const uint32_t quad = lds0 + (uint32_t)(wave & 3) * (36u * 1024u) + (uint32_t)lane * 16u;
    if (kh == 1) {
#pragma unroll
        for (int m = 0; m < 6; ++m)
#pragma unroll
            for (int n = 0; n < 6; ++n)
                *(__attribute__((address_space(3))) f32x4 *)(uintptr_t)(quad + (uint32_t)(m * 6 + n) * 1024u) = acc[m][n];
    }
    __syncthreads();
    const int32_t o_lane = to * kTile + oh * 96 + (lane & 15);
    const int32_t i_lane = ti * kTile + ih * 96 + (lane >> 4) * 4;
    if (kh == 0) {
#pragma unroll
        for (int n = 0; n < 6; ++n) {
            const int32_t o = o_lane + n * 16;
            if (o >= a.Do)
                continue;
            float *const row = a.part + ((int64_t)split * a.Do + o) * a.Di;
#pragma unroll
            for (int m = 0; m < 6; ++m) {
                const int32_t i = i_lane + m * 16;
                if (i < a.Di)
                    *(f32x4 *)(row + i) = acc[m][n] + *(const __attribute__((address_space(3))) f32x4 *)(uintptr_t)(
                                                          quad + (uint32_t)(m * 6 + n) * 1024u);
            }
        }
    }
    if (a.bpart && lane < 16) {
#pragma unroll
        for (int n = 0; n < 6; ++n) {
            const int32_t o = o_lane + n * 16;
            if (o < a.Do)
                a.bpart[(((int64_t)split * shares + share) * 2 + kh) * a.Do + o] = bacc[n][0];
        }
    }
}

// Adds the partials in range order.  Workgroups below `main_blocks`: four consecutive elements of dW per
// lane; the others: 16 columns of dbias each, 16 lanes per column that add every 16th row, then in lane order.
__global__ __launch_bounds__(256) void grkan_linear_wgrad_sum_kernel(const float *__restrict__ part,
                                                                     const float *__restrict__ bpart,
                                                                     char *__restrict__ dW, char *__restrict__ dbias,
                                                                     int64_t elems, int32_t Do, int32_t splits,
                                                                     int32_t brows, int32_t main_blocks)
{
    const int tid = threadIdx.x;
    if ((int32_t)blockIdx.x < main_blocks) {
        const int64_t e = ((int64_t)blockIdx.x * 256 + tid) * 4;
        if (e >= elems)
            return;
        f32x4 v = *(const f32x4 *)(part + e);
#pragma unroll 8
        for (int32_t s = 1; s < splits; ++s)
            v += *(const f32x4 *)(part + (int64_t)s * elems + e);
        f32x2 lo, hi;
        lo[0] = v[0], lo[1] = v[1], hi[0] = v[2], hi[1] = v[3];
        u32x2 r;
        r[0] = __builtin_bit_cast(uint32_t, __builtin_convertvector(lo, bf16x2));
        r[1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(hi, bf16x2));
        *(u32x2 *)(dW + e * 2) = r;
    } else {
        __shared__ float part_sum[16][17];
        const int c = tid & 15, l = tid >> 4;
        const int32_t o = ((int32_t)blockIdx.x - main_blocks) * 16 + c;
        float s = 0.0f;
        if (o < Do) {
#pragma unroll 4
            for (int32_t r = l; r < brows; r += 16)
                s += bpart[(int64_t)r * Do + o];
        }
        part_sum[l][c] = s;
        __syncthreads();
        if (tid < 16 && o < Do) {
            float t = 0.0f;
            for (int k = 0; k < 16; ++k)
                t += part_sum[k][tid];
            *(uint16_t *)(dbias + (int64_t)o * 2) = __builtin_bit_cast(uint16_t, static_cast<__bf16>(t));
        }
    }
}

// --------------------------------------------------------------------------
// host side
// --------------------------------------------------------------------------
struct Plan {
    int32_t tiles_o, tiles_i, splits;
    size_t part_bytes, bias_bytes;
};

static grkan_status_t make_plan(int64_t rows, int32_t D_in, int32_t D_out, Plan *pl)
{
    if (rows < 0 || D_in <= 0 || D_out <= 0)
        return GRKAN_ERR_SHAPE;
    // 16-byte pieces of rows; 32-bit lane offsets of 64 rows; row ranges counted in 31 bits
    if (D_in % 8 != 0 || D_out % 8 != 0 || D_in > (1 << 24) || D_out > (1 << 24) || rows > ((int64_t)1 << 36))
        return GRKAN_ERR_UNSUPPORTED;
    pl->tiles_o = (D_out + kTile - 1) / kTile;
    pl->tiles_i = (D_in + kTile - 1) / kTile;
    const int64_t tiles = (int64_t)pl->tiles_o * pl->tiles_i;
    const int64_t stages = (rows + kRows - 1) / kRows;
    // as many row ranges as fill the 256 compute units once (one workgroup each: 144 KB of LDS), each of four
    // stages at least: a shorter one would mostly fill and drain its pipeline and write its partial tile
    int64_t splits = 256 / tiles;
    if (splits > stages / 4)
        splits = stages / 4;
    if (splits < 1)
        splits = 1;
    if (tiles * splits > INT32_MAX / 16)
        return GRKAN_ERR_UNSUPPORTED;
    pl->splits = (int32_t)splits;
    pl->part_bytes = (size_t)splits * (size_t)D_out * (size_t)D_in * 4;
    pl->bias_bytes = (size_t)splits * (size_t)(4 * pl->tiles_i) * (size_t)D_out * 4;
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

} // namespace wgrad
} // namespace grkan

using namespace grkan::wgrad;

extern "C" size_t grkan_linear_wgrad_workspace_bytes(int64_t rows, int32_t D_in, int32_t D_out)
{
    Plan pl;
    if (make_plan(rows, D_in, D_out, &pl) != GRKAN_OK)
        return 0;
    return pl.part_bytes + pl.bias_bytes;
}

extern "C" grkan_status_t grkan_linear_wgrad(const void *dout, const void *y, void *dW, void *dbias, void *workspace,
                                             size_t workspace_bytes, int64_t rows, int32_t D_in, int32_t D_out,
                                             grkan_dtype_t io, void *hip_stream)
{
    if (io != GRKAN_BF16)
        return GRKAN_ERR_DTYPE;
    Plan pl;
    const grkan_status_t st = make_plan(rows, D_in, D_out, &pl);
    if (st != GRKAN_OK)
        return st;
    if (!dW || (rows > 0 && (!dout || !y)))
        return GRKAN_ERR_NULL;
    if ((reinterpret_cast<uintptr_t>(dout) | reinterpret_cast<uintptr_t>(y) | reinterpret_cast<uintptr_t>(dW)) % 16 != 0 ||
        reinterpret_cast<uintptr_t>(dbias) % 2 != 0)
        return GRKAN_ERR_ALIGN;
    if (!workspace || workspace_bytes < pl.part_bytes + pl.bias_bytes || reinterpret_cast<uintptr_t>(workspace) % 16 != 0)
        return GRKAN_ERR_WORKSPACE;
    if (!allow_lds())
        return GRKAN_ERR_LAUNCH;
    Args a;
    a.dout = static_cast<const char *>(dout);
    a.y = static_cast<const char *>(y);
    a.part = static_cast<float *>(workspace);
    a.bpart = dbias ? reinterpret_cast<float *>(static_cast<char *>(workspace) + pl.part_bytes) : nullptr;
    a.rows = rows;
    a.Do = D_out;
    a.Di = D_in;
    a.tiles_i = pl.tiles_i;
    a.tiles = pl.tiles_o * pl.tiles_i;
    a.splits = pl.splits;
    a.per_xcd = (a.tiles * a.splits + 7) / 8;
    void *args[] = {&a};
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    if (hipLaunchKernel(reinterpret_cast<const void *>(grkan_linear_wgrad_kernel), dim3((unsigned)a.per_xcd * 8u), dim3(512),
                        args, kLds, stream) != hipSuccess)
        return GRKAN_ERR_LAUNCH;
    const float *part = a.part, *bpart = a.bpart;
    char *w_arg = static_cast<char *>(dW), *b_arg = static_cast<char *>(dbias);
    int64_t elems = (int64_t)D_out * D_in;
    int32_t Do = D_out, splits = a.splits, brows = a.splits * 4 * pl.tiles_i;
    const int64_t blocks = (elems / 4 + 255) / 256;
    if (blocks + (D_out + 15) / 16 > INT32_MAX)
        return GRKAN_ERR_UNSUPPORTED;
    int32_t main_blocks = (int32_t)blocks;
    const unsigned grid = (unsigned)(main_blocks + (dbias ? (D_out + 15) / 16 : 0));
    void *args2[] = {&part, &bpart, &w_arg, &b_arg, &elems, &Do, &splits, &brows, &main_blocks};
    const hipError_t e = hipLaunchKernel(reinterpret_cast<const void *>(grkan_linear_wgrad_sum_kernel), dim3(grid), dim3(256),
                                         args2, 0, stream);
    return e == hipSuccess ? GRKAN_OK : GRKAN_ERR_LAUNCH;
}
