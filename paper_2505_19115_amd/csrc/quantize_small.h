// Device code of the quantizers for small tensors that quantize_small.hip and fused_small.hip share.
#pragma once
#include <type_traits>

#include "quantize_tile.h"

namespace nvfp4 {

// A tensor of a few workgroup tiles is quantized by a few waves, and what bounds it is one wave's serial chain: 64 elements per lane
// along one axis, then along the other, at the 8 cycles per instruction of a wave that is alone on its SIMD (dual SR+SR of 64 x 256:
// 11.7 us, here 3.6).  Here the two orientations are separate jobs of one launch and a lane holds as little as the blocks allow: 8 elements of a row,
// or one block of a column.  The draws of a column's block (one per row and 8 columns) are shared by the wave through LDS.
constexpr int SMALL_NT = 512;

// Column of its group of 64 that a lane holds.  bf16: two lanes 32 apart share a dword of two columns (below).
template <int DT>
__device__ __forceinline__ int lane_column(int lane) { return DT == NVFP4_BF16 ? 2 * (lane & 31) + (lane >> 5) : lane; }

// The lane's column of B rows from row0 on (whole groups of 64 columns or their first 8 n).  bf16 columns come two to a dword: the lower
// half of the wave loads the even rows, the upper half the odd ones, and each lane takes its 16 bits of both (one element per load, 64 x 256
// took 4.5 us instead of 3.6).  A lane without a column reads the tensor's first elements: with a predicate on each load the compiler may wait
// for them one by one (binary32 480 x 64 dual 6.1 us instead of 4.6).
template <int DT, int B>
__device__ __forceinline__ void load_column(const QuantArgs &P, int64_t row0, int64_t col0, int lane, bool live, float (&v)[B])
{
    if constexpr (DT == NVFP4_BF16) {
        const int odd = lane >> 5;
        const uint16_t *const p = reinterpret_cast<const uint16_t *>(P.x) + (live ? (row0 + odd) * P.ld + col0 + 2 * (lane & 31) : 0);
        const int64_t ld = live ? P.ld : 0;
        uint32_t w[B / 2];
#pragma unroll
        for (int r = 0; r < B / 2; ++r) w[r] = *reinterpret_cast<const uint32_t *>(p + 2 * r * ld);
#pragma unroll
        for (int r = 0; r < B / 2; ++r) {
            const auto both = __builtin_amdgcn_permlane32_swap(w[r], w[r], false, false);
            v[2 * r] = u2f(odd ? both[0] & 0xFFFF0000u : both[0] << 16);
            v[2 * r + 1] = u2f(odd ? both[1] & 0xFFFF0000u : both[1] << 16);
        }
    } else {
        const float *const p = reinterpret_cast<const float *>(P.x) + (live ? row0 * P.ld + col0 + lane : 0);
        const int64_t ld = live ? P.ld : 0;
#pragma unroll
        for (int r = 0; r < B; ++r) v[r] = p[r * ld];
    }
}

// The draws of B rows of a wave's 64 columns, 16 bits each: [row][column] (one draw per row and 8 columns, shared by the wave through LDS).
template <int B>
__device__ __forceinline__ void column_draws(const QuantArgs &P, int64_t row0, int64_t col0, int lane, uint16_t *mine)
{
#pragma unroll
    for (int i = 0; i < B / 8; ++i) {
        const int r = lane / 8 + 8 * i, cg = lane % 8;
        const u32x4 d = sr_draw(P.seed, (uint64_t)(row0 + r) * ((uint64_t)P.cols >> 3) + ((uint64_t)col0 >> 3) + cg);
        *reinterpret_cast<uint4 *>(mine + r * 64 + cg * 8) = make_uint4(d.x, d.y, d.z, d.w);
    }
    asm volatile("" ::: "memory");  // (other lanes of the wave read them below: the LDS keeps a wave's order, and so must the compiler)
}
template <int B>
__device__ __forceinline__ float column_max(const float (&v)[B])
{
    float a = 0.0f;
#pragma unroll
    for (int r = 0; r < B; ++r) a = fmaxf(a, fabsf(v[r]));
    return a;
}
// The lane's rows of a block of a column, whose maximum is a -> the block's scale byte and their codes.
template <int DT, int B, int SF, int RND>
__device__ __forceinline__ uint32_t column_block(const float (&v)[B], float a, float g, float k, const uint16_t *mine, int lane, uint32_t (&words)[B / 8])
{
    constexpr bool MXS = SF == NVFP4_SCALE_E8M0;
    float q;
    const uint32_t sbyte = block_scale<SF, true, false>(a, g, k, &q);
    if (MXS) q = mx_scale_operand(sbyte);
#pragma unroll
    for (int w = 0; w < B / 8; ++w) {
        uint32_t lo = 0, hi = 0;
        auto pair = [&](auto byte) {
            constexpr int BYTE = decltype(byte)::value;
            const int r = 8 * w + 2 * BYTE;
            const float x0 = MXS ? v[r] : v[r] * q, x1 = MXS ? v[r + 1] : v[r + 1] * q;
            if constexpr (RND == NVFP4_RTN) {
                lo = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(lo, x0, x1, MXS ? q : 1.0f, BYTE);
            } else {
                const uint32_t s0 = sr_seed_first(mine[r * 64 + lane_column<DT>(lane)]), s1 = sr_seed_first(mine[(r + 1) * 64 + lane_column<DT>(lane)]);
                lo = sr_scaled<BYTE>(lo, x0, s0, MXS ? q : 1.0f);
                hi = sr_scaled<BYTE>(hi, x1, s1, MXS ? q : 1.0f);
            }
        };
        pair(std::integral_constant<int, 0>());
        pair(std::integral_constant<int, 1>());
        pair(std::integral_constant<int, 2>());
        pair(std::integral_constant<int, 3>());
        words[w] = lo | (hi << 4);
    }
    return sbyte;
}

// One lane = one block of B rows of one column (of blocks of 64 and 128 rows: 32 rows, and two or four waves share a block and exchange
// its maximum through LDS), a wave = 64 columns, the waves of a workgroup one below the other, so that the 8 or 16 code bytes that they
// store to an output row make up one line; row-major outputs, cols a multiple of 8.
constexpr int small_rows(int block) { return block < 32 ? block : 32; }
template <int DT, int B, int SF, int RND>
__device__ __forceinline__ float cols_small(const QuantArgs &P, const unsigned wg, uint32_t *draws)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    constexpr int H = small_rows(B), WPB = B / H;  // rows of a lane, waves of a block
    const unsigned groups = (unsigned)((P.cols + 63) / 64), nblk = (unsigned)(P.rows / H);
    const unsigned band = wg / groups, blk = band * (SMALL_NT / 64) + wave;
    const int64_t row0 = (int64_t)blk * H, col0 = (int64_t)(wg - band * groups) * 64, col = col0 + lane_column<DT>(lane);
    const bool live = blk < nblk && col < P.cols;  // (of two lanes that share a dword both or neither: cols is even)
    float v[H];
    load_column<DT, H>(P, row0, col0, lane, live, v);
    uint16_t *const mine = reinterpret_cast<uint16_t *>(draws) + wave * (H * 64);
    if (RND == NVFP4_SR) column_draws<H>(P, row0, col0, lane, mine);
    const float g = resolve_g<DT, SMALL_NT, SF == NVFP4_SCALE_E4M3>(P);
    const float k = 1.0f / (6.0f * g);
    float a = column_max(v);
    if constexpr (WPB > 1) {
        __shared__ float part[SMALL_NT];
        part[threadIdx.x] = a;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < WPB; ++w) a = fmaxf(a, part[(wave / WPB * WPB + w) * 64 + lane]);
    }
    uint32_t words[H / 8];
    const uint32_t sbyte = column_block<DT, H, SF, RND>(v, a, g, k, mine, lane, words);
    if (live) {
        uint8_t *const dst = P.codes + col * (P.rows >> 1) + (row0 >> 1);
#pragma unroll
        for (int w = 0; w < H / 8; w += 2) *reinterpret_cast<uint2 *>(dst + 4 * w) = make_uint2(words[w], words[w + 1]);
        if (WPB == 1 || blk % WPB == 0) P.scales[col * (int64_t)(nblk / WPB) + blk / WPB] = (uint8_t)sbyte;
    }
    return g;
}

// (host) the job of one orientation of a tensor
SmallJob small_job(const QuantArgs &q, int axis, int rounding, int block);

}  // namespace nvfp4
