// What the kernels for small products share (gemm_ksplit.hip, fused_small.hip): a K tile's products from an LDS stage, and the sum of the waves'
// partial tiles.
#pragma once
#include "kernels.h"
#include "nvfp4_math.h"

namespace nvfp4 {

namespace ks {

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef int int8v_t __attribute__((ext_vector_type(8)));
typedef float float16_t __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float float2v_t __attribute__((ext_vector_type(2)));
typedef float float4v_t __attribute__((ext_vector_type(4)));

constexpr int KT = 128, KTB = 64;  // contraction elements and code bytes per row of a K tile
constexpr int QUAD = 1024 + 16;    // LDS bytes between the float4 planes of a partial tile (64 lanes, shifted by four banks)

template <int SF, int TA, int TB, int NW>
struct Geom {
    static constexpr int BM = 32 * TA, BN = 32 * TB, ROWS = BM + BN;
    static constexpr int CODES = ROWS * KTB;
    // E4M3: [4 chunks of 32 elements][ROWS] dwords, two fp16 scales each; E8M0: one dword (four bytes) per row
    static constexpr int SCALES = SF == NVFP4_SCALE_E4M3 ? ROWS * 16 : ROWS * 4;
    static constexpr int STAGE = CODES + SCALES;
    static constexpr int PARTIAL = TA * TB * 4 * QUAD;
    static constexpr int LDS = NW * (2 * STAGE > PARTIAL ? 2 * STAGE : PARTIAL);
};

// 8 codes (one dword) of one block -> 8 fp16 values times the block scale (see gemm.hip)
__device__ __forceinline__ half8_t dequant8(uint32_t w, _Float16 s)
{
    const half2_t s2 = {s, s};
    half2_t h0 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 256.0f, 0), h1 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 256.0f, 1);
    half2_t h2 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 256.0f, 2), h3 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 256.0f, 3);
    asm("" : "+v"(h0), "+v"(h1), "+v"(h2), "+v"(h3));  // (in fours, see gemm.hip: 1024 x 1024 x 2048 8.5 / 8.4 us, x 2048 in blocks of 64 9.3 / 8.9)
    h0 *= s2; h1 *= s2; h2 *= s2; h3 *= s2;
    half8_t r;
    r[0] = h0[0]; r[1] = h0[1]; r[2] = h1[0]; r[3] = h1[1];
    r[4] = h2[0]; r[5] = h2[1]; r[6] = h3[0]; r[7] = h3[1];
    return r;
}

}  // namespace ks

// One K tile of a wave: codes [ROWS][64 bytes, swizzled], then the scales (Geom).  tail: elements from `rem` on are missing.
template <int SF, int TA, int TB, int NW>
__device__ __forceinline__ void ksplit_compute(const uint8_t *stage, bool tail, int rem, ks::float16_t (&acc)[TA][TB], int lane)
{
    using namespace ks;
    using G = Geom<SF, TA, TB, NW>;
    constexpr bool MX = SF == NVFP4_SCALE_E8M0;
    constexpr int BM = G::BM, ROWS = G::ROWS;
    const int r = lane & 31, h = lane >> 5, sw = (r >> 2) & 3;
    const uint8_t *const p = stage + r * KTB;
    const uint32_t *const sS = reinterpret_cast<const uint32_t *>(stage + G::CODES) + r;
    if constexpr (MX) {
        uint32_t sa[TA], sb[TB];
#pragma unroll
        for (int a = 0; a < TA; ++a) sa[a] = sS[32 * a] >> (16 * h);
#pragma unroll
        for (int b = 0; b < TB; ++b) sb[b] = sS[BM + 32 * b] >> (16 * h);
        // MFMA step s of lane half h multiplies chunk 2 h + s
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            uint4 fa[TA], fb[TB];
            const int slot = ((2 * h + s) ^ sw) << 4;
#pragma unroll
            for (int a = 0; a < TA; ++a) {
                fa[a] = *reinterpret_cast<const uint4 *>(p + 32 * a * KTB + slot);
                if (tail && (2 * h + s) * 32 >= rem) fa[a] = make_uint4(0, 0, 0, 0);
            }
#pragma unroll
            for (int b = 0; b < TB; ++b) fb[b] = *reinterpret_cast<const uint4 *>(p + (BM + 32 * b) * KTB + slot);
#pragma unroll
            for (int a = 0; a < TA; ++a)
#pragma unroll
                for (int b = 0; b < TB; ++b) {
                    const int8v_t va = {(int)fa[a].x, (int)fa[a].y, (int)fa[a].z, (int)fa[a].w, 0, 0, 0, 0};
                    const int8v_t vb = {(int)fb[b].x, (int)fb[b].y, (int)fb[b].z, (int)fb[b].w, 0, 0, 0, 0};
                    if (s == 0)
                        acc[a][b] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(vb, va, acc[a][b], 4, 4, 0, (int)sb[b], 0, (int)sa[a]);
                    else
                        acc[a][b] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(vb, va, acc[a][b], 4, 4, 1, (int)sb[b], 1, (int)sa[a]);
                }
        }
    } else {
        // lane half h multiplies chunks h and 2 + h, a dword (8 codes) per MFMA step
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            uint4 ca[TA], cb[TB];
            half2_t sa[TA], sb[TB];
            const int slot = ((2 * q + h) ^ sw) << 4;
#pragma unroll
            for (int a = 0; a < TA; ++a) {
                ca[a] = *reinterpret_cast<const uint4 *>(p + 32 * a * KTB + slot);
                sa[a] = __builtin_bit_cast(half2_t, sS[(2 * q + h) * ROWS + 32 * a]);
            }
#pragma unroll
            for (int b = 0; b < TB; ++b) {
                cb[b] = *reinterpret_cast<const uint4 *>(p + (BM + 32 * b) * KTB + slot);
                sb[b] = __builtin_bit_cast(half2_t, sS[(2 * q + h) * ROWS + BM + 32 * b]);
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                auto dword = [&](const uint4 &v) { return t == 0 ? v.x : t == 1 ? v.y : t == 2 ? v.z : v.w; };
                half8_t fa[TA], fb[TB];
#pragma unroll
                for (int a = 0; a < TA; ++a) fa[a] = dequant8(dword(ca[a]), t >= 2 ? sa[a][1] : sa[a][0]);
#pragma unroll
                for (int b = 0; b < TB; ++b) fb[b] = dequant8(dword(cb[b]), t >= 2 ? sb[b][1] : sb[b][0]);
#pragma unroll
                for (int a = 0; a < TA; ++a)
#pragma unroll
                    for (int b = 0; b < TB; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fb[b], fa[a], acc[a][b], 0, 0, 0);
            }
        }
    }
}

// (scale() gives the product of the tensor scales, which is not needed, and in the kernels on packed operands not loaded, before the sums)
template <int SF, int TA, int TB, int NW, int OUT_DT, class SCALE>
__device__ __forceinline__ void ksplit_finish(const GemmArgs &P, const ks::float16_t (&acc)[TA][TB], uint8_t *lds, int64_t m0, int64_t n0, SCALE scale)
{
    using namespace ks;
    using G = Geom<SF, TA, TB, NW>;
    constexpr int BM = G::BM, BN = G::BN;
    const int tid = threadIdx.x, lane = tid & 63;
    // ---- the NW partial tiles: accumulator register 4 q + e of lane (r, h) of MFMA tile (a, b) is output row 32 a + r, column
    // 32 b + 8 q + 4 h + e.  Plane (a, b, q) of a wave's partial holds 64 lanes x float4.
    __syncthreads();  // every wave is done with the stages
    {
        uint8_t *const part = lds + (tid >> 6) * G::PARTIAL + lane * 16;
#pragma unroll
        for (int a = 0; a < TA; ++a)
#pragma unroll
            for (int b = 0; b < TB; ++b)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<float4 *>(part + ((a * TB + b) * 4 + q) * QUAD) =
                        make_float4(acc[a][b][4 * q], acc[a][b][4 * q + 1], acc[a][b][4 * q + 2], acc[a][b][4 * q + 3]);
    }
    __syncthreads();
    const float gg = scale();
    // one thread sums 8 consecutive columns of a row over the waves, in their order
    constexpr int CPR = BN / 8;
    const bool wide = (OUT_DT == NVFP4_F32 ? (P.ldc & 3) : (P.ldc & 7)) == 0;
    for (int id = tid; id < BM * CPR; id += 64 * NW) {
        const int row = id / CPR, c8 = id % CPR;
        const uint8_t *src = lds + (((row >> 5) * TB + (c8 >> 2)) * 4 + (c8 & 3)) * QUAD + (row & 31) * 16;
        float y[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float4 lo = *reinterpret_cast<const float4 *>(src + w * G::PARTIAL);
            const float4 hi = *reinterpret_cast<const float4 *>(src + w * G::PARTIAL + 512);
            y[0] += lo.x; y[1] += lo.y; y[2] += lo.z; y[3] += lo.w;
            y[4] += hi.x; y[5] += hi.y; y[6] += hi.z; y[7] += hi.w;
        }
        const int64_t grow = m0 + row, gcol = n0 + 8 * c8;
        if (grow >= P.M || gcol >= P.N) continue;
#pragma unroll
        for (int t = 0; t < 8; ++t) y[t] *= gg;
        if (OUT_DT == NVFP4_F32) {
            float *dst = reinterpret_cast<float *>(P.out) + grow * P.ldc + gcol;
            if (wide && gcol + 8 <= P.N) {
                // (vector values, not structs of four: see store_lines.h)
                *reinterpret_cast<float4v_t *>(dst) = float4v_t{y[0], y[1], y[2], y[3]};
                *reinterpret_cast<float4v_t *>(dst + 4) = float4v_t{y[4], y[5], y[6], y[7]};
            } else {
#pragma unroll
                for (int t = 0; t < 8; ++t)
                    if (gcol + t < P.N) dst[t] = y[t];
            }
        } else {
            uint32_t w[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float2v_t f = {y[2 * t], y[2 * t + 1]};
                w[t] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2_t));
            }
            uint16_t *dst = reinterpret_cast<uint16_t *>(P.out) + grow * P.ldc + gcol;
            if (wide && gcol + 8 <= P.N) {
                *reinterpret_cast<uint4 *>(dst) = make_uint4(w[0], w[1], w[2], w[3]);
            } else if ((P.ldc & 3) == 0 && gcol + 8 <= P.N) {
                *reinterpret_cast<uint2 *>(dst) = make_uint2(w[0], w[1]);
                *reinterpret_cast<uint2 *>(dst + 4) = make_uint2(w[2], w[3]);
            } else {
#pragma unroll
                for (int t = 0; t < 8; ++t)
                    if (gcol + t < P.N) dst[t] = (uint16_t)(w[t >> 1] >> (16 * (t & 1)));
            }
        }
    }
}

}  // namespace nvfp4
