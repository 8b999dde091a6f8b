// GEMM epilogue shared by the tile kernels: a wave's TA x TB accumulator tiles of 32 x 32 -> output rows in complete pieces.
#pragma once
#include "kernels.h"

namespace nvfp4 {

// Accumulator register 4 q + e of lane (r = lane % 32, h = lane / 32) of tile (a, b) is output row 32 a + r, column
// 32 b + 8 q + 4 h + e of the wave's part, which starts at (row0, col0).  32 rows at a time are transposed through a private
// piece of LDS (`mine`, 32 rows x 32 TB elements; 16-byte pieces XOR-swizzled by row) so that a store instruction writes
// whole rows of 64 or 128 bytes instead of 32 pieces of 8: measured 2.5-5 % of a GEMM.  Pieces past the edge are cut
// element by element, so a tile at the edge of a ragged output keeps wide stores everywhere else.
// No wave may still read `mine`, no load may still write it.  The lane coordinates are re-derived from an opaque copy so
// that none of the addressing is computed before the K loop and kept in registers across it.
template <int OUT_DT, int TA, int TB, class ACC>
__device__ __forceinline__ void store_lines(const GemmArgs &P, const ACC (&acc)[TA][TB], int64_t row0, int64_t col0, uint8_t *mine,
                                            int lane)
{
    typedef __bf16 b2_t __attribute__((ext_vector_type(2)));
    typedef float f2_t __attribute__((ext_vector_type(2)));
    constexpr int ESZ = OUT_DT == NVFP4_F32 ? 4 : 2, EPC = 16 / ESZ;   // element size, elements per piece
    constexpr int ROWB = 32 * TB * ESZ, CPR = ROWB / 16, SWZ = CPR - 1;  // bytes and pieces per row (CPR a power of two)
    static_assert((CPR & SWZ) == 0, "the swizzle needs a power of two");
    asm volatile("" : "+v"(lane));
    const int r = lane & 31, h = lane >> 5;
    const float gg = P.gA[0] * P.gB[0];
    const bool wide = P.ldc % EPC == 0;
    const bool full = wide && row0 + 32 * TA <= P.M && col0 + 32 * TB <= P.N;  // (uniform: no predicate inside)
#pragma unroll
    for (int a = 0; a < TA; ++a) {
#pragma unroll
        for (int b = 0; b < TB; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float y0 = acc[a][b][4 * q] * gg, y1 = acc[a][b][4 * q + 1] * gg;
                const float y2 = acc[a][b][4 * q + 2] * gg, y3 = acc[a][b][4 * q + 3] * gg;
                if (OUT_DT == NVFP4_F32) {
                    const int c = 8 * b + 2 * q + h;
                    *reinterpret_cast<float4 *>(mine + r * ROWB + ((c ^ (r & SWZ)) << 4)) = make_float4(y0, y1, y2, y3);
                } else {
                    const f2_t lo = {y0, y1}, hi = {y2, y3};
                    uint2 w;
                    w.x = __builtin_bit_cast(uint32_t, __builtin_convertvector(lo, b2_t));
                    w.y = __builtin_bit_cast(uint32_t, __builtin_convertvector(hi, b2_t));
                    const int c = 4 * b + q;
                    *reinterpret_cast<uint2 *>(mine + r * ROWB + ((c ^ (r & SWZ)) << 4) + 8 * h) = w;
                }
            }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int i = 0; i < CPR / 2; ++i) {
            const int id = 64 * i + lane, rowl = id / CPR, c = id % CPR;
            const uint4 v = *reinterpret_cast<const uint4 *>(mine + rowl * ROWB + ((c ^ (rowl & SWZ)) << 4));
            const int64_t grow = row0 + 32 * a + rowl, gcol = col0 + EPC * c;
            uint8_t *const dst = reinterpret_cast<uint8_t *>(P.out) + (grow * P.ldc + gcol) * ESZ;
            if (full) {
                *reinterpret_cast<uint4 *>(dst) = v;
            } else if (grow < P.M) {
                if (wide && gcol + EPC <= P.N) {
                    *reinterpret_cast<uint4 *>(dst) = v;
                } else {
                    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int e = 0; e < EPC; ++e)
                        if (gcol + e < P.N) {
                            if (OUT_DT == NVFP4_F32)
                                reinterpret_cast<uint32_t *>(dst)[e] = w[e];
                            else
                                reinterpret_cast<uint16_t *>(dst)[e] = (uint16_t)(w[e >> 1] >> (16 * (e & 1)));
                        }
                }
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
}

}  // namespace nvfp4
