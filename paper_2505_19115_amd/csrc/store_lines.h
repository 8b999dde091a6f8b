// GEMM epilogue shared by the tile kernels: a wave's TA x TB accumulator tiles of 32 x 32 or 16 x 16 -> output rows in complete pieces.
#pragma once
#include "kernels.h"

namespace nvfp4 {

// Tiles of 32 x 32 (16 accumulators a lane) or of 16 x 16 (4 a lane).  32 x 32: register 4 q + e of lane (r = lane % 32,
// h = lane / 32) of tile (a, b) is output row 32 a + r, column 32 b + 8 q + 4 h + e of the wave's part, which starts at (row0, col0);
// 16 x 16: register e of lane (r = lane % 16, g = lane / 16) is row 16 a + r, column 16 b + 4 g + e.  acc holds TB tiles a row, one row of
// them or two in each of its S strips.  A strip at a time (32 rows, or 16) is transposed
// through a private piece of LDS (`mine`, the strip's rows of the wave's columns; 16-byte pieces XOR-swizzled by row) so that a store instruction writes
// whole rows of 64 or 128 bytes instead of 32 pieces of 8: measured 2.5-5 % of a GEMM.  Pieces past the edge are cut
// element by element, so a tile at the edge of a ragged output keeps wide stores everywhere else.
// No wave may still read `mine`, no load may still write it.  The lane coordinates are re-derived from an opaque copy so
// that none of the addressing is computed before the K loop and kept in registers across it.
// Forms for a wave's part inside the output (the usual case: no predicate, nothing between the LDS reads and the stores; streaming or not),
// for one at the edge of an output whose rows end with a whole piece, where a lane past the edge stores the last piece inside once more instead
// of being left out (four waves of 128 columns, one per SIMD, whose branches nothing covers: 6624 x 1376 x 1408, 192 x 256 tiles, 27.2
// against 32.7 us; MXFP4 4000 x 4000 x 1024 15.5 against 21.2), and for any other edge.  Pieces are vector values: in one form, with pieces as structs of four words, the compiler stored the last
// word of a piece apart, sharing that store with the cut pieces, and binary32 rows left in 12 + 4 bytes: 8192 x 8192 x 1024 (E4M3,
// 256 x 256 tiles) 151 us against 137.
enum { STORE_INSIDE, STORE_STREAMED, STORE_WHOLE_PIECES, STORE_EDGE };
template <int OUT_DT, int TB, int FORM, int S, int C, class ACC>
__device__ __forceinline__ void store_lines_form(const TileArgs &P, const ACC (&acc)[S][C], int64_t row0, int64_t col0, uint8_t *mine,
                                                 unsigned lane, float gg, bool wide, bool half)
{
    typedef __bf16 b2_t __attribute__((ext_vector_type(2)));
    typedef float f2_t __attribute__((ext_vector_type(2)));
    typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
    typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
    constexpr int MT = sizeof(ACC) == 16 ? 16 : 32;                    // rows and columns of an MFMA tile
    constexpr int IN = C / TB, ROWS = MT * IN;                         // tile rows and rows of a strip
    static_assert(C == IN * TB && ROWS <= 32, "whole tile rows");
    constexpr int ESZ = OUT_DT == NVFP4_F32 ? 4 : 2, EPC = 16 / ESZ;   // element size, elements per piece
    constexpr int ROWB = MT * TB * ESZ, CPR = ROWB / 16, SWZ = CPR - 1;  // bytes and pieces per row (CPR a power of two)
    constexpr int RPS = 64 / CPR;                                        // rows per store instruction
    static_assert((CPR & SWZ) == 0, "the swizzle needs a power of two");
    const unsigned r = lane & (MT - 1), g = lane / MT;
    const unsigned rowl0 = lane / CPR;
    unsigned c = lane % CPR;
    if (FORM == STORE_WHOLE_PIECES) {
        const unsigned last = P.N - col0 < EPC * CPR ? (unsigned)(P.N - col0) / EPC - 1 : CPR - 1;
        c = c < last ? c : last;
    }
    const int64_t grow0 = row0 + rowl0, gcol = col0 + EPC * c;
    uint8_t *const dst0 = reinterpret_cast<uint8_t *>(P.out) + ((FORM == STORE_WHOLE_PIECES ? row0 : grow0) * P.ldc + gcol) * ESZ;
#pragma unroll
    for (int a = 0; a < S; ++a) {
        if (FORM == STORE_WHOLE_PIECES && row0 + ROWS * a >= P.M) return;
#pragma unroll
        for (int i = 0; i < IN; ++i)
#pragma unroll
            for (int b = 0; b < TB; ++b)
#pragma unroll
                for (int q = 0; q < MT * MT / 256; ++q) {
                    const ACC &t = acc[a][TB * i + b];
                    const float y0 = t[4 * q] * gg, y1 = t[4 * q + 1] * gg, y2 = t[4 * q + 2] * gg, y3 = t[4 * q + 3] * gg;
                    const unsigned row = MT * i + r, col4 = MT / 4 * b + 64 / MT * q + g;  // (column / 4)
                    if (OUT_DT == NVFP4_F32) {
                        *reinterpret_cast<float4 *>(mine + row * ROWB + ((col4 ^ (row & SWZ)) << 4)) = make_float4(y0, y1, y2, y3);
                    } else {
                        const f2_t lo = {y0, y1}, hi = {y2, y3};
                        uint2 w;
                        w.x = __builtin_bit_cast(uint32_t, __builtin_convertvector(lo, b2_t));
                        w.y = __builtin_bit_cast(uint32_t, __builtin_convertvector(hi, b2_t));
                        *reinterpret_cast<uint2 *>(mine + row * ROWB + (((col4 >> 1) ^ (row & SWZ)) << 4) + 8 * (col4 & 1)) = w;
                    }
                }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int i = 0; i < ROWS / RPS; ++i) {
            unsigned rowl = rowl0 + RPS * i;
            if (FORM == STORE_WHOLE_PIECES) asm volatile("" : "+v"(rowl));  // (addresses of one store at a time: registers)
            if (FORM == STORE_WHOLE_PIECES) {
                const unsigned last = P.M - (row0 + ROWS * a) < ROWS ? (unsigned)(P.M - (row0 + ROWS * a)) - 1 : ROWS - 1;
                rowl = rowl < last ? rowl : last;
            }
            const u32x4_t v = *reinterpret_cast<const u32x4_t *>(mine + rowl * ROWB + ((c ^ (rowl & SWZ)) << 4));
            uint8_t *const dst = dst0 + (FORM == STORE_WHOLE_PIECES ? ROWS * a + (int64_t)rowl : (int64_t)(ROWS * a + RPS * i)) * P.ldc * ESZ;
            if (FORM == STORE_STREAMED) {
                __builtin_nontemporal_store(v, reinterpret_cast<u32x4_t *>(dst));
            } else if (FORM != STORE_EDGE) {
                *reinterpret_cast<u32x4_t *>(dst) = v;
            } else if (grow0 + ROWS * a + RPS * i < P.M) {
                if (wide && gcol + EPC <= P.N) {
                    *reinterpret_cast<u32x4_t *>(dst) = v;
                } else if (OUT_DT == NVFP4_BF16 && half && gcol + EPC <= P.N) {
                    *reinterpret_cast<u32x2_t *>(dst) = v.xy;
                    *reinterpret_cast<u32x2_t *>(dst + 8) = v.zw;
                } else {
#pragma unroll
                    for (int e = 0; e < EPC; ++e)
                        if (gcol + e < P.N) {
                            if (OUT_DT == NVFP4_F32)
                                reinterpret_cast<uint32_t *>(dst)[e] = v[e];
                            else
                                reinterpret_cast<uint16_t *>(dst)[e] = (uint16_t)(v[e >> 1] >> (16 * (e & 1)));
                        }
                }
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
}

template <int OUT_DT, int TB, int S, int C, class ACC>
__device__ __forceinline__ void store_lines(const TileArgs &P, const ACC (&acc)[S][C], int64_t row0, int64_t col0, uint8_t *mine,
                                            int lane)
{
    asm volatile("" : "+v"(lane));
    const float gg = P.gA[0] * P.gB[0];
    const bool wide = P.ldc % (OUT_DT == NVFP4_F32 ? 4 : 8) == 0;
    const bool half = P.ldc % 4 == 0;  // (bf16 rows start at multiples of 8 bytes: 303 x 6548 x 128 8.5 us in single elements)
    // (row0 and col0 are the same in the whole wave)
    constexpr int MT = sizeof(ACC) == 16 ? 16 : 32;
    if (wide && row0 + MT * (C / TB) * S <= P.M && col0 + MT * TB <= P.N) {
        if (P.stream) store_lines_form<OUT_DT, TB, STORE_STREAMED>(P, acc, row0, col0, mine, (unsigned)lane, gg, wide, half);
        else store_lines_form<OUT_DT, TB, STORE_INSIDE>(P, acc, row0, col0, mine, (unsigned)lane, gg, wide, half);
    } else if (wide && P.N % (OUT_DT == NVFP4_F32 ? 4 : 8) == 0) {
        if (row0 < P.M && col0 < P.N) store_lines_form<OUT_DT, TB, STORE_WHOLE_PIECES>(P, acc, row0, col0, mine, (unsigned)lane, gg, wide, half);
    } else
        store_lines_form<OUT_DT, TB, STORE_EDGE>(P, acc, row0, col0, mine, (unsigned)lane, gg, wide, half);
}

}  // namespace nvfp4
