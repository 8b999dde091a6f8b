// GEMM epilogue shared by the tile kernels: a wave's TA x TB accumulator tiles of 32 x 32 -> output rows in complete pieces.
#pragma once
#include "kernels.h"

namespace nvfp4 {

// Outputs up to this size leave by nontemporal stores, which do not wait for a place in the L2 (us, kept / streamed: NVFP4 1024 x 4096 x 4096,
// binary32 outputs, 38.1 / 36.6, bf16 35.5 / 34.4, 2048 x 4096 x 4096 66.7 / 65.8; MXFP4 2048 x 4096 x 4096 29.6 / 27.9), and still together
// with a kernel that reads the output next (quantizer 39.2 / 38.3, 71.5 / 70.9, 34.4 / 33.4).  Of larger ones the next kernel finds more in the
// last-level cache than the product gains: MXFP4 4096 x 11008 x 4096, 86 MB, 135.9 / 125.7, with a quantizer behind it 134.0 / 138.6; 40 MB 65.6 /
// 67.8.  (Weight gradients, which are not read next, of 90 MB: the backward half of an MLP of 4096 / 11008 at 2048 tokens 697 / 706, the whole
// one at 4096 tokens 2872 / 2848: not done.)
// Calls on packed weights, quantizer and product, us, kept / streamed, one by one and from a graph, MXFP4: 2048 x 4096 x 4096 34.0 / 32.9 and 35.0 / 33.5,
// 1024 x 4096 x 4096 with binary32 outputs 31.4 / 29.9 and 30.5 / 29.2, 4096 x 4096 x 2048 (32 MB) 32.3 / 31.3 and 31.8 / 30.6; of 70 random ones with 4 to
// 32 MB 0.97 to 1.10 times as fast (less than 0.99: 3076 x 928 x 928 and 3857 x 928 x 960, NVFP4), 628 x 5888 x 5504 with binary32 outputs 40.8 / 41.0 and
// 39.7 / 38.7.  Rows 32 KB apart are an exception near the line: MXFP4 1024 x 8192 x 1024 with binary32 outputs 17.2 / 18.2 and 17.1 / 18.3, x 2048 23.2 /
// 24.0 and 24.8 / 25.9, 1000 x 8192 x 2048 23.1 / 23.5 and 23.6 / 24.2, NVFP4 1024 x 8192 x 1024 28.5 / 29.2 and 28.4 / 28.8; 896 x 8192 x 1024 15.8 / 14.9
// and 1.02 times as fast (31 KB apart, 1024 x 7936 x 2048, 22.1 / 21.7 and 21.9 / 21.6; 64 KB apart, 512 x 16384 x 4096, 34.0 / 32.8).
// The kernels take the size from M and ldc: as a flag in GemmArgs it lengthened the arguments of every product's kernel (two of them are the
// small products' argument, 196 -> 212 bytes), and with them the host's work for a launch, by 0 to 0.2 us a call from box to box (us, 32 x 4096 x
// 4096 MXFP4 on packed weights, which is bound by that work, flag / none: 8.86 / 8.64, 11.11 / 11.12, 12.11 / 12.08).
__device__ __forceinline__ bool streamed_output(int64_t rows, int64_t row_bytes)
{
    return rows * row_bytes <= (row_bytes == 32 << 10 ? (int64_t)28 << 20 : (int64_t)32 << 20);
}

// Accumulator register 4 q + e of lane (r = lane % 32, h = lane / 32) of tile (a, b) is output row 32 a + r, column
// 32 b + 8 q + 4 h + e of the wave's part, which starts at (row0, col0).  32 rows at a time are transposed through a private
// piece of LDS (`mine`, 32 rows x 32 TB elements; 16-byte pieces XOR-swizzled by row) so that a store instruction writes
// whole rows of 64 or 128 bytes instead of 32 pieces of 8: measured 2.5-5 % of a GEMM.  Pieces past the edge are cut
// element by element, so a tile at the edge of a ragged output keeps wide stores everywhere else.
// No wave may still read `mine`, no load may still write it.  The lane coordinates are re-derived from an opaque copy so
// that none of the addressing is computed before the K loop and kept in registers across it.
// Forms for a wave's part inside the output (the usual case: no predicate, nothing between the LDS reads and the stores; streaming or not) and
// for one at its edge, and pieces as vector values: in one form, with pieces as structs of four words, the compiler stored the last
// word of a piece apart, sharing that store with the cut pieces, and binary32 rows left in 12 + 4 bytes: 8192 x 8192 x 1024 (E4M3,
// 256 x 256 tiles) 151 us against 137.
template <int OUT_DT, int TA, int TB, bool FULL, bool STREAM, class ACC>
__device__ __forceinline__ void store_lines_form(const GemmArgs &P, const ACC (&acc)[TA][TB], int64_t row0, int64_t col0, uint8_t *mine,
                                                 unsigned lane, float gg, bool wide, bool half)
{
    typedef __bf16 b2_t __attribute__((ext_vector_type(2)));
    typedef float f2_t __attribute__((ext_vector_type(2)));
    typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
    typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
    constexpr int ESZ = OUT_DT == NVFP4_F32 ? 4 : 2, EPC = 16 / ESZ;   // element size, elements per piece
    constexpr int ROWB = 32 * TB * ESZ, CPR = ROWB / 16, SWZ = CPR - 1;  // bytes and pieces per row (CPR a power of two)
    constexpr int RPS = 64 / CPR;                                        // rows per store instruction
    static_assert((CPR & SWZ) == 0, "the swizzle needs a power of two");
    const unsigned r = lane & 31, h = lane >> 5;
    const unsigned rowl0 = lane / CPR, c = lane % CPR;
    const int64_t grow0 = row0 + rowl0, gcol = col0 + EPC * c;
    uint8_t *const dst0 = reinterpret_cast<uint8_t *>(P.out) + (grow0 * P.ldc + gcol) * ESZ;
#pragma unroll
    for (int a = 0; a < TA; ++a) {
#pragma unroll
        for (int b = 0; b < TB; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float y0 = acc[a][b][4 * q] * gg, y1 = acc[a][b][4 * q + 1] * gg;
                const float y2 = acc[a][b][4 * q + 2] * gg, y3 = acc[a][b][4 * q + 3] * gg;
                if (OUT_DT == NVFP4_F32) {
                    const unsigned p = 8 * b + 2 * q + h;
                    *reinterpret_cast<float4 *>(mine + r * ROWB + ((p ^ (r & SWZ)) << 4)) = make_float4(y0, y1, y2, y3);
                } else {
                    const f2_t lo = {y0, y1}, hi = {y2, y3};
                    uint2 w;
                    w.x = __builtin_bit_cast(uint32_t, __builtin_convertvector(lo, b2_t));
                    w.y = __builtin_bit_cast(uint32_t, __builtin_convertvector(hi, b2_t));
                    const unsigned p = 4 * b + q;
                    *reinterpret_cast<uint2 *>(mine + r * ROWB + ((p ^ (r & SWZ)) << 4) + 8 * h) = w;
                }
            }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int i = 0; i < CPR / 2; ++i) {
            const unsigned rowl = rowl0 + RPS * i;
            const u32x4_t v = *reinterpret_cast<const u32x4_t *>(mine + rowl * ROWB + ((c ^ (rowl & SWZ)) << 4));
            uint8_t *const dst = dst0 + (int64_t)(32 * a + RPS * i) * P.ldc * ESZ;
            if (FULL && STREAM) {
                __builtin_nontemporal_store(v, reinterpret_cast<u32x4_t *>(dst));
            } else if (FULL) {
                *reinterpret_cast<u32x4_t *>(dst) = v;
            } else if (grow0 + 32 * a + RPS * i < P.M) {
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

template <int OUT_DT, int TA, int TB, class ACC>
__device__ __forceinline__ void store_lines(const GemmArgs &P, const ACC (&acc)[TA][TB], int64_t row0, int64_t col0, uint8_t *mine,
                                            int lane)
{
    asm volatile("" : "+v"(lane));
    const float gg = P.gA[0] * P.gB[0];
    const bool wide = P.ldc % (OUT_DT == NVFP4_F32 ? 4 : 8) == 0;
    const bool half = P.ldc % 4 == 0;  // (bf16 rows start at multiples of 8 bytes: 303 x 6548 x 128 8.5 us in single elements)
    // (row0 and col0 are the same in the whole wave)
    if (wide && row0 + 32 * TA <= P.M && col0 + 32 * TB <= P.N) {
        if (streamed_output(P.M, P.ldc * (OUT_DT == NVFP4_F32 ? 4 : 2))) store_lines_form<OUT_DT, TA, TB, true, true>(P, acc, row0, col0, mine, (unsigned)lane, gg, wide, half);
        else store_lines_form<OUT_DT, TA, TB, true, false>(P, acc, row0, col0, mine, (unsigned)lane, gg, wide, half);
    } else
        store_lines_form<OUT_DT, TA, TB, false, false>(P, acc, row0, col0, mine, (unsigned)lane, gg, wide, half);
}

}  // namespace nvfp4
