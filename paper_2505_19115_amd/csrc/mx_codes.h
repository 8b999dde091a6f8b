// Where the direct-to-LDS MXFP4 kernel (gemm_mx.hip) fetches one operand's packed codes from: addresses alone, so that a host program can
// walk them (tests/mx_codes_main.cpp).
#pragma once
#include "kernels.h"

namespace nvfp4 {

// A workgroup's 256 rows of an operand of K tiles of 64 bytes a row.  A wave's lane fetches 16 bytes in each of four instructions: part u is row
// row(wave, u, lane) at chunk `c` of the K tile (the caller's choice: it is the swizzle of the LDS image).  Row-major rows past the edge are clamped to the
// last one.  A slab holds all 256 rows, and 16 rows further lie 128 bytes further (slab_row(16 u + j) = 2 u + slab_row(j), 64 bytes a position): a constant
// of the instruction, so that ONE lane offset serves the four parts.
template <bool SLAB>
struct MxCodes {
    static constexpr int OFFSETS = SLAB ? 1 : 4;
    uint32_t off[OFFSETS];  // of the lane, from p
    const uint8_t *tile;    // the operand's first K tile of these rows
    const uint8_t *p;       // the K tile that is fetched next
    uint32_t step;          // from one K tile to the next: 64 bytes along every row, or a slab of 16 KB

    __host__ __device__ static int row(int wave, int u, int lane) { return (wave * 4 + u) * 16 + (lane >> 2); }
    __host__ __device__ static constexpr int more(int u) { return SLAB ? 128 * u : 0; }
    // (rows: those of the operand from the first of these on, 256 at most)
    __host__ __device__ __forceinline__ void lane_offsets(int wave, int lane, int c, int64_t rows, int64_t Kb)
    {
#pragma unroll
        for (int u = 0; u < OFFSETS; ++u) {
            const int r = row(wave, u, lane);
            off[u] = SLAB ? (uint32_t)(slab_row(r) * 64 + c * 16) : (uint32_t)((r < rows ? r : rows - 1) * Kb + c * 16);
        }
    }
    __host__ __device__ __forceinline__ void start(const uint8_t *first)
    {
        tile = p = first;
        step = SLAB ? (uint32_t)SLAB_CODE_BYTES : 64u;
    }
    __host__ __device__ __forceinline__ void advance() { p += step; }
    // Past the last K tile the loads repeat the first bytes of the operand's OWN first tile: a part's constant stays in the instruction, and only there is
    // it known to be in range (a slab has 16 KB, the single row of another operand's last tile 256 bytes).
    __host__ __device__ __forceinline__ void past_end()
    {
#pragma unroll
        for (int u = 0; u < OFFSETS; ++u) off[u] = 0;
        p = tile;
        step = 0;
    }
};

}  // namespace nvfp4
