// Sums of the groups of waves that share out the contraction of a product's tile.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace nvfp4 {

// Sums of two halves of a workgroup (SIDE waves each, wave `w` of one facing wave `w` of the other) over the same N x TB accumulator tiles (4 or 16 registers a lane):
// the lower half keeps the first (N + 1) / 2 tile rows, the upper half the rest, each sends the other what it does not keep
// through the LDS (64 lanes x float4 per four registers: 1 KB, no bank conflicts).
template <int N, int TB, int SIDE, class ACC>
__device__ __forceinline__ void fold_groups(const ACC (&acc)[N][TB], ACC (&kept)[(N + 1) / 2][TB], uint8_t *lds, bool upper, int w,
                                            int lane)
{
    constexpr int Q = sizeof(ACC) / 16, LO = (N + 1) / 2, HI = N - LO, ROW = TB * Q * 1024;
    uint8_t *const from_lower = lds + w * (HI * ROW) + lane * 16, *const from_upper = lds + SIDE * (HI * ROW) + w * (LO * ROW) + lane * 16;
    const uint8_t *const theirs = upper ? from_lower : from_upper;
    uint8_t *const ours = upper ? from_upper : from_lower;
    // (what goes and what stays is chosen by value: a choice between array elements would put the accumulators into memory)
#pragma unroll
    for (int a = 0; a < LO; ++a)
#pragma unroll
        for (int b = 0; b < TB; ++b)
            if (a < HI || upper) {
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    float y[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float lo = acc[a][b][4 * q + e], hi = a < HI ? acc[LO + a < N ? LO + a : 0][b][4 * q + e] : 0.0f;
                        y[e] = upper ? lo : hi;
                        kept[a][b][4 * q + e] = upper ? hi : lo;
                    }
                    *reinterpret_cast<float4 *>(ours + ((a * TB + b) * Q + q) * 1024) = make_float4(y[0], y[1], y[2], y[3]);
                }
            } else {
                kept[a][b] = acc[a][b];
            }
    __syncthreads();
#pragma unroll
    for (int a = 0; a < LO; ++a)
#pragma unroll
        for (int b = 0; b < TB; ++b)
            if (a < HI || !upper) {
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    const float4 o = *reinterpret_cast<const float4 *>(theirs + ((a * TB + b) * Q + q) * 1024);
                    kept[a][b][4 * q] += o.x; kept[a][b][4 * q + 1] += o.y; kept[a][b][4 * q + 2] += o.z; kept[a][b][4 * q + 3] += o.w;
                }
            }
    __syncthreads();
}

}  // namespace nvfp4
