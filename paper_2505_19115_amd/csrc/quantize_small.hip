// Quantizer kernels for small tensors (small_tensor()): columns or both orientations of one or two tensors, and rows, in one launch.
#include "quantize_small.h"

namespace nvfp4 {

template <int DT, int B, int SF>
__global__ __launch_bounds__(SMALL_NT) void quantize_small_kernel(SmallJob j0, SmallJob j1, SmallJob j2, SmallJob j3)
{
    __shared__ __align__(16) uint32_t draws[SMALL_NT / 64 * small_rows(B) * 32];
    unsigned wg = blockIdx.x;
    const unsigned e0 = j0.wgs, e1 = e0 + j1.wgs, e2 = e1 + j2.wgs;
    const SmallJob &J = wg < e0 ? j0 : wg < e1 ? j1 : wg < e2 ? j2 : j3;
    wg -= wg < e0 ? 0 : wg < e1 ? e0 : wg < e2 ? e1 : e2;
    float g;
    if (J.axis == 1)
        g = J.rounding == NVFP4_RTN ? rows_tile<DT, B, SF, NVFP4_RTN, true, SMALL_NT, 1>(J.q, wg) : rows_tile<DT, B, SF, NVFP4_SR, true, SMALL_NT, 1>(J.q, wg);
    else
        g = J.rounding == NVFP4_RTN ? cols_small<DT, B, SF, NVFP4_RTN>(J.q, wg, draws) : cols_small<DT, B, SF, NVFP4_SR>(J.q, wg, draws);
    if (wg == 0 && threadIdx.x == 0 && J.q.g_out) {
        // (a `saved` buffer that is not the one this call expects poisons the scale the GEMMs will multiply by)
        const float g_gemm = tag_apply(J.tag) ? g : __builtin_nanf("");
        *J.q.g_out = g_gemm;
        if (J.g_out2) *J.g_out2 = g_gemm;
    }
}

// Rows of one tensor, or of two (round to nearest; the first `wgs` workgroups take the first), by themselves: a chunk per lane as above.  At
// 2-3 us what counts is what a launch brings along, so these have neither the other kernel's four jobs nor its 16 or 32 KB of LDS.  GPU
// time, us, bf16 RtN / SR, the kernel with four chunks per thread / the jobs kernel / this one:
//              NVFP4                                          NVFP4, scale preset                           MXFP4
//      1 x 64  2.62 / 3.04 / 2.36   3.32 / 3.28 / 2.53        2.00 / 2.37 / 1.86   2.73 / 2.59 / 1.91       1.85 / 2.13 / 1.82   2.46 / 2.41 / 1.86
//     64 x 256 3.33 / 3.36 / 2.87   3.88 / 3.56 / 3.01        2.75 / 2.55 / 2.13   3.30 / 2.74 / 2.24       2.14 / 2.25 / 1.99   2.80 / 2.59 / 2.06
//   1024 x 512 5.85 / 5.61 / 5.03   6.37 / 5.84 / 5.31        2.95 / 2.64 / 2.20   3.49 / 2.93 / 2.45       2.51 / 2.34 / 2.03   3.07 / 2.76 / 2.35
// (workgroups of 256: 16 x 4096 NVFP4 4.3 instead of 3.8, which take the maximum of the whole tensor in each; elsewhere alike.)
template <int DT, int B, int SF, int RND>
__global__ __launch_bounds__(SMALL_NT) void quantize_small_rows_kernel(QuantArgs P)
{
    const float g = rows_tile<DT, B, SF, RND, true, SMALL_NT, 1>(P, blockIdx.x);
    if (blockIdx.x == 0 && threadIdx.x == 0) *P.g_out = g;
}
template <int DT, int B, int SF>
__global__ __launch_bounds__(SMALL_NT) void quantize_small_rows_pair_kernel(QuantArgs P0, QuantArgs P1, unsigned wgs)
{
    const bool first = blockIdx.x < wgs;
    const QuantArgs &P = first ? P0 : P1;
    const unsigned wg = first ? blockIdx.x : blockIdx.x - wgs;
    const float g = rows_tile<DT, B, SF, NVFP4_RTN, true, SMALL_NT, 1>(P, wg);
    if (wg == 0 && threadIdx.x == 0) *P.g_out = g;
}

// ------------------------------------------------------------------ host side

// Tensors that go through quantize_small_kernel, in elements.  Its lanes reload nothing and share nothing between the orientations, so a
// large tensor is read twice by its dual form and stored in smaller pieces; us, the other kernels / this one, scale preset, blocks of 16:
//                  bf16 rows SR  columns RtN  columns SR   RtN+RtN      SR+SR         binary32 rows SR  columns SR   RtN+RtN      SR+SR
//     64 x  256     3.6 / 3.0    5.5 / 3.1    7.6 / 3.7    6.7 / 3.0   10.4 / 3.6       3.4 / 3.0    7.5 / 3.4    6.6 / 2.9   10.3 / 3.4
//   1024 x 1024     3.7 / 3.2    6.4 / 3.9    8.4 / 4.5    9.0 / 4.4   12.6 / 5.2       3.7 / 3.4    9.9 / 4.3    9.7 / 4.2   12.9 / 4.9
//   1024 x 2048     3.8 / 3.9    6.5 / 4.3    8.5 / 4.9    9.3 / 5.1   13.0 / 6.1       4.1 / 4.2   10.1 / 4.8    9.9 / 5.2   13.2 / 6.2
//   2048 x 2048     4.6 / 5.3    8.8 / 5.8   10.5 / 6.4   11.0 / 8.0   14.8 / 8.9       6.0 / 5.6   10.6 / 6.5   10.7 / 8.8   14.2 / 9.8
//   2080 x 2784     5.7 / 6.6    9.8 / 7.5   12.0 / 8.2   12.4 / 11.6  16.5 / 12.7      7.3 / 7.2   12.0 / 8.3   11.9 / 13.3  15.6 / 14.7
//   2048 x 4096     6.6 / 8.6    9.2 / 8.5   11.0 / 9.4   11.6 / 13.6  15.6 / 15.6      9.0 / 9.7   11.6 / 9.9   11.5 / 18.5  14.9 / 19.4
//   4096 x 4096     9.8 / 14.8  11.4 / 15.2  15.6 / 15.8  15.1 / 28.0  22.5 / 31.4     15.6 / 17.8  19.6 / 18.5  20.1 / 35.5  22.0 / 36.2
// (MXFP4: the same lines, columns SR of 4096 x 4096 binary32 21.9 / 16.2.  The rows as jobs of the columns' kernel; by themselves, as they
// are launched now, 0.4 us less.)
// E4M3 blocks of 64 (of 128 the same within 3 %), whose dual form is otherwise two launches; their rows by themselves stay where they are:
//                  bf16 columns RtN  columns SR   RtN+RtN      SR+SR         binary32 columns RtN  columns SR   RtN+RtN      SR+SR
//    256 x  256        5.8 / 3.8      7.8 / 5.0    8.5 / 3.7   10.9 / 5.0          7.3 / 3.4        8.6 / 4.6    9.2 / 3.4   11.6 / 4.6
//   1024 x 1024        6.0 / 4.0      7.9 / 5.1    9.5 / 4.4   12.2 / 5.9          7.6 / 3.7        9.7 / 4.8   11.3 / 4.3   13.5 / 5.7
//   2048 x 2048        8.5 / 5.3     10.6 / 6.4   12.5 / 9.6   15.5 / 11.0         8.5 / 6.4       10.6 / 7.3   13.7 / 11.8  16.4 / 12.1
//   2048 x 4096        9.2 / 8.2     11.4 / 9.1   14.2 / 13.7  18.0 / 16.6        10.1 / 9.0       11.7 / 9.9   18.5 / 17.5  20.4 / 19.0
//   4096 x 4096       11.7 / 11.7    16.3 / 16.4  20.0 / 20.2  26.0 / 26.0        17.5 / 18.2      19.9 / 19.1  32.4 / 32.1  35.3 / 34.4
// (forward and backward of 1024 x 1024 x 1024 with saved operands, bf16, blocks of 64: 71.3 / 43.8)
bool small_tensor(int dt, const QuantArgs &P, int block, int sf, bool hw, SmallUse use)
{
    const bool bf16 = dt == NVFP4_BF16;
    const int64_t M = 1 << 20;
    // (narrow ones of more than 512 workgroup tiles of 128 x 256 are walked by the streaming kernels)
    if (block > 32)
        return hw && sf == NVFP4_SCALE_E4M3 && use != SMALL_ROWS && (P.cols & 7) == 0 && P.rows * P.cols <= 8 * M &&
               ((P.rows + 127) / 128) * ((P.cols + 255) / 256) <= 512;
    const int64_t most = use == SMALL_ROWS ? (bf16 ? M : 4 * M) : use == SMALL_COLUMNS ? (bf16 ? 8 * M : 16 * M) : 4 * M;
    return hw && (P.cols & 7) == 0 && P.rows * P.cols <= most;
}
SmallJob small_job(const QuantArgs &q, int axis, int rounding, int block)
{
    SmallJob j = {q, axis, rounding, 0, nullptr, {}};
    constexpr int WAVES = SMALL_NT / 64;
    j.wgs = (unsigned)(axis == 1 ? (q.rows * (q.cols >> 3) + SMALL_NT - 1) / SMALL_NT : (q.rows / small_rows(block) + WAVES - 1) / WAVES * ((q.cols + 63) / 64));
    return j;
}
// the jobs of a dual quantization (row-major outputs): rows, which also write the scale, and columns
static void small_dual_jobs(const DualArgs &D, int rnd_r, int rnd_c, int block, SmallJob *j)
{
    QuantArgs r = D.c;
    r.codes = D.codes_r;
    r.scales = D.scales_r;
    r.seed = D.seed_r;
    j[0] = small_job(r, 1, rnd_r, block);
    j[0].g_out2 = D.g_out2;
    j[0].tag = D.tag;
    QuantArgs c = D.c;
    c.g_out = nullptr;
    j[1] = small_job(c, 0, rnd_c, block);
}
template <int DT>
static void launch_small_dt(const SmallJob (&j)[4], int block, int sf, hipStream_t st)
{
    const dim3 grid(j[0].wgs + j[1].wgs + j[2].wgs + j[3].wgs), wg(SMALL_NT);
    if (block == 64) hipLaunchKernelGGL((quantize_small_kernel<DT, 64, NVFP4_SCALE_E4M3>), grid, wg, 0, st, j[0], j[1], j[2], j[3]);
    else if (block == 128) hipLaunchKernelGGL((quantize_small_kernel<DT, 128, NVFP4_SCALE_E4M3>), grid, wg, 0, st, j[0], j[1], j[2], j[3]);
    else if (block == 16 && sf == NVFP4_SCALE_E4M3) hipLaunchKernelGGL((quantize_small_kernel<DT, 16, NVFP4_SCALE_E4M3>), grid, wg, 0, st, j[0], j[1], j[2], j[3]);
    else if (block == 16) hipLaunchKernelGGL((quantize_small_kernel<DT, 16, NVFP4_SCALE_E8M0>), grid, wg, 0, st, j[0], j[1], j[2], j[3]);
    else if (sf == NVFP4_SCALE_E4M3) hipLaunchKernelGGL((quantize_small_kernel<DT, 32, NVFP4_SCALE_E4M3>), grid, wg, 0, st, j[0], j[1], j[2], j[3]);
    else hipLaunchKernelGGL((quantize_small_kernel<DT, 32, NVFP4_SCALE_E8M0>), grid, wg, 0, st, j[0], j[1], j[2], j[3]);
}
static hipError_t launch_small(const SmallJob (&j)[4], int dt, int block, int sf, hipStream_t st)
{
    if (dt == NVFP4_BF16) launch_small_dt<NVFP4_BF16>(j, block, sf, st);
    else launch_small_dt<NVFP4_F32>(j, block, sf, st);
    return hipGetLastError();
}

template <int DT, int B, int SF>
static void launch_small_rows(const QuantArgs &P, const QuantArgs *P1, int rounding, hipStream_t st)
{
    const unsigned w0 = small_job(P, 1, rounding, B).wgs, w1 = P1 ? small_job(*P1, 1, rounding, B).wgs : 0;
    if (P1) hipLaunchKernelGGL((quantize_small_rows_pair_kernel<DT, B, SF>), dim3(w0 + w1), dim3(SMALL_NT), 0, st, P, *P1, w0);
    else if (rounding == NVFP4_RTN) hipLaunchKernelGGL((quantize_small_rows_kernel<DT, B, SF, NVFP4_RTN>), dim3(w0), dim3(SMALL_NT), 0, st, P);
    else hipLaunchKernelGGL((quantize_small_rows_kernel<DT, B, SF, NVFP4_SR>), dim3(w0), dim3(SMALL_NT), 0, st, P);
}
template <int DT>
static void launch_small_rows_dt(const QuantArgs &P, const QuantArgs *P1, int rounding, int block, int sf, hipStream_t st)
{
    if (block == 16 && sf == NVFP4_SCALE_E4M3) launch_small_rows<DT, 16, NVFP4_SCALE_E4M3>(P, P1, rounding, st);
    else if (block == 16) launch_small_rows<DT, 16, NVFP4_SCALE_E8M0>(P, P1, rounding, st);
    else if (sf == NVFP4_SCALE_E4M3) launch_small_rows<DT, 32, NVFP4_SCALE_E4M3>(P, P1, rounding, st);
    else launch_small_rows<DT, 32, NVFP4_SCALE_E8M0>(P, P1, rounding, st);
}
hipError_t launch_quantize_small_rows(const QuantArgs &P, const QuantArgs *P1, int dt, int rounding, int block, int sf, hipStream_t st)
{
    if (dt == NVFP4_BF16) launch_small_rows_dt<NVFP4_BF16>(P, P1, rounding, block, sf, st);
    else launch_small_rows_dt<NVFP4_F32>(P, P1, rounding, block, sf, st);
    return hipGetLastError();
}

hipError_t launch_quantize_small_columns(const QuantArgs &P, int dt, int rounding, int block, int sf, hipStream_t st)
{
    const SmallJob j[4] = {small_job(P, 0, rounding, block)};
    return launch_small(j, dt, block, sf, st);
}

hipError_t launch_quantize_small_dual(const DualArgs &D, const DualArgs *W, int dt, int rnd_r, int rnd_c, int block, int sf, hipStream_t st)
{
    SmallJob j[4] = {};
    small_dual_jobs(D, rnd_r, rnd_c, block, j);
    if (W) small_dual_jobs(*W, NVFP4_RTN, NVFP4_RTN, block, j + 2);
    return launch_small(j, dt, block, sf, st);
}

hipError_t launch_quantize_small_backward(const DualArgs &dY, const QuantArgs *W, const QuantArgs *X, int dt, int block, int sf, hipStream_t st)
{
    SmallJob j[4] = {};
    small_dual_jobs(dY, NVFP4_SR, NVFP4_SR, block, j);
    if (W) j[2] = small_job(*W, 0, NVFP4_RTN, block);
    if (X) j[3] = small_job(*X, 0, NVFP4_SR, block);
    return launch_small(j, dt, block, sf, st);
}

}  // namespace nvfp4
