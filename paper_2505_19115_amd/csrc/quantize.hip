// Block quantizer kernels for gfx950: tensor maximum, row-blocked quantizer, column-blocked
// (transposed-output) quantizer.  Implements the operation Q of Eqs. 1-6 of "FP4 All the Way"
// for the formats of Sec. 3 / Table 1 and the two rounding modes of Sec. 3.2.
//
// Memory plan (the kernels are HBM-bound, so everything is about 16-byte coalesced access):
//   rows kernel   : one lane = 8 consecutive elements of a row (one 16 B load for bf16), a
//                   block of B elements = B/8 adjacent lanes, block maximum by DPP max across
//                   those lanes, one 4 B store of 8 packed codes per lane.
//   columns kernel: one lane = 16 or 8 consecutive rows x 8 consecutive columns held in registers.
//                   Lanes that are adjacent in the wave hold vertically adjacent row groups of
//                   the same 8 columns, so the waves of a workgroup read 512 B (bf16)
//                   contiguous per row and a wave writes 64 B contiguous per output row of the
//                   transposed code matrix, without staging through LDS.
#include "quantize_tile.h"

namespace nvfp4 {

// ------------------------------------------------------------------ tensor maximum (Q0)

// max|x| over a [rows, cols] tensor: one partial maximum (bit pattern) per workgroup into
// part_out[blockIdx.y * gridDim.x + blockIdx.x]; a single small workgroup folds them afterwards.
// (One atomic max per workgroup on a single address serializes: 8192 of them cost ~80 us.)
// grid.x covers the 8-element chunks of a row span (4 per thread, all four loads in flight
// before the first use), grid.y the row spans; for a dense tensor the host passes one span of
// rows*cols elements.  Loads are ordinary (cacheable): the quantizer reads the tensor again
// right after, and up to 256 MB of it are then still in the last-level cache.
constexpr int AMAX_UNROLL = 4;
template <int DT>
__global__ __launch_bounds__(256) void amax_kernel(const void *x, int64_t cols, int64_t ld,
                                                   uint32_t *part_out)
{
    const int64_t row = blockIdx.y;
    const int64_t nchunk = cols >> 3;
    const int64_t base = (int64_t)blockIdx.x * (256 * AMAX_UNROLL) + threadIdx.x;
    Chunk<DT> v[AMAX_UNROLL];
#pragma unroll
    for (int u = 0; u < AMAX_UNROLL; ++u) {
        const int64_t c = base + u * 256;
        if (c < nchunk)
            v[u].template load<false>(x, row * ld + c * 8);
        else
            v[u].zero();
    }
    float a = 0.0f;
#pragma unroll
    for (int u = 0; u < AMAX_UNROLL; ++u) a = fmaxf(a, chunk_amax(v[u]));
    if (blockIdx.x == 0 && threadIdx.x == 0 && (cols & 7)) {
        Chunk<DT> t;
        t.load_partial(x, row * ld + nchunk * 8, (int)(cols & 7));
        a = fmaxf(a, chunk_amax(t));
    }
    a = group_max<16>(a);
    // 4 rows of 16 lanes per wave, 4 waves: finish through LDS
    __shared__ uint32_t part[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if ((lane & 15) == 0) part[wave * 4 + (lane >> 4)] = f2u(a);
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t m = 0;
#pragma unroll
        for (int t = 0; t < 16; ++t) m = umax(m, part[t]);
        part_out[(int64_t)blockIdx.y * gridDim.x + blockIdx.x] = m;
    }
}

// A fixed grid of large workgroups strides over the chunks of one or two tensors (blockIdx.y), one partial each, which the
// consumer folds.  A strided tensor is walked as its rows of ceil(cols / 8) chunks (32-bit chunk numbers: one division per
// 16-byte load hides under the load).  Two tensors in one launch: a call on a small layer is bound by the launches in its
// chain (2-4 us each), not by their work.
constexpr int AMAX_DENSE_THREADS = 1024;
struct AmaxArgs {
    const void *x;
    int64_t n;           // dense: elements
    uint32_t rows, cpr;  // strided: rows, chunks per row
    int64_t cols, ld;
    uint32_t *part_out;
    unsigned grid;
};
template <int DT>
__device__ __forceinline__ void amax_store(float a, uint32_t *dst)
{
    a = group_max<16>(a);
    __shared__ uint32_t part[AMAX_DENSE_THREADS / 16];
    if ((threadIdx.x & 15) == 0) part[threadIdx.x >> 4] = f2u(a);
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t m = 0;
#pragma unroll
        for (int t = 0; t < AMAX_DENSE_THREADS / 16; ++t) m = umax(m, part[t]);
        *dst = m;
    }
}
template <int DT>
__global__ __launch_bounds__(AMAX_DENSE_THREADS) void amax_dense_kernel(AmaxArgs T0, AmaxArgs T1)
{
    const AmaxArgs &T = blockIdx.y == 0 ? T0 : T1;
    if (blockIdx.x >= T.grid) return;
    const int64_t nchunk = T.n >> 3;
    const int64_t stride = (int64_t)T.grid * (AMAX_DENSE_THREADS * AMAX_UNROLL);
    float a = 0.0f;
    for (int64_t base = (int64_t)blockIdx.x * (AMAX_DENSE_THREADS * AMAX_UNROLL) + threadIdx.x; base < nchunk; base += stride) {
        Chunk<DT> v[AMAX_UNROLL];
#pragma unroll
        for (int u = 0; u < AMAX_UNROLL; ++u) {
            const int64_t c = base + u * AMAX_DENSE_THREADS;
            if (c < nchunk)
                v[u].template load<false>(T.x, c * 8);
            else
                v[u].zero();
        }
#pragma unroll
        for (int u = 0; u < AMAX_UNROLL; ++u) a = fmaxf(a, chunk_amax(v[u]));
    }
    if (blockIdx.x == 0 && threadIdx.x == 0 && (T.n & 7)) {
        Chunk<DT> t;
        t.load_partial(T.x, nchunk * 8, (int)(T.n & 7));
        a = fmaxf(a, chunk_amax(t));
    }
    amax_store<DT>(a, T.part_out + blockIdx.x);
}
// The last chunk of a row that ends inside one is moved back to end with the row: a maximum may see elements twice, and every chunk
// is one wide load then.  (Element by element, the ends kept the loads around them from being in flight together: binary32 [2432, 6980]
// 14.6 us; rows shorter than a chunk still go that way.)
template <int DT>
__global__ __launch_bounds__(AMAX_DENSE_THREADS) void amax_strided_kernel(AmaxArgs T)
{
    const int64_t total = (int64_t)T.rows * T.cpr;  // (below 2^31)
    const int64_t stride = (int64_t)T.grid * (AMAX_DENSE_THREADS * AMAX_UNROLL);
    float a = 0.0f;
    if (T.cols < 8) {
        for (int64_t row = (int64_t)blockIdx.x * AMAX_DENSE_THREADS + threadIdx.x; row < T.rows; row += (int64_t)T.grid * AMAX_DENSE_THREADS) {
            Chunk<DT> v;
            v.load_partial(T.x, row * T.ld, (int)T.cols);
            a = fmaxf(a, chunk_amax(v));
        }
        amax_store<DT>(a, T.part_out + blockIdx.x);
        return;
    }
    for (int64_t base = (int64_t)blockIdx.x * (AMAX_DENSE_THREADS * AMAX_UNROLL) + threadIdx.x; base < total; base += stride) {
        Chunk<DT> v[AMAX_UNROLL];
#pragma unroll
        for (int u = 0; u < AMAX_UNROLL; ++u) {
            const int64_t id = base + u * AMAX_DENSE_THREADS;
            if (id < total) {
                const uint32_t row = (uint32_t)id / T.cpr, c = (uint32_t)id - row * T.cpr;
                const int64_t col = (int64_t)c * 8 + 8 <= T.cols ? (int64_t)c * 8 : T.cols - 8;
                v[u].load_unaligned(T.x, (int64_t)row * T.ld + col);
            } else {
                v[u].zero();
            }
        }
#pragma unroll
        for (int u = 0; u < AMAX_UNROLL; ++u) a = fmaxf(a, chunk_amax(v[u]));
    }
    amax_store<DT>(a, T.part_out + blockIdx.x);
}

// Folds n partial maxima into amax_bits[0]; with g_out != nullptr also writes the tensor scale.
__global__ __launch_bounds__(1024) void fold_amax_kernel(const uint32_t *partials, int64_t n,
                                                         uint32_t *amax_bits, float *g_out)
{
    uint32_t m = 0;
    for (int64_t i = threadIdx.x; i < n; i += 1024) m = umax(m, partials[i]);
    m = f2u(group_max<16>(u2f(m)));
    __shared__ uint32_t part[64];
    if ((threadIdx.x & 15) == 0) part[threadIdx.x >> 4] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t r = 0;
#pragma unroll
        for (int t = 0; t < 64; ++t) r = umax(r, part[t]);
        *amax_bits = r;
        if (g_out) *g_out = tensor_scale_from_amax(u2f(r));
    }
}

// ------------------------------------------------------------------ row-blocked quantizer

template <int DT, int B, int SF, int RND, bool HW>
__global__ __launch_bounds__(256) void quantize_rows_kernel(QuantArgs P)
{
    const float g = rows_tile<DT, B, SF, RND, HW>(P, blockIdx.x);
    if (blockIdx.x == 0 && threadIdx.x == 0) *P.g_out = g;
}

// Two tensors in one launch, round to nearest: the forward call's X and W.  The first `wgs` workgroups take the first.
template <int DT, int B, int SF>
__global__ __launch_bounds__(256) void quantize_rows_pair_kernel(QuantArgs P0, QuantArgs P1, unsigned wgs)
{
    const bool first = blockIdx.x < wgs;
    const QuantArgs &P = first ? P0 : P1;
    const unsigned wg = first ? blockIdx.x : blockIdx.x - wgs;
    const float g = rows_tile<DT, B, SF, NVFP4_RTN, true>(P, wg);
    if (wg == 0 && threadIdx.x == 0) *P.g_out = g;
}

// ------------------------------------------------------------------ column-blocked quantizer

// Lane tile: RPL rows x 8 columns; a workgroup covers 128 rows x 256 columns, lanes with consecutive ids stacked
// vertically, so that it reads 512 contiguous bytes (bf16) per row and writes 64 per output row.
// RPL = 16 (4 waves) does the least work per element, RPL = 8 (8 waves: a block of 16 spans two lanes) has half the serial
// chain per wave and half the registers, 512 tiles resident at once.
// bf16: what bounds a tensor of up to 512 tiles is that chain (one batch of loads, the arithmetic, the stores); larger ones have
// 16 rows, one tile per workgroup or streamed (streams()).  us, RPL = 16 / 8, dual quantizer with row-major outputs:
//                      bf16 RtN+RtN   bf16 SR+SR    MXFP4 bf16 SR+SR
//     2048 x  4096     13.9 / 11.6    18.1 / 16.0   19.7 / 16.4
//     4096 x  4096     18.2 / 15.2    25.1 / 21.9   26.9 / 23.4
//     4096 x 11008     43.6 / 43.8    56.8 / 58.4   57.2 / 57.8
//     8192 x  8192     53.9 / 57.5    67.6 / 72.3   72.0 / 75.3
// Binary32 tiles of 16 rows take 160 to 190 registers with E4M3 scales, and three workgroups per CU (768 tiles resident) where they
// stay within 168: both sides RtN, RtN columns with blocks of 64 and 128 or E8M0 scales.  They are the faster ones
//     from 257 to 512 tiles (all resident either way: the fewer instructions win)    columns, RtN duals into slabs, SwiGLU
//     from 513 to 768 (one generation of them, two of the others)                    those of up to 168 registers, columns or slabs
//     from 1025 to 1536 (two, or three as full as the others')                       RtN columns, duals into slabs, SwiGLU
// and everywhere else 8 rows are, also for MXFP4 with SR, whose 16-row tiles take 285 registers.  us, RPL = 16 / 8, with the maximum
// pass of the call (E4M3):
//                      dual RtN+RtN slabs   dual SR+SR slabs   dual SR+SR     columns RtN, block 64   columns SR, block 16   MXFP4 SR+SR slabs
//     3456 x  3072     25.7 / 26.2          31.6 / 31.1        32.6 / 31.6    23.6 / 25.0             27.6 / 29.1            36.1 / 27.4
//     2048 x 11008     41.7 / 42.5          46.8 / 47.4        48.4 / 49.4    35.7 / 40.4             45.1 / 43.4            56.0 / 43.0
//     8192 x  4096     62.1 / 57.8          67.6 / 62.3        68.9 / 62.0    53.2 / 50.6             59.5 / 56.6            78.4 / 56.3
//     4096 x 11008     74.8 / 78.5          84.3 / 83.5        88.7 / 86.9    67.5 / 70.0             80.9 / 81.4           112.2 / 84.6
//     8192 x  8192    113.5 / 107.7        118.1 / 112.6      121.5 / 114.3   97.1 / 95.9            114.3 / 104.6          155.8 / 111.7
// (with the scale preset, dual SR+SR slabs, 4096 x 11008: 56.3 / 61.5; SwiGLU 3456 x 3072: 90.7 / 98.2, 4096 x 11008 335 / 346)
constexpr int64_t PAIR_TILES = 512;  // of X and W together: where both would take 8-row lane tiles, resident at once
enum TileUse { COLUMNS, DUAL, DUAL_SLABS, SWIGLU };
static bool short_lane_tile(int dt, int block, int sf, int rnd_r, int rnd_c, TileUse use, int64_t rows, int64_t cols)
{
    const int64_t tiles = ((rows + 127) / 128) * ((cols + 255) / 256);
    if (dt == NVFP4_BF16) return tiles <= 512;
    const bool sr = rnd_c == NVFP4_SR;
    if (use == DUAL || (sf == NVFP4_SCALE_E8M0 && sr) || tiles <= 256 || tiles > 1536) return true;
    if (tiles <= 512) return use == DUAL_SLABS && sr;
    if (tiles <= 768) return !(use == COLUMNS ? !sr && (block >= 64 || sf == NVFP4_SCALE_E8M0) : use == DUAL_SLABS && rnd_r == NVFP4_RTN && !sr);
    if (tiles <= 1024) return true;
    return use == COLUMNS && sr;
}
template <int ROWS_PER_LANE>
struct ColGeom {
    static constexpr int RPL = ROWS_PER_LANE;
    static constexpr int WG_ROWS = 128, WG_COLS = 256;
    static constexpr int LANES_V = WG_ROWS / RPL;      // lanes stacked vertically
    static constexpr int LANES_H = 64 / LANES_V;       // column groups per wave
    static constexpr int WAVE_COLS = 8 * LANES_H;
    static constexpr int NT = 64 * WG_COLS / WAVE_COLS;  // threads per workgroup
};

// 16 bits of the column c of a lane's 8 in row-major element order: from draw d0 when the 8
// columns are aligned to a draw (shift = 0), else from d0 or d1.
template <bool ALIGNED>
__device__ __forceinline__ uint32_t col_bits(const u32x4 &d0, const u32x4 &d1, uint32_t shift, int c)
{
    if (ALIGNED) return sr_bits_of(d0, c);
    const uint32_t pos = shift + c;
    return pos < 8 ? sr_bits_of(d0, pos) : sr_bits_of(d1, pos - 8);
}

// Stochastic rounding of a lane's RPL x 8 tile through the hardware convert, two rows at a time
// (the byte select of the convert must be a constant, hence the recursion over row pairs).
// ALIGNED (every row holds a whole number of draws and the lane's 8 columns are one of them): ctr is the draw
// counter of row row0 + R at the lane's columns and cstep = cols / 8 the distance to the next row's, both carried
// along instead of being recomputed from 64-bit element indices for every row.
// MXS: q holds the converts' scale operands instead of multipliers.
template <int DT, int RND, bool ALIGNED, int BL, int R, bool MXS, int RPL>
__device__ __forceinline__ void col_sr_hw(const QuantArgs &P, Chunk<DT> (&v)[RPL], float (&q)[8][RPL / BL],
                                          int64_t row0, int64_t col0, uint32_t (&weven)[8][RPL / 8],
                                          uint32_t (&wodd)[8][RPL / 8], uint64_t ctr, uint64_t cstep)
{
    if constexpr (R < RPL) {
        const uint64_t e0 = (uint64_t)(row0 + R) * (uint64_t)P.cols + (uint64_t)col0;
        const uint64_t e1 = e0 + (uint64_t)P.cols;
        const u32x4 z = {0, 0, 0, 0};
        const u32x4 a0 = sr_draw(P.seed, ALIGNED ? ctr : e0 >> 3), b0 = sr_draw(P.seed, ALIGNED ? ctr + cstep : e1 >> 3);
        const u32x4 a1 = ALIGNED ? z : sr_draw(P.seed, (e0 >> 3) + 1);
        const u32x4 b1 = ALIGNED ? z : sr_draw(P.seed, (e1 >> 3) + 1);
        const uint32_t sa = (uint32_t)e0 & 7u, sb = (uint32_t)e1 & 7u;
        if constexpr (ALIGNED) {
            // (odd rows are converted into the low nibbles of wodd; the caller shifts them up)
            const uint32_t na[4] = {~a0.x, ~a0.y, ~a0.z, ~a0.w}, nb[4] = {~b0.x, ~b0.y, ~b0.z, ~b0.w};
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                if constexpr (MXS) {
                    weven[c][R / 8] = mx_sr_elem0<DT, (R % 8) / 2>(weven[c][R / 8], v[R], c, sr_seed0(na[c / 2], c & 1), q[c][R / BL]);
                    wodd[c][R / 8] = mx_sr_elem0<DT, (R % 8) / 2>(wodd[c][R / 8], v[R + 1], c, sr_seed0(nb[c / 2], c & 1), q[c][(R + 1) / BL]);
                } else {
                    weven[c][R / 8] = sr_elem0<(R % 8) / 2>(weven[c][R / 8], v[R].get(c) * q[c][R / BL], sr_seed0(na[c / 2], c & 1));
                    wodd[c][R / 8] = sr_elem0<(R % 8) / 2>(wodd[c][R / 8], v[R + 1].get(c) * q[c][(R + 1) / BL], sr_seed0(nb[c / 2], c & 1));
                }
            }
        } else {
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                weven[c][R / 8] = sr_elem_hw<0, (R % 8) / 2>(weven[c][R / 8], v[R].get(c) * q[c][R / BL],
                                                             col_bits<ALIGNED>(a0, a1, sa, c));
                wodd[c][R / 8] = sr_elem_hw<1, (R % 8) / 2>(wodd[c][R / 8], v[R + 1].get(c) * q[c][(R + 1) / BL],
                                                            col_bits<ALIGNED>(b0, b1, sb, c));
            }
        }
        col_sr_hw<DT, RND, ALIGNED, BL, R + 2, MXS, RPL>(P, v, q, row0, col0, weven, wodd, ctr + 2 * cstep, cstep);
    }
}

// Round-to-nearest of a lane's RPL x 8 tile through the hardware convert: rows R and R + 1 of a column share a
// byte, which the convert writes in place (its byte select must be a constant, hence the recursion over row pairs).
template <int DT, int BL, int R, bool MXS, int RPL>
__device__ __forceinline__ void col_rtn_hw(Chunk<DT> (&v)[RPL], float (&q)[8][RPL / BL], uint32_t (&words)[8][RPL / 8])
{
    if constexpr (R < RPL) {
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            if constexpr (MXS)
                words[c][R / 8] = mx_rtn_rows<DT, (R % 8) / 2>(words[c][R / 8], v[R], v[R + 1], c, q[c][R / BL]);
            else
                words[c][R / 8] = quant_pair_hw<(R % 8) / 2>(words[c][R / 8], v[R].get(c), v[R + 1].get(c), q[c][R / BL]);
        }
        col_rtn_hw<DT, BL, R + 2, MXS, RPL>(v, q, words);
    }
}

// Where a lane's column-blocked outputs go in the slab layout: column c of the lane stores its RPL / 2 code bytes at
// codes + 512 c and its scale byte at scales + 64 c (blocks of 16) or, from the lowest of the stacked lanes,
// the column's four scale bytes at scales + 32 c (blocks of 32); the lane index is folded into the two pointers.
struct ColSlab {
    uint8_t *codes, *scales;
};

// the codes of a lane's column: RPL rows, one nibble each
template <int RPL>
__device__ __forceinline__ void store_codes(uint8_t *p, const uint32_t (&w)[RPL / 8])
{
    if constexpr (RPL == 16) store8_stream(p, w[0], w[1]);
    else store4_stream(p, w[0]);
}

template <int DT, int B, int SF, int RND, bool HW, bool ALIGNED, int RPL>
__device__ __forceinline__ void cols_tile(const QuantArgs &P, Chunk<DT> (&v)[RPL], float g, float k, int64_t row0,
                                          int64_t col0, int ncol, int lv, const ColSlab *slab = nullptr);

// ALIGNED: cols is a multiple of 8, so the 8 columns of a lane share one random draw per row.
template <int DT, int B, int SF, int RND, bool HW, bool ALIGNED, int RPL>
__global__ __launch_bounds__(ColGeom<RPL>::NT) void quantize_cols_kernel(QuantArgs P)
{
    using G = ColGeom<RPL>;

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int lv = lane % G::LANES_V, lh = lane / G::LANES_V;
    const int64_t row0 = (int64_t)blockIdx.y * G::WG_ROWS + lv * RPL;
    const int64_t col0 = (int64_t)blockIdx.x * G::WG_COLS + wave * G::WAVE_COLS + lh * 8;
    const int ncol = col0 >= P.cols ? 0 : (P.cols - col0 >= 8 ? 8 : (int)(P.cols - col0));

    Chunk<DT> v[RPL];
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
        const int64_t i = row0 + r;
        if (i < P.rows && ncol == 8)
            v[r].template load<true>(P.x, i * P.ld + col0);
        else if (i < P.rows && ncol > 0)
            v[r].load_partial(P.x, i * P.ld + col0, ncol);
        else
            v[r].zero();
    }
    // (tensors small enough to take their maximum here have few tiles, hence 8 rows per lane; the forms that only 16 rows serve aside)
    const float g = resolve_g<DT, G::NT, SF == NVFP4_SCALE_E4M3 && (RPL == 8 || !HW || !ALIGNED)>(P);
    const float k = 1.0f / (6.0f * g);
    build_qtab<SF, HW>(g);
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *P.g_out = g;
    cols_tile<DT, B, SF, RND, HW, ALIGNED, RPL>(P, v, g, k, row0, col0, ncol, lv);
}

// The column-blocked quantization of one lane tile (RPL rows x 8 columns in v): block maxima,
// scale bytes, codes, and the stores into the transposed outputs.
template <int DT, int B, int SF, int RND, bool HW, bool ALIGNED, int RPL>
__device__ __forceinline__ void cols_tile(const QuantArgs &P, Chunk<DT> (&v)[RPL], float g, float k, int64_t row0,
                                          int64_t col0, int ncol, int lv, const ColSlab *slab)
{
    using G = ColGeom<RPL>;
    constexpr int BL = B < RPL ? B : RPL;        // rows of one block held by this lane
    constexpr int NB = RPL / BL;                 // blocks (or block parts) per lane per column
    constexpr int LPB = B / BL;                  // lanes sharing one block
    const int64_t rows_half = P.rows >> 1;
    const int64_t nblk = P.rows / B;

    // pass 1: block maxima -> scale bytes and multipliers, per column and per block part
    // MXS: the multipliers are replaced by the converts' scale operands, and an unaligned tile (whose stochastic
    // rounding goes through the two-slot form) keeps multipliers.
    constexpr bool MXS = HW && SF == NVFP4_SCALE_E8M0 && (ALIGNED || RND == NVFP4_RTN);
    float q[8][NB];
    uint32_t sbytes[8][NB];
    if constexpr (MXS && DT == NVFP4_BF16) {
        // maxima on the packed bf16 magnitudes, two columns per instruction
#pragma unroll
        for (int cp = 0; cp < 4; ++cp) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                uint32_t m = 0;
#pragma unroll
                for (int r = 0; r < BL; ++r) m = pk_umax16(m, v[nb * BL + r].word(cp) & 0x7FFF7FFFu);
                const float a0 = group_max<LPB>(pk_even(m)), a1 = group_max<LPB>(pk_odd(m));
                sbytes[2 * cp][nb] = block_scale<SF, HW, false>(a0, g, k, &q[2 * cp][nb]);
                sbytes[2 * cp + 1][nb] = block_scale<SF, HW, false>(a1, g, k, &q[2 * cp + 1][nb]);
            }
        }
    } else {
#pragma unroll
        for (int c = 0; c < 8; ++c) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                float a = 0.0f;
#pragma unroll
                for (int r = 0; r < BL; ++r) a = fmaxf(a, fabsf(v[nb * BL + r].get(c)));
                a = group_max<LPB>(a);
                sbytes[c][nb] = block_scale<SF, HW, HW && SF == NVFP4_SCALE_E4M3>(a, g, k, &q[c][nb]);
            }
        }
    }
    if constexpr (MXS) {
#pragma unroll
        for (int c = 0; c < 8; ++c)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) q[c][nb] = mx_scale_operand(sbytes[c][nb]);
    }

    // (the empty asm makes the compiler unpack the raw registers again in pass 2 instead of
    // keeping 128 unpacked floats alive across the passes)
#pragma unroll
    for (int r = 0; r < RPL; ++r) v[r].launder();

    // pass 2: codes.  words[c][w] collects rows 8w..8w+7 of column c, one nibble per row.
    uint32_t words[8][RPL / 8];
#pragma unroll
    for (int c = 0; c < 8; ++c)
#pragma unroll
        for (int w = 0; w < RPL / 8; ++w) words[c][w] = 0;

    if (RND == NVFP4_RTN && HW) {
        col_rtn_hw<DT, BL, 0, MXS, RPL>(v, q, words);
    } else if (RND == NVFP4_SR && HW) {
        // rows 2p and 2p+1 of a column share a byte: even rows go through slot 0, odd rows
        // through slot 1 of the convert, into two sets of words that are OR-ed at the end
        uint32_t wodd[8][RPL / 8];
#pragma unroll
        for (int c = 0; c < 8; ++c)
#pragma unroll
            for (int w = 0; w < RPL / 8; ++w) wodd[c][w] = 0;
        const uint64_t cstep = (uint64_t)P.cols >> 3;
        col_sr_hw<DT, RND, ALIGNED, BL, 0, MXS, RPL>(P, v, q, row0, col0, words, wodd, (uint64_t)row0 * cstep + ((uint64_t)col0 >> 3), cstep);
#pragma unroll
        for (int c = 0; c < 8; ++c)
#pragma unroll
            for (int w = 0; w < RPL / 8; ++w) words[c][w] |= ALIGNED ? wodd[c][w] << 4 : wodd[c][w];
    } else {
        // the 8 columns of a lane are 8 consecutive elements of a row; their random bits come
        // from one draw when that group is aligned in the row-major numbering, else from two
#pragma clang loop unroll(full)
        for (int r = 0; r < RPL; ++r) {
            u32x4 d0 = {0, 0, 0, 0}, d1 = {0, 0, 0, 0};
            uint32_t shift = 0;
            if (RND == NVFP4_SR) {
                const uint64_t e0 = (uint64_t)(row0 + r) * (uint64_t)P.cols + (uint64_t)col0;
                d0 = sr_draw(P.seed, e0 >> 3);
                shift = (uint32_t)e0 & 7u;
                if (!ALIGNED) d1 = sr_draw(P.seed, (e0 >> 3) + 1);
            }
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                uint32_t u16 = 0;
                if (RND == NVFP4_SR) {
                    if (ALIGNED) {
                        u16 = sr_bits_of(d0, c);
                    } else {
                        const uint32_t pos = shift + c;
                        u16 = pos < 8 ? sr_bits_of(d0, pos) : sr_bits_of(d1, pos - 8);
                    }
                }
                words[c][r / 8] |= quant_elem<RND>(v[r].get(c), q[c][r / BL], u16) << (4 * (r % 8));
            }
        }
    }

    // Scale bytes, row-major [cols, rows / B]: the lanes stacked vertically hold consecutive bytes of a column's
    // row (blocks of 16: 8 per workgroup tile; blocks of 32: 4), each in LPB adjacent lanes.  Where
    // the rows allow, four bytes are gathered into the lowest of their lanes through DPP row shifts (lane + n; every
    // lane takes part) and leave as one aligned dword instead of single bytes.
    constexpr bool GATHER = NB == 1 && (B == 16 || B == 32);
    constexpr int GSTEP = LPB;  // lanes between consecutive bytes
    uint32_t sw[8];
    bool wide = false, owner = false;
    if constexpr (GATHER) {
        // (the whole 128-row tile inside the tensor, whole dwords per tile, aligned rows of the scale matrix)
        wide = (nblk & 3) == 0 && (reinterpret_cast<uintptr_t>(P.scales) & 3) == 0 && (row0 - lv * RPL) + G::WG_ROWS <= P.rows;
        owner = (lv & (4 * GSTEP - 1)) == 0;  // blocks of 16: two of the stacked lanes; blocks of 32: the lowest
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            sw[c] = sbytes[c][0];
            sw[c] |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)sw[c], 0x100 + GSTEP, 0xF, 0xF, true) << 8;       // lane + GSTEP
            sw[c] |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)sw[c], 0x100 + 2 * GSTEP, 0xF, 0xF, true) << 16;  // lanes + 2, + 3 GSTEP
        }
    }

    if (slab != nullptr) {
        // slab layout (the caller guarantees a lane tile entirely inside the tensor or entirely outside, blocks of
        // 16 or 32): the stacked lanes of a column write its 64 code bytes of this K tile, the lane groups of two
        // (four) waves 512 contiguous ones
        if (ncol == 8) {
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                store_codes<RPL>(slab->codes + 512 * c, words[c]);
                if (B == 16) {
                    if (lv % LPB == 0) slab->scales[64 * c] = (uint8_t)sbytes[c][0];
                } else if (GATHER) {
                    // blocks of 32: the lowest of the stacked lanes holds the column's four bytes of this K tile
                    if (owner) *reinterpret_cast<uint32_t *>(slab->scales + 32 * c) = sw[c];
                }
            }
        }
        return;
    }
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        if (c < ncol) {
            const int64_t col = col0 + c;
            if (row0 < P.rows) store_codes<RPL>(P.codes + col * rows_half + (row0 >> 1), words[c]);
            if (GATHER && wide) {
                if (owner) *reinterpret_cast<uint32_t *>(P.scales + col * nblk + row0 / B) = sw[c];
            } else if (lv % LPB == 0) {
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    if (row0 + nb * BL < P.rows)
                        P.scales[col * nblk + (row0 + nb * BL) / B] = (uint8_t)sbytes[c][nb];
            }
        }
    }
}

// ------------------------------------------------------------------ bf16 tensors of many tiles: the next tile in flight

// The 16 x 8 lane tiles of one wave, one workgroup tile after the other, each requested before the one in hand is worked on.  The kernels
// above load, compute and store, one tile per wave: two generations of waves that do each of the three at the same time, 70 % of a
// wave's life spent waiting for memory.  The first LR rows of the next tile go from memory straight into a piece of LDS that only
// this wave uses (global_load_lds: 1 KB per row, 16 bytes per lane, read back by the lane that fetched them: no barriers), the others
// into registers.  Whole tiles in registers take 240 and more of them, whole tiles in LDS leave room for two workgroups per CU.
template <int LR>
struct TileStream {
    using G = ColGeom<16>;
    static constexpr int LDS_BYTES = G::NT / 64 * LR * 1024;
    const uint8_t *mine;  // this lane's 16 bytes of row 0
    uint32_t lds_wave;    // LDS address of the wave's piece
    int lv, lcol;         // the lane's tile: rows 16 lv .. of the workgroup tile, columns lcol ..
    Chunk<NVFP4_BF16> rest[16 - LR];

    __device__ __forceinline__ TileStream(uint8_t *lds)
    {
        typedef __attribute__((address_space(3))) void *lds_ptr_t;
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        mine = lds + wave * (LR * 1024) + (threadIdx.x & 63) * 16;
        lds_wave = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_ptr_t)lds + wave * (LR * 1024));
        place(threadIdx.x);
    }
    // (also once per tile, from a thread index that the compiler cannot trace back: what derives from it is then computed again instead of
    // kept from tile to tile, dual RtN+RtN with 15 rows in LDS 186 -> 116 registers)
    __device__ __forceinline__ void place(int tid)
    {
        lv = (tid & 63) % G::LANES_V;
        lcol = (tid >> 6) * G::WAVE_COLS + (tid & 63) / G::LANES_V * 8;
    }
    // (rows is a multiple of 16 and cols of 8: a lane tile is inside or outside as a whole)
    __device__ __forceinline__ bool inside(const QuantArgs &P, int tx, int ty) const
    {
        return (int64_t)ty * G::WG_ROWS + lv * 16 < P.rows && (int64_t)tx * G::WG_COLS + lcol < P.cols;
    }
    // A lane outside the tensor fetches the workgroup tile's first lane tile, which is inside.
    __device__ __forceinline__ void request(const QuantArgs &P, int tx, int ty)
    {
        const uint16_t *base = reinterpret_cast<const uint16_t *>(P.x) + (int64_t)ty * G::WG_ROWS * P.ld + (int64_t)tx * G::WG_COLS;
        const uint32_t off = inside(P, tx, ty) ? (uint32_t)(lv * 16 * P.ld + lcol) : 0u;  // elements; the byte offset has 32 bits (streams())
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            if (r < LR)
                asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" : : "s"(lds_wave + r * 1024), "v"(off * 2u), "s"(base) : "memory", "m0");
            else
                rest[r < LR ? 0 : r - LR].template load<true>(base, off);
            base += P.ld;
        }
    }
    // The tile requested last; its LDS may be written again afterwards.  (Waits for the stores of the tile before as well: counting those
    // out changed no time.)
    __device__ __forceinline__ void take(bool live, Chunk<NVFP4_BF16> (&v)[16])
    {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            if (r < LR) v[r].raw = *reinterpret_cast<const uint4 *>(mine + r * 1024);
            else v[r] = rest[r < LR ? 0 : r - LR];
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (!live) {
#pragma unroll
            for (int r = 0; r < 16; ++r) v[r].zero();
        }
    }
};
// Workgroups per CU, and rows in LDS that leave room for them: three need 168 registers or fewer, and 53 KB of LDS each, of which the
// dual kernel's own output takes 18.
constexpr int STREAM_WGS = 3, COLS_LDS_ROWS = 12, DUAL_LDS_ROWS = 8;

template <int B, int SF, int RND>
__global__ __launch_bounds__(ColGeom<16>::NT, STREAM_WGS) void quantize_cols_stream_kernel(QuantArgs P, unsigned gx, unsigned tiles)
{
    using G = ColGeom<16>;
    extern __shared__ __attribute__((aligned(16))) uint8_t stream_lds[];
    TileStream<COLS_LDS_ROWS> T(stream_lds);
    unsigned id = blockIdx.x;
    T.request(P, (int)(id % gx), (int)(id / gx));
    const float g = resolve_g<NVFP4_BF16, G::NT, false>(P);
    const float k = 1.0f / (6.0f * g);
    build_qtab<SF, true>(g);
    if (id == 0 && threadIdx.x == 0) *P.g_out = g;
    for (bool more = true; more;) {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        T.place(tid);
        const int tx = (int)(id % gx), ty = (int)(id / gx);
        const bool live = T.inside(P, tx, ty);
        Chunk<NVFP4_BF16> v[16];
        T.take(live, v);
        id += gridDim.x;
        more = id < tiles;
        if (more) T.request(P, (int)(id % gx), (int)(id / gx));
        cols_tile<NVFP4_BF16, B, SF, RND, true, true, 16>(P, v, g, k, (int64_t)ty * G::WG_ROWS + T.lv * 16, (int64_t)tx * G::WG_COLS + T.lcol,
                                                         live ? 8 : 0, T.lv);
    }
}

// ------------------------------------------------------------------ SwiGLU backward as a tile source

// Where the dual quantizer's tile comes from: a tensor in memory, or dG / dU of the SwiGLU backward evaluated from
// dH, G, U while loading (nvfp4_math.h: swiglu_bwd_elem), rounded to the element type like a stored tensor would be.
enum { SRC_TENSOR = 0, SRC_SWIGLU_DG = 1, SRC_SWIGLU_DU = 2 };

// 8 consecutive elements of dG (WHICH = SRC_SWIGLU_DG), of dU (SRC_SWIGLU_DU), or both (0: og and ou)
template <int DT, int WHICH>
__device__ __forceinline__ void swiglu_chunk(const void *dH, const void *G, const void *U, int64_t off, Chunk<DT> *og, Chunk<DT> *ou)
{
    Chunk<DT> h, g, u;
    // (cacheable loads: the three tensors are read by the maximum pass and by both quantizer passes)
    h.template load<false>(dH, off);
    g.template load<false>(G, off);
    u.template load<false>(U, off);
    float rg[8], ru[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) swiglu_bwd_elem(h.get(t), g.get(t), u.get(t), &rg[t], &ru[t]);
    if (WHICH != SRC_SWIGLU_DU) og->set(rg);
    if (WHICH != SRC_SWIGLU_DG) ou->set(ru);
}

// max|dG| and max|dU| (of the values as rounded to the element type) over n = 8 * nchunk elements: one partial
// maximum of each per workgroup, as amax_dense_kernel leaves them for a tensor in memory.
// STORE: the two results are also written out as tensors (dG_out, dU_out), for quantizer passes that read them back
// instead of evaluating them again.
template <int DT, bool STORE>
__global__ __launch_bounds__(1024) void swiglu_amax_kernel(const void *dH, const void *G, const void *U, int64_t n,
                                                           uint32_t *part_g, uint32_t *part_u, void *dG_out, void *dU_out)
{
    const int64_t nchunk = n >> 3;
    const int64_t stride = (int64_t)gridDim.x * (1024 * 2);
    float ag = 0.0f, au = 0.0f;
    for (int64_t base = (int64_t)blockIdx.x * (1024 * 2) + threadIdx.x; base < nchunk; base += stride) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int64_t c = base + k * 1024;
            if (c < nchunk) {
                Chunk<DT> cg, cu;
                swiglu_chunk<DT, 0>(dH, G, U, c * 8, &cg, &cu);
                if (STORE) {
                    cg.store(dG_out, c * 8);
                    cu.store(dU_out, c * 8);
                }
                ag = fmaxf(ag, chunk_amax(cg));
                au = fmaxf(au, chunk_amax(cu));
            }
        }
    }
    ag = group_max<16>(ag);
    au = group_max<16>(au);
    __shared__ uint32_t pg[64], pu[64];
    if ((threadIdx.x & 15) == 0) {
        pg[threadIdx.x >> 4] = f2u(ag);
        pu[threadIdx.x >> 4] = f2u(au);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t mg = 0, mu = 0;
#pragma unroll
        for (int t = 0; t < 64; ++t) {
            mg = umax(mg, pg[t]);
            mu = umax(mu, pu[t]);
        }
        part_g[blockIdx.x] = mg;
        part_u[blockIdx.x] = mu;
    }
}

// dG and dU stored as tensors (the unfused form of the same step): n = 8 * nchunk elements.
template <int DT>
__global__ __launch_bounds__(256) void swiglu_bwd_kernel(const void *dH, const void *G, const void *U, int64_t n, void *dG, void *dU)
{
    const int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (c >= (n >> 3)) return;
    Chunk<DT> cg, cu;
    swiglu_chunk<DT, 0>(dH, G, U, c * 8, &cg, &cu);
    cg.store(dG, c * 8);
    cu.store(dU, c * 8);
}

hipError_t launch_swiglu_bwd(const void *dH, const void *G, const void *U, int dt, int64_t n, void *dG, void *dU, hipStream_t st)
{
    const unsigned grid = (unsigned)(((n >> 3) + 255) / 256);
    if (grid == 0) return hipSuccess;
    if (dt == NVFP4_BF16)
        hipLaunchKernelGGL(swiglu_bwd_kernel<NVFP4_BF16>, dim3(grid), dim3(256), 0, st, dH, G, U, n, dG, dU);
    else
        hipLaunchKernelGGL(swiglu_bwd_kernel<NVFP4_F32>, dim3(grid), dim3(256), 0, st, dH, G, U, n, dG, dU);
    return hipGetLastError();
}

// ------------------------------------------------------------------ both orientations in one pass

// Eqs. 5-6 use the output gradient twice, blocked along N for dX and along M for dW; Eqs. 4-5
// do the same with W.  This kernel reads the tensor once and writes both quantizations, each
// identical to what the single-orientation kernels produce (same scale rule, same convert, same
// draws: seed_r for the row-blocked output, P.seed for the column-blocked one), each with its
// own rounding mode (X is needed round-to-nearest along K for Eq. 4 and stochastically rounded
// along M for Eq. 6).
// Geometry of the columns kernel (lane = RPL rows x 8 columns, workgroup = 128 rows x 256
// columns).  A row block of B = 16 or 32 columns spans 2 or 4 lanes that are LANES_V apart in the wave
// (DPP row rotate / lane swaps for the maximum).  The row-blocked codes of the tile (128 rows x 128
// bytes) and its scale bytes are staged in LDS and written out 16 bytes per lane, so both outputs
// leave in full lines although the lanes hold the data column-wise.
// Host guarantees: rows % B == 0, cols % B == 0 (so a lane's RPL x 8 tile is entirely inside or
// outside the tensor), 16-byte aligned rows of x.
// One workgroup tile (128 rows x 256 columns at tile coordinates tx, ty; the lane's RPL x 8 part of it in v) through
// both quantizers and out to memory.  Every thread of the workgroup must call it (barriers inside).
template <int DT, int B, int SF, int RND_R, int RND_C, int RPL>
__device__ __forceinline__ void dual_tile(const DualArgs &D, Chunk<DT> (&v)[RPL], float g, float k, int tx, int ty, const int tid,
                                          uint32_t *lds_codes, uint8_t *lds_scales)
{
    using G = ColGeom<RPL>;
    constexpr int LPBR = B / 8;                  // lanes sharing one row block
    constexpr bool MXS = SF == NVFP4_SCALE_E8M0;  // block scale as the convert's scale operand
    constexpr int ROW_BYTES = G::WG_COLS / 2;    // 128 code bytes per tile row
    constexpr int ROW_SC = G::WG_COLS / B;       // scale bytes per tile row
    const QuantArgs &P = D.c;
    const int lane = tid & 63, wave = tid >> 6;
    const int lv = lane % G::LANES_V, lh = lane / G::LANES_V;
    const int64_t wrow0 = (int64_t)ty * G::WG_ROWS, wcol0 = (int64_t)tx * G::WG_COLS;
    const int64_t row0 = wrow0 + lv * RPL;
    const int64_t col0 = wcol0 + wave * G::WAVE_COLS + lh * 8;
    const bool inside = row0 < P.rows && col0 < P.cols;

    // row-blocked side: one block scale and 8 codes per row of the lane tile
    const uint64_t cstep_r = (uint64_t)P.cols >> 3;
    uint64_t ctr_r = (uint64_t)row0 * cstep_r + ((uint64_t)col0 >> 3);
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
        float a = MXS ? chunk_amax_packed(v[r]) : chunk_amax(v[r]);
        a = lane_pair_max<G::LANES_V>(a);  // the neighbouring column group
        if (LPBR == 4) a = lane_pair_max<2 * G::LANES_V>(a);
        float q;
        const uint32_t sbyte = block_scale<SF, true, SF == NVFP4_SCALE_E4M3>(a, g, k, &q);
        if (MXS) q = mx_scale_operand(sbyte);
        // (cols is a multiple of the block, col0 of 8: the lane's 8 columns are one draw, cols / 8 draws per row)
        const uint32_t packed = chunk_codes_hw<DT, RND_R, MXS>(v[r], q, D.seed_r, ctr_r);
        ctr_r += cstep_r;
        // tile row R = RPL lv + r holds 32 dwords; dword w is stored at w ^ (4 lv % 32): the
        // 16-byte chunk c of the row sits at chunk c ^ (lv % 8), which spreads the rows a wave writes at a
        // time over the banks
        const int R = lv * RPL + r;
        lds_codes[R * (ROW_BYTES / 4) + ((wave * G::LANES_H + lh) ^ ((lv & 7) << 2))] = packed;
        if ((lh & (LPBR - 1)) == 0) lds_scales[R * 16 + (wave * G::WAVE_COLS + lh * 8) / B] = (uint8_t)sbyte;
    }

    // (unpack the raw registers again below instead of keeping 128 floats alive)
#pragma unroll
    for (int r = 0; r < RPL; ++r) v[r].launder();

    // column-blocked side: exactly the columns kernel's tile.  In the slab layout the workgroup's 256 columns are
    // one tile of operand rows and its 128 rows one K tile: it fills exactly one slab.
    ColSlab cs;
    if (D.slab_c) {
        const int64_t slab = (int64_t)tx * (P.rows / SLAB_K) + ty;
        // (tile column 64 w + 8 j + c sits at position 64 w + 8 c + j; this lane's column group is 8 w + j)
        const int cg = wave * G::LANES_H + lh, w = cg >> 3, j = cg & 7;
        cs.codes = P.codes + slab * SLAB_CODE_BYTES + w * 4096 + j * 64 + lv * (RPL / 2);
        cs.scales = B == 16 ? P.scales + slab * SLAB_SCALE_BYTES + w * 512 + j * 8 + lv * RPL / 16
                            : P.scales + slab * SLAB_MX_SCALE_BYTES + w * 256 + j * 4;
    }
    cols_tile<DT, B, SF, RND_C, true, true, RPL>(P, v, g, k, row0, col0, inside ? 8 : 0, lv, D.slab_c ? &cs : nullptr);

    __syncthreads();
    if (D.slab_r) {
        // slab layout: the tile is rows (wrow0 % 256) .. + 127 of two slabs (K tiles 2 tx and + 1 of row
        // tile wrow0 / 256).  Threads walk the slab positions q; position q holds tile row slab_row(q).
        const int64_t nkt = P.cols / SLAB_K;
        const int64_t slab0 = (wrow0 / SLAB_ROWS) * nkt + 2 * (int64_t)tx;
        const int half = (int)(wrow0 & 128);
#pragma unroll
        for (int i = 0; i < 1024 / G::NT; ++i) {
            const int id = tid + G::NT * i, q = id >> 3, c = id & 7, R = slab_row(q);
            if (wrow0 + R < P.rows && wcol0 + c * 32 < P.cols) {
                const uint4 w = *reinterpret_cast<const uint4 *>(&lds_codes[R * (ROW_BYTES / 4) + ((c ^ (R / RPL & 7)) << 2)]);
                const u32x4_t o = {w.x, w.y, w.z, w.w};
                __builtin_nontemporal_store(o, reinterpret_cast<u32x4_t *>(D.codes_r + (slab0 + (c >> 2)) * SLAB_CODE_BYTES + (half + q) * 64 + (c & 3) * 16));
            }
        }
        if (tid < G::WG_ROWS) {
            const int q = tid, R = slab_row(q);
            if (wrow0 + R < P.rows) {
                const uint32_t *src = reinterpret_cast<const uint32_t *>(&lds_scales[R * 16]);
                if (B == 16) {
                    uint8_t *dst = D.scales_r + slab0 * SLAB_SCALE_BYTES + (half + q) * 8;
                    store8_stream(dst, src[0], src[1]);
                    if (wcol0 + 128 < P.cols) store8_stream(dst + SLAB_SCALE_BYTES, src[2], src[3]);
                } else {
                    // blocks of 32: four bytes per row and K tile
                    uint8_t *dst = D.scales_r + slab0 * SLAB_MX_SCALE_BYTES + (half + q) * 4;
                    store4_stream(dst, src[0]);
                    if (wcol0 + 128 < P.cols) store4_stream(dst + SLAB_MX_SCALE_BYTES, src[1]);
                }
            }
        }
        return;
    }
    const int64_t cpr = P.cols >> 1;
    const bool wide = (cpr & 15) == 0;  // rows of the code matrix are 16-byte aligned
    if (!D.slab_r) {
#pragma unroll
        for (int i = 0; i < 1024 / G::NT; ++i) {
            const int id = tid + G::NT * i, R = id >> 3, c = id & 7;
            const int64_t row = wrow0 + R, col = wcol0 + c * 32;
            if (row < P.rows && col < P.cols) {
                const uint4 w = *reinterpret_cast<const uint4 *>(&lds_codes[R * (ROW_BYTES / 4) + ((c ^ (R / RPL & 7)) << 2)]);
                uint8_t *dst = D.codes_r + row * cpr + (col >> 1);
                if (col + 32 <= P.cols && wide) {
                    const u32x4_t o = {w.x, w.y, w.z, w.w};
                    __builtin_nontemporal_store(o, reinterpret_cast<u32x4_t *>(dst));
                } else {
                    store8_stream(dst, w.x, w.y);
                    if (col + 32 <= P.cols) store8_stream(dst + 8, w.z, w.w);
                }
            }
        }
    }
    if (tid < G::WG_ROWS) {
        const int R = tid;
        const int64_t row = wrow0 + R, nsc = P.cols / B, s0 = wcol0 / B;
        if (row < P.rows && s0 < nsc) {
            uint8_t *dst = D.scales_r + row * nsc + s0;
            const uint32_t *src = reinterpret_cast<const uint32_t *>(&lds_scales[R * 16]);
            if (s0 + ROW_SC <= nsc && nsc % ROW_SC == 0) {
                store8_stream(dst, src[0], src[1]);
                if (ROW_SC == 16) store8_stream(dst + 8, src[2], src[3]);
            } else {
                const int n = (int)(nsc - s0 < ROW_SC ? nsc - s0 : ROW_SC);
                for (int j = 0; j < n; ++j) dst[j] = lds_scales[R * 16 + j];
            }
        }
    }
}

struct DualLds {
    uint32_t codes[128 * 128 / 4];
    uint8_t scales[128 * 16];
};
template <int DT, int B, int SF, int RND_R, int RND_C, int RPL, int SRC>
__device__ __forceinline__ void dual_wg(const DualArgs &D, int tx, int ty, DualLds &lds)
{
    using G = ColGeom<RPL>;
    static_assert(B == 16 || B == 32, "row blocks must fit the column groups of a wave");
    const QuantArgs &P = D.c;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int lv = lane % G::LANES_V, lh = lane / G::LANES_V;
    const int64_t row0 = (int64_t)ty * G::WG_ROWS + lv * RPL;
    const int64_t col0 = (int64_t)tx * G::WG_COLS + wave * G::WAVE_COLS + lh * 8;
    const bool inside = row0 < P.rows && col0 < P.cols;

    Chunk<DT> v[RPL];
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
        if (!inside)
            v[r].zero();
        else if (SRC == SRC_TENSOR)
            v[r].template load<true>(P.x, (row0 + r) * P.ld + col0);
        else
            swiglu_chunk<DT, SRC>(P.x, D.src_g, D.src_u, (row0 + r) * P.ld + col0, &v[r], &v[r]);
    }

    const float g = resolve_g<DT, G::NT, SF == NVFP4_SCALE_E4M3 && RPL == 8 && SRC == SRC_TENSOR>(P);
    const float k = 1.0f / (6.0f * g);
    build_qtab<SF, true>(g);
    if (tx == 0 && ty == 0 && threadIdx.x == 0) {
        // (a `saved` buffer that is not the one this call expects poisons the scale the GEMMs will multiply by)
        const float g_gemm = tag_apply(D.tag) ? g : __builtin_nanf("");
        *P.g_out = g_gemm;
        if (D.g_out2) *D.g_out2 = g_gemm;
    }
    dual_tile<DT, B, SF, RND_R, RND_C, RPL>(D, v, g, k, tx, ty, (int)threadIdx.x, lds.codes, lds.scales);
}

// Waves per SIMD asked of the compiler with 16 rows per lane, where the registers lie within a few of the line (128 and 168 registers);
// 0: as they come.
constexpr int dual_waves(int dt, int b, int sf, int rnd_r, int rnd_c, int rpl)
{
    if (rpl != 16 || (b == 16 && sf == NVFP4_SCALE_E8M0)) return 0;
    return dt == NVFP4_BF16 ? 4 : rnd_r == NVFP4_RTN && rnd_c == NVFP4_RTN ? 3 : 0;
}
template <int DT, int B, int SF, int RND_R, int RND_C, int RPL, int SRC = SRC_TENSOR>
__global__ __launch_bounds__(ColGeom<RPL>::NT, dual_waves(DT, B, SF, RND_R, RND_C, RPL)) void quantize_dual_kernel(DualArgs D)
{
    __shared__ __align__(16) DualLds lds;
    dual_wg<DT, B, SF, RND_R, RND_C, RPL, SRC>(D, (int)blockIdx.x, (int)blockIdx.y, lds);
}

template <int B, int SF, int RND_R, int RND_C>
__global__ __launch_bounds__(ColGeom<16>::NT, STREAM_WGS) void quantize_dual_stream_kernel(DualArgs D, unsigned gx, unsigned tiles)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t stream_lds[];
    __shared__ __align__(16) DualLds lds;
    const QuantArgs &P = D.c;
    TileStream<DUAL_LDS_ROWS> T(stream_lds);
    unsigned id = blockIdx.x;
    T.request(P, (int)(id % gx), (int)(id / gx));
    const float g = resolve_g<NVFP4_BF16, ColGeom<16>::NT, false>(P);
    const float k = 1.0f / (6.0f * g);
    build_qtab<SF, true>(g);
    if (id == 0 && threadIdx.x == 0) {
        // (a `saved` buffer that is not the one this call expects poisons the scale the GEMMs will multiply by)
        const float g_gemm = tag_apply(D.tag) ? g : __builtin_nanf("");
        *P.g_out = g_gemm;
        if (D.g_out2) *D.g_out2 = g_gemm;
    }
    for (bool more = true; more;) {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        T.place(tid);
        const int tx = (int)(id % gx), ty = (int)(id / gx);
        Chunk<NVFP4_BF16> v[16];
        T.take(T.inside(P, tx, ty), v);
        __syncthreads();  // (every wave has stored its share of the codes that the tile before left in lds)
        id += gridDim.x;
        more = id < tiles;
        if (more) T.request(P, (int)(id % gx), (int)(id / gx));
        dual_tile<NVFP4_BF16, B, SF, RND_R, RND_C, 16>(D, v, g, k, tx, ty, tid, lds.codes, lds.scales);
    }
}

// X (round to nearest / stochastic) and W (round to nearest) of a forward call that saves both, in one launch: the first
// `tiles` workgroups take X.
template <int DT, int B, int SF>
__global__ __launch_bounds__(ColGeom<8>::NT) void quantize_dual_pair_kernel(DualArgs X, DualArgs W, unsigned tiles, unsigned tx_x, unsigned tx_w)
{
    __shared__ __align__(16) DualLds lds;
    if (blockIdx.x < tiles) {
        dual_wg<DT, B, SF, NVFP4_RTN, NVFP4_SR, 8, SRC_TENSOR>(X, (int)(blockIdx.x % tx_x), (int)(blockIdx.x / tx_x), lds);
    } else {
        const unsigned id = blockIdx.x - tiles;
        dual_wg<DT, B, SF, NVFP4_RTN, NVFP4_RTN, 8, SRC_TENSOR>(W, (int)(id % tx_w), (int)(id / tx_w), lds);
    }
}

// The same for bf16 tensors of many tiles: one run of tiles over both tensors, X's first.
template <int B, int SF>
__global__ __launch_bounds__(ColGeom<16>::NT, STREAM_WGS) void quantize_dual_stream_pair_kernel(DualArgs X, DualArgs W, unsigned gx, unsigned tiles_x, unsigned gw,
                                                                                                unsigned tiles)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t stream_lds[];
    __shared__ __align__(16) DualLds lds;
    TileStream<DUAL_LDS_ROWS> T(stream_lds);
    unsigned id = blockIdx.x;
    auto request = [&]() {
        if (id < tiles_x) T.request(X.c, (int)(id % gx), (int)(id / gx));
        else T.request(W.c, (int)((id - tiles_x) % gw), (int)((id - tiles_x) / gw));
    };
    request();
    const float g_x = resolve_g<NVFP4_BF16, ColGeom<16>::NT, false>(X.c);
    __syncthreads();  // (both folds use the same LDS)
    const float g_w = resolve_g<NVFP4_BF16, ColGeom<16>::NT, false>(W.c);
    if (id == 0 && threadIdx.x == 0) {
        const float to_x = tag_apply(X.tag) ? g_x : __builtin_nanf(""), to_w = tag_apply(W.tag) ? g_w : __builtin_nanf("");
        *X.c.g_out = to_x;
        if (X.g_out2) *X.g_out2 = to_x;
        *W.c.g_out = to_w;
        if (W.g_out2) *W.g_out2 = to_w;
    }
    Chunk<NVFP4_BF16> v[16];
    int tid;
    auto next = [&](const DualArgs &D, int tx, int ty) {
        tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        T.place(tid);
        T.take(T.inside(D.c, tx, ty), v);
        __syncthreads();  // (every wave has stored its share of the codes that the tile before left in lds)
        id += gridDim.x;
        if (id < tiles) request();
    };
    build_qtab<SF, true>(g_x);
    while (id < tiles_x) {
        const int tx = (int)(id % gx), ty = (int)(id / gx);
        next(X, tx, ty);
        dual_tile<NVFP4_BF16, B, SF, NVFP4_RTN, NVFP4_SR, 16>(X, v, g_x, 1.0f / (6.0f * g_x), tx, ty, tid, lds.codes, lds.scales);
    }
    __syncthreads();  // (the table of X is no longer read)
    build_qtab<SF, true>(g_w);
    while (id < tiles) {
        const int tx = (int)((id - tiles_x) % gw), ty = (int)((id - tiles_x) / gw);
        next(W, tx, ty);
        dual_tile<NVFP4_BF16, B, SF, NVFP4_RTN, NVFP4_RTN, 16>(W, v, g_w, 1.0f / (6.0f * g_w), tx, ty, tid, lds.codes, lds.scales);
    }
}

__global__ void saved_tag_kernel(TagArgs t, float *g1, float *g2)
{
    if (!tag_apply(t)) {
        if (g1) *g1 = __builtin_nanf("");
        if (g2) *g2 = __builtin_nanf("");
    }
}

// ------------------------------------------------------------------ host-side launchers

static inline hipError_t launch_status() { return hipGetLastError(); }

int64_t tensor_amax_partials(int64_t rows, int64_t cols, int64_t ld)
{
    int64_t span_rows = rows, span_cols = cols;
    if (ld == cols) {
        span_cols = rows * cols;
        span_rows = 1;
    }
    int64_t gx = ((span_cols >> 3) + 256 * AMAX_UNROLL - 1) / (256 * AMAX_UNROLL);
    if (gx < 1) gx = 1;
    return gx * (span_rows < 1 ? 1 : span_rows);
}

hipError_t launch_tensor_amax(const void *x, int dt, int64_t rows, int64_t cols, int64_t ld,
                              uint32_t *amax_bits, uint32_t *partials, float *g_out, hipStream_t st)
{
    if (rows <= 0 || cols <= 0) {
        // an empty tensor has no partial maxima: the fold alone leaves max = 0, scale = 1
        hipLaunchKernelGGL(fold_amax_kernel, dim3(1), dim3(1024), 0, st, partials, (int64_t)0, amax_bits, g_out);
        return launch_status();
    }
    int64_t span_rows = rows, span_cols = cols;
    if (ld == cols) {
        span_cols = rows * cols;
        span_rows = 1;
    }
    int64_t gx = ((span_cols >> 3) + 256 * AMAX_UNROLL - 1) / (256 * AMAX_UNROLL);
    if (gx < 1) gx = 1;
    // grid.y is limited to 65535: walk taller tensors in slabs
    for (int64_t r0 = 0; r0 < span_rows; r0 += 65535) {
        const int64_t nr = span_rows - r0 < 65535 ? span_rows - r0 : 65535;
        const char *base = reinterpret_cast<const char *>(x) + r0 * ld * (dt == NVFP4_BF16 ? 2 : 4);
        if (dt == NVFP4_BF16)
            hipLaunchKernelGGL(amax_kernel<NVFP4_BF16>, dim3((unsigned)gx, (unsigned)nr), dim3(256), 0, st,
                               base, span_cols, ld, partials + r0 * gx);
        else
            hipLaunchKernelGGL(amax_kernel<NVFP4_F32>, dim3((unsigned)gx, (unsigned)nr), dim3(256), 0, st,
                               base, span_cols, ld, partials + r0 * gx);
    }
    hipLaunchKernelGGL(fold_amax_kernel, dim3(1), dim3(1024), 0, st, partials, gx * span_rows, amax_bits, g_out);
    return launch_status();
}

static unsigned amax_grid(int64_t chunks)
{
    const int64_t gx = (chunks + AMAX_DENSE_THREADS * AMAX_UNROLL - 1) / (AMAX_DENSE_THREADS * AMAX_UNROLL);
    return (unsigned)(gx < 1 ? 1 : (gx > AMAX_DENSE_PARTIALS ? AMAX_DENSE_PARTIALS : gx));
}
static AmaxArgs amax_dense_args(const void *x, int64_t n, uint32_t *partials) { return {x, n, 0, 0, 0, 0, partials, amax_grid(n >> 3)}; }

hipError_t launch_tensor_amax_dense(const void *x, int dt, int64_t n_elements, uint32_t *partials, int *n, hipStream_t st)
{
    const AmaxArgs T = amax_dense_args(x, n_elements, partials);
    if (dt == NVFP4_BF16)
        hipLaunchKernelGGL(amax_dense_kernel<NVFP4_BF16>, dim3(T.grid), dim3(AMAX_DENSE_THREADS), 0, st, T, T);
    else
        hipLaunchKernelGGL(amax_dense_kernel<NVFP4_F32>, dim3(T.grid), dim3(AMAX_DENSE_THREADS), 0, st, T, T);
    *n = (int)T.grid;
    return launch_status();
}

hipError_t launch_tensor_amax_dense2(const void *x0, int64_t n_elements0, uint32_t *partials0, int *n0, const void *x1,
                                     int64_t n_elements1, uint32_t *partials1, int *n1, int dt, hipStream_t st)
{
    const AmaxArgs T0 = amax_dense_args(x0, n_elements0, partials0), T1 = amax_dense_args(x1, n_elements1, partials1);
    const dim3 grid(T0.grid > T1.grid ? T0.grid : T1.grid, 2);
    if (dt == NVFP4_BF16)
        hipLaunchKernelGGL(amax_dense_kernel<NVFP4_BF16>, grid, dim3(AMAX_DENSE_THREADS), 0, st, T0, T1);
    else
        hipLaunchKernelGGL(amax_dense_kernel<NVFP4_F32>, grid, dim3(AMAX_DENSE_THREADS), 0, st, T0, T1);
    *n0 = (int)T0.grid;
    *n1 = (int)T1.grid;
    return launch_status();
}

bool tensor_amax_partials_only(int64_t rows, int64_t cols) { return rows * ((cols + 7) >> 3) < ((int64_t)1 << 31) - AMAX_DENSE_THREADS * AMAX_UNROLL * AMAX_DENSE_PARTIALS; }

hipError_t launch_tensor_amax_strided(const void *x, int dt, int64_t rows, int64_t cols, int64_t ld, uint32_t *partials, int *n, hipStream_t st)
{
    const int64_t cpr = (cols + 7) >> 3;
    const AmaxArgs T = {x, 0, (uint32_t)rows, (uint32_t)cpr, cols, ld, partials, amax_grid(rows * cpr)};
    if (dt == NVFP4_BF16)
        hipLaunchKernelGGL(amax_strided_kernel<NVFP4_BF16>, dim3(T.grid), dim3(AMAX_DENSE_THREADS), 0, st, T);
    else
        hipLaunchKernelGGL(amax_strided_kernel<NVFP4_F32>, dim3(T.grid), dim3(AMAX_DENSE_THREADS), 0, st, T);
    *n = (int)T.grid;
    return launch_status();
}

template <int DT, int B, int SF, int RND, bool HW, bool ALIGNED, int RPL>
static void launch_cols(const QuantArgs &P, hipStream_t st)
{
    using G = ColGeom<RPL>;
    dim3 grid((unsigned)((P.cols + G::WG_COLS - 1) / G::WG_COLS), (unsigned)((P.rows + G::WG_ROWS - 1) / G::WG_ROWS));
    hipLaunchKernelGGL((quantize_cols_kernel<DT, B, SF, RND, HW, ALIGNED, RPL>), grid, dim3(G::NT), 0, st, P);
}

// bf16 tensors of more than 512 workgroup tiles may go through the streaming kernels (their lane tiles are whole, and the byte offset of a
// row inside a workgroup tile has 32 bits).  us, NVFP4, one tile per workgroup with 16 rows per lane / streaming, scale preset:
//                     columns                      dual, row-major                            dual, slabs
//                     RtN          SR              RtN+RtN       RtN+SR        SR+SR           RtN+RtN       RtN+SR        SR+SR
//     3072 x  6144    17.1 / 15.0  22.9 / 16.6     21.8 / 17.3   27.8 / 22.6   33.8 / 28.5     (host)        27.5 / 23.0   33.1 / 28.0
//     4096 x  8192    20.4 / 20.8  27.9 / 23.8     26.7 / 23.8   34.7 / 30.8   42.7 / 39.2     26.2 / 23.8   34.3 / 30.8   42.4 / 38.7
//     4096 x 11008    36.5 / 32.2  45.2 / 36.0     44.9 / 38.6   53.6 / 47.6   60.7 / 57.3     41.9 / 33.7   49.1 / 43.4   57.2 / 53.7
//     8192 x  8192    44.5 / 41.6  54.8 / 45.9     55.2 / 51.8   63.6 / 54.7   75.7 / 73.8     52.3 / 42.9   61.4 / 52.6   75.3 / 70.7
//     8192 x 12288    68.9 / 60.5  82.8 / 68.0     85.3 / 83.9   94.9 / 93.3   111 / 107       74.4 / 65.2   88.0 / 84.6   109 / 104
//    16384 x  8192    84.8 / 81.6  104 / 87.9      110 / 114     124 / 123     143 / 138       97.4 / 86.0   116 / 109     138 / 135
//    16384 x 12288     129 / 126   150 / 133       164 / 170     176 / 176     199 / 203       142 / 128     161 / 156     189 / 191
// The same in MXFP4:
//     3072 x  6144    17.9 / 16.0  20.1 / 16.0     22.9 / 19.3   27.0 / 22.4   33.6 / 27.6     (host)        26.8 / 26.1   32.7 / 27.9
//     4096 x 11008    34.1 / 29.1  37.8 / 34.3     43.8 / 40.6   50.1 / 42.9   58.9 / 52.0     40.2 / 33.5   47.4 / 39.5   57.3 / 50.2
//     8192 x  8192    43.4 / 42.2  48.6 / 46.1     58.3 / 56.4   62.9 / 54.7   72.1 / 64.4     51.3 / 47.9   58.7 / 50.1   70.9 / 62.9
//    16384 x 12288     126 / 126   129 / 129       169 / 168     181 / 182     193 / 192       137 / 130     156 / 141     182 / 177
// Handing each workgroup tiles one below the other instead of 768 apart: 8192 x 8192 dual RtN+RtN 72.
// Sizes between these have cut tiles, row pitches and rounds of all kinds.  Streaming / one tile per workgroup, mean over 10 to 50 random
// shapes each (preset: scale given or none, the tensor comes from memory; cached: right behind its maximum pass):
//     tiles                        513-768  -1024  -1152  -1536  -2048  -3072  -4096  -5000
//     columns RtN  NVFP4  preset      1.00   1.06   0.86   0.93   0.98   0.98   1.04   1.08
//                         cached      0.99   1.04   0.91   0.96   0.99   0.97   0.96   0.98
//                  MXFP4              0.97   1.06   0.86   0.94   1.02   1.03   1.08   1.13
//              E4M3, 64   preset      1.06   1.09   1.10   1.02   1.05   1.10   1.17   1.24
//                         cached      1.02   1.03   0.99   0.99   0.99   1.01   1.05   1.07
//              E8M0, 16               1.00   1.04   0.96   1.01   1.03   1.05   1.07   1.09
//     columns SR   NVFP4  preset      0.83   0.89   0.78   0.86   0.97   0.94   0.98   1.03
//                         cached      0.92   0.96   0.88   0.90   1.00   0.95   0.95   0.93
//                  MXFP4              0.87   0.94   0.87   0.95   0.96   1.01   1.06   1.05
//              E4M3, 64   preset      0.85   0.90   0.82   0.88   0.97   1.04   1.09   1.18
//                         cached      0.93   0.96   0.89   0.94   0.98   0.95   0.94   0.95
//         rows 64 beyond 128 preset   0.92   1.03   0.98   1.02   1.15
//                         cached      0.93   0.99   0.92   1.01   1.10   1.10   1.15   1.15
//     RtN+RtN rows NVFP4  preset      0.88   1.04   0.84   0.93   1.01   1.01
//                         cached      0.96   0.99   0.89   0.95   0.99   0.97
//                  MXFP4              1.03   1.07   0.91   0.95   0.98   0.99
//     RtN+SR rows  MXFP4              0.84   0.94   0.84   0.93   0.96   0.97
//     RtN+RtN slabs NVFP4 preset      0.99   1.03   0.83   0.90   0.94   0.92   0.93   0.95
//                  MXFP4              0.99   1.02   0.89   0.90   0.97   0.95   0.98   0.98
//     (slabs with stochastic rounding, MXFP4: 0.83 to 0.99 in every column)
// One tile per workgroup holds 1024 at once and is in its first round up to there, streaming holds 768.  Wide blocks leave their scale
// bytes one by one, with rows of an odd multiple of 64 each run of codes cuts two lines, and a walk waits for its stores.  With many
// tiles one workgroup's phases drift apart from the next one's by themselves.
static bool streams(const QuantArgs &P) { return (P.cols & 7) == 0 && P.ld <= (1 << 22); }
static bool behind_maximum(const QuantArgs &P) { return P.g_mode != G_NONE && P.g_mode != G_PRESET; }
static int64_t workgroup_tiles(int64_t rows, int64_t cols) { return ((rows + 127) / 128) * ((cols + 255) / 256); }
constexpr int64_t ONE_ROUND_TILES = 1024, STREAM_ROUND_TILES = 768;
constexpr bool columns_streamable(int block, int sf, int rnd) { return rnd == NVFP4_SR || (block <= 32 && !(block == 16 && sf == NVFP4_SCALE_E8M0)); }
static bool streams_columns(const QuantArgs &P, int block, int sf, int rnd, bool cached)
{
    const int64_t tiles = workgroup_tiles(P.rows, P.cols);
    if (!columns_streamable(block, sf, rnd) || !streams(P)) return false;
    if (rnd == NVFP4_SR) return (block <= 32 || P.rows % 128 == 0) && (cached || tiles <= (sf == NVFP4_SCALE_E4M3 && block <= 32 ? 4096 : 2048));
    return (tiles <= STREAM_ROUND_TILES || tiles > ONE_ROUND_TILES) && (cached || tiles <= (sf == NVFP4_SCALE_E4M3 ? 2048 : 1536));
}
constexpr int64_t STREAM_ROW_MAJOR_TILES = 3072;
// Right behind its maximum pass much of the tensor comes from the last-level cache, there is less latency to hide, and dual kernels with
// stochastic rounding are bound by their arithmetic, for which four waves per SIMD are better than three.  us, one tile per workgroup /
// streaming, maximum pass included:   RtN+RtN slabs   RtN+SR slabs   SR+SR slabs    columns RtN    columns SR
//     2048 x 11008                    28.7 / 28.1     34.4 / 34.3    40.2 / 39.2    25.2 / 23.8    31.2 / 29.5
//     4608 x  8192                    44.4 / 41.4     51.6 / 51.4    60.8 / 59.6    38.2 / 33.8    46.3 / 42.4
//     4096 x 11008                    50.8 / 50.2     59.4 / 61.5    69.6 / 70.4    45.5 / 42.2    55.8 / 52.1
//     8192 x  8192                    69.0 / 65.4     80.2 / 82.8    94.3 / 94.2    58.0 / 54.1    71.3 / 68.0
//     8192 x 12288                    98.8 / 96.0      112 / 116      131 / 136     84.0 / 78.8     101 / 95.9
constexpr int64_t STREAM_CACHED_SR_TILES = 1152;
static bool streams_dual(const QuantArgs &P, int block, int sf, int rnd_c, bool slabs, bool cached)
{
    const int64_t tiles = workgroup_tiles(P.rows, P.cols);
    if (!streams(P) || (cached && rnd_c == NVFP4_SR && tiles > STREAM_CACHED_SR_TILES)) return false;
    if (slabs) return rnd_c == NVFP4_SR || cached || tiles <= STREAM_ROUND_TILES || tiles > ONE_ROUND_TILES;
    // (blocks of 16 with E8M0 scales: the kernel of one tile takes too many registers for 1024 at once, 0.83 in that column)
    const bool one_round = tiles <= ONE_ROUND_TILES && !(block == 16 && sf == NVFP4_SCALE_E8M0);
    if (rnd_c == NVFP4_RTN && (tiles > STREAM_ROUND_TILES ? one_round : sf == NVFP4_SCALE_E8M0)) return false;
    return tiles <= STREAM_ROW_MAJOR_TILES;
}
bool quantize_streams(const QuantArgs &P, int block, int sf, bool both, int rnd_r, int rnd_c, bool slabs, bool cached, bool hw_convert)
{
    if (!hw_convert || short_lane_tile(NVFP4_BF16, block, sf, rnd_r, rnd_c, COLUMNS, P.rows, P.cols)) return false;
    if (!both) return !small_tensor(NVFP4_BF16, P, block, sf, true, SMALL_COLUMNS) && streams_columns(P, block, sf, rnd_c, cached);
    return (slabs || !small_tensor(NVFP4_BF16, P, block, sf, true, SMALL_DUAL)) && quantize_dual_fused(NVFP4_BF16, P.rows, P.cols, P.ld, block, true) &&
           !(rnd_r == NVFP4_SR && rnd_c == NVFP4_RTN) && streams_dual(P, block, sf, rnd_c, slabs, cached);
}
template <typename K, typename A>
static void launch_stream(K kernel, const A &args, const QuantArgs &P, int lds, hipStream_t st)
{
    using G = ColGeom<16>;
    const unsigned gx = (unsigned)((P.cols + G::WG_COLS - 1) / G::WG_COLS), tiles = gx * (unsigned)((P.rows + G::WG_ROWS - 1) / G::WG_ROWS);
    // (as many workgroups as are resident at once)
    hipLaunchKernelGGL(kernel, dim3(tiles < 256 * STREAM_WGS ? tiles : 256 * STREAM_WGS), dim3(G::NT), lds, st, args, gx, tiles);
}

template <int DT, int B, int SF, int RND, bool HW>
static void launch_q(const QuantArgs &P, int axis, hipStream_t st)
{
    if (axis == 1) {
        const int64_t total = P.rows * (P.cols >> 3);
        const int64_t per = 256 * ROWS_UNROLL;
        hipLaunchKernelGGL((quantize_rows_kernel<DT, B, SF, RND, HW>), dim3((unsigned)((total + per - 1) / per)),
                           dim3(256), 0, st, P);
    } else {
        // (the cross-check formulation and stochastic rounding with unaligned draws have the 16-row tile only)
        if (RND == NVFP4_SR && (P.cols & 7) != 0)
            launch_cols<DT, B, SF, RND, HW, RND == NVFP4_RTN, 16>(P, st);
        else if (HW && short_lane_tile(DT, B, SF, RND, RND, COLUMNS, P.rows, P.cols))
            launch_cols<DT, B, SF, RND, HW, true, HW ? 8 : 16>(P, st);
        else if constexpr (HW && DT == NVFP4_BF16 && columns_streamable(B, SF, RND)) {
            if (streams_columns(P, B, SF, RND, behind_maximum(P))) launch_stream(quantize_cols_stream_kernel<B, SF, RND>, P, P, TileStream<COLS_LDS_ROWS>::LDS_BYTES, st);
            else launch_cols<DT, B, SF, RND, HW, true, 16>(P, st);
        } else
            launch_cols<DT, B, SF, RND, HW, true, HW && DT == NVFP4_F32 && SF == NVFP4_SCALE_E8M0 && RND == NVFP4_SR ? 8 : 16>(P, st);
    }
}

template <int DT, int B, int SF>
static void launch_q_rnd(const QuantArgs &P, int axis, int rounding, bool hw, hipStream_t st)
{
    if (rounding == NVFP4_SR && hw)
        launch_q<DT, B, SF, NVFP4_SR, true>(P, axis, st);
    else if (rounding == NVFP4_SR)
        launch_q<DT, B, SF, NVFP4_SR, false>(P, axis, st);
    else if (hw)
        launch_q<DT, B, SF, NVFP4_RTN, true>(P, axis, st);
    else
        launch_q<DT, B, SF, NVFP4_RTN, false>(P, axis, st);
}

template <int DT>
static void launch_q_fmt(const QuantArgs &P, int axis, int rounding, int block, int sf, bool hw,
                         hipStream_t st)
{
#define NVFP4_CASE(BB)                                                                   \
    case BB:                                                                             \
        if (sf == NVFP4_SCALE_E4M3)                                                      \
            launch_q_rnd<DT, BB, NVFP4_SCALE_E4M3>(P, axis, rounding, hw, st);           \
        else                                                                             \
            launch_q_rnd<DT, BB, NVFP4_SCALE_E8M0>(P, axis, rounding, hw, st);           \
        break;
    switch (block) {
        NVFP4_CASE(16)
        NVFP4_CASE(32)
        NVFP4_CASE(64)
        NVFP4_CASE(128)
    default: break;
    }
#undef NVFP4_CASE
}

hipError_t launch_quantize(const QuantArgs &P, int dt, int axis, int rounding, int block, int sf,
                           bool hw_convert, hipStream_t st)
{
    if (axis == 1 && small_tensor(dt, P, block, sf, hw_convert, SMALL_ROWS)) return launch_quantize_small_rows(P, nullptr, dt, rounding, block, sf, st);
    if (axis == 0 && small_tensor(dt, P, block, sf, hw_convert, SMALL_COLUMNS)) return launch_quantize_small_columns(P, dt, rounding, block, sf, st);
    if (dt == NVFP4_BF16)
        launch_q_fmt<NVFP4_BF16>(P, axis, rounding, block, sf, hw_convert, st);
    else
        launch_q_fmt<NVFP4_F32>(P, axis, rounding, block, sf, hw_convert, st);
    return launch_status();
}

template <int DT, int B, int SF, int RND_R, int RND_C>
static void launch_dual_rpl(const DualArgs &D, hipStream_t st)
{
    // (the binary32 kernels that no tensor takes with 16 rows are not built)
    constexpr int LONG = DT == NVFP4_F32 && ((B == 16) != (SF == NVFP4_SCALE_E4M3) || (SF == NVFP4_SCALE_E8M0 && RND_C == NVFP4_SR)) ? 8 : 16;
    const unsigned gx = (unsigned)((D.c.cols + 255) / 256), gy = (unsigned)((D.c.rows + 127) / 128);
    if (short_lane_tile(DT, B, SF, RND_R, RND_C, D.slab_r || D.slab_c ? DUAL_SLABS : DUAL, D.c.rows, D.c.cols))
        hipLaunchKernelGGL((quantize_dual_kernel<DT, B, SF, RND_R, RND_C, 8>), dim3(gx, gy), dim3(ColGeom<8>::NT), 0, st, D);
    else if (DT == NVFP4_BF16 && streams_dual(D.c, B, SF, RND_C, D.slab_r || D.slab_c, behind_maximum(D.c)))
        launch_stream(quantize_dual_stream_kernel<B, SF, RND_R, RND_C>, D, D.c, TileStream<DUAL_LDS_ROWS>::LDS_BYTES, st);
    else
        hipLaunchKernelGGL((quantize_dual_kernel<DT, B, SF, RND_R, RND_C, LONG>), dim3(gx, gy), dim3(ColGeom<LONG>::NT), 0, st, D);
}

template <int DT, int B, int SF>
static void launch_dual_rnd(const DualArgs &D, int rnd_r, int rnd_c, hipStream_t st)
{
    if (rnd_r == NVFP4_SR && rnd_c == NVFP4_SR) launch_dual_rpl<DT, B, SF, NVFP4_SR, NVFP4_SR>(D, st);
    else if (rnd_r == NVFP4_RTN && rnd_c == NVFP4_SR) launch_dual_rpl<DT, B, SF, NVFP4_RTN, NVFP4_SR>(D, st);
    else launch_dual_rpl<DT, B, SF, NVFP4_RTN, NVFP4_RTN>(D, st);
}

template <int DT>
static void launch_dual_fmt(const DualArgs &D, int rnd_r, int rnd_c, int block, int sf, hipStream_t st)
{
    if (block == 16 && sf == NVFP4_SCALE_E4M3) launch_dual_rnd<DT, 16, NVFP4_SCALE_E4M3>(D, rnd_r, rnd_c, st);
    else if (block == 16) launch_dual_rnd<DT, 16, NVFP4_SCALE_E8M0>(D, rnd_r, rnd_c, st);
    else if (sf == NVFP4_SCALE_E4M3) launch_dual_rnd<DT, 32, NVFP4_SCALE_E4M3>(D, rnd_r, rnd_c, st);
    else launch_dual_rnd<DT, 32, NVFP4_SCALE_E8M0>(D, rnd_r, rnd_c, st);
}

template <int DT, int B, int SF, int RPL>
static void launch_swiglu_dual_rpl(const DualArgs &g, const DualArgs &u, hipStream_t st)
{
    using G = ColGeom<RPL>;
    dim3 grid((unsigned)((g.c.cols + G::WG_COLS - 1) / G::WG_COLS), (unsigned)((g.c.rows + G::WG_ROWS - 1) / G::WG_ROWS));
    hipLaunchKernelGGL((quantize_dual_kernel<DT, B, SF, NVFP4_SR, NVFP4_SR, RPL, SRC_SWIGLU_DG>), grid, dim3(G::NT), 0, st, g);
    hipLaunchKernelGGL((quantize_dual_kernel<DT, B, SF, NVFP4_SR, NVFP4_SR, RPL, SRC_SWIGLU_DU>), grid, dim3(G::NT), 0, st, u);
}

template <int DT, int B, int SF>
static void launch_swiglu_dual_fmt(const DualArgs &g, const DualArgs &u, hipStream_t st)
{
    if (short_lane_tile(DT, B, SF, NVFP4_SR, NVFP4_SR, SWIGLU, g.c.rows, g.c.cols)) launch_swiglu_dual_rpl<DT, B, SF, 8>(g, u, st);
    else launch_swiglu_dual_rpl<DT, B, SF, DT == NVFP4_F32 && SF == NVFP4_SCALE_E8M0 ? 8 : 16>(g, u, st);
}

hipError_t launch_swiglu_bwd_dual(DualArgs &g, DualArgs &u, int dt, int block, int sf, uint32_t *partials_g,
                                  uint32_t *partials_u, void *dG_store, void *dU_store, hipStream_t st)
{
    const int64_t n = g.c.rows * g.c.cols;
    const bool nv = block == 16 && sf == NVFP4_SCALE_E4M3, mxf = block == 32 && sf == NVFP4_SCALE_E8M0;
    if (!nv && !mxf) return hipErrorInvalidValue;
    const bool store = dG_store != nullptr;
    if (g.c.g_mode == G_FROM_AMAX || store) {
        int64_t gx = ((n >> 3) + 2047) / 2048;
        gx = gx < 1 ? 1 : (gx > AMAX_DENSE_PARTIALS ? AMAX_DENSE_PARTIALS : gx);
        const dim3 grid((unsigned)gx), wg(1024);
        if (dt == NVFP4_BF16 && store)
            hipLaunchKernelGGL((swiglu_amax_kernel<NVFP4_BF16, true>), grid, wg, 0, st, g.c.x, g.src_g, g.src_u, n, partials_g, partials_u, dG_store, dU_store);
        else if (dt == NVFP4_BF16)
            hipLaunchKernelGGL((swiglu_amax_kernel<NVFP4_BF16, false>), grid, wg, 0, st, g.c.x, g.src_g, g.src_u, n, partials_g, partials_u, dG_store, dU_store);
        else if (store)
            hipLaunchKernelGGL((swiglu_amax_kernel<NVFP4_F32, true>), grid, wg, 0, st, g.c.x, g.src_g, g.src_u, n, partials_g, partials_u, dG_store, dU_store);
        else
            hipLaunchKernelGGL((swiglu_amax_kernel<NVFP4_F32, false>), grid, wg, 0, st, g.c.x, g.src_g, g.src_u, n, partials_g, partials_u, dG_store, dU_store);
        if (g.c.g_mode == G_FROM_AMAX) {
            g.c.g_src = reinterpret_cast<const float *>(partials_g);
            u.c.g_src = reinterpret_cast<const float *>(partials_u);
            g.c.n_partials = u.c.n_partials = (int)gx;
        }
    }
    if (store) {
        // the quantizers read the stored results (the ordinary dual kernel), not dH, G, U again
        g.c.x = dG_store;
        u.c.x = dU_store;
        g.src_g = g.src_u = u.src_g = u.src_u = nullptr;
        hipError_t e = launch_quantize_dual(g, dt, NVFP4_SR, NVFP4_SR, block, sf, true, st);
        if (e != hipSuccess) return e;
        return launch_quantize_dual(u, dt, NVFP4_SR, NVFP4_SR, block, sf, true, st);
    }
    if (dt == NVFP4_BF16) {
        if (nv) launch_swiglu_dual_fmt<NVFP4_BF16, 16, NVFP4_SCALE_E4M3>(g, u, st);
        else launch_swiglu_dual_fmt<NVFP4_BF16, 32, NVFP4_SCALE_E8M0>(g, u, st);
    } else {
        if (nv) launch_swiglu_dual_fmt<NVFP4_F32, 16, NVFP4_SCALE_E4M3>(g, u, st);
        else launch_swiglu_dual_fmt<NVFP4_F32, 32, NVFP4_SCALE_E8M0>(g, u, st);
    }
    return launch_status();
}

template <int B, int SF>
static void launch_dual_stream_pair(const DualArgs &x, const DualArgs &w, hipStream_t st)
{
    using G = ColGeom<16>;
    auto across = [](const DualArgs &d) { return (unsigned)((d.c.cols + G::WG_COLS - 1) / G::WG_COLS); };
    auto down = [](const DualArgs &d) { return (unsigned)((d.c.rows + G::WG_ROWS - 1) / G::WG_ROWS); };
    const unsigned tiles_x = across(x) * down(x), tiles = tiles_x + across(w) * down(w);
    hipLaunchKernelGGL((quantize_dual_stream_pair_kernel<B, SF>), dim3(tiles < 256 * STREAM_WGS ? tiles : 256 * STREAM_WGS), dim3(G::NT),
                       TileStream<DUAL_LDS_ROWS>::LDS_BYTES, st, x, w, across(x), tiles_x, across(w), tiles);
}

template <int DT, int B, int SF>
static void launch_dual_pair_fmt(const DualArgs &x, const DualArgs &w, hipStream_t st)
{
    using G = ColGeom<8>;
    auto across = [](const DualArgs &d) { return (unsigned)((d.c.cols + G::WG_COLS - 1) / G::WG_COLS); };
    auto down = [](const DualArgs &d) { return (unsigned)((d.c.rows + G::WG_ROWS - 1) / G::WG_ROWS); };
    const unsigned tiles = across(x) * down(x);
    hipLaunchKernelGGL((quantize_dual_pair_kernel<DT, B, SF>), dim3(tiles + across(w) * down(w)), dim3(G::NT), 0, st, x, w, tiles, across(x), across(w));
}

// The two single-orientation passes of a dual quantization; each writes one of the scale's destinations.
static QuantArgs row_side(const DualArgs &D)
{
    QuantArgs r = D.c;
    r.codes = D.codes_r;
    r.scales = D.scales_r;
    r.seed = D.seed_r;
    return r;
}
static hipError_t launch_column_side(const DualArgs &D, int dt, int rounding, int block, int sf, bool hw_convert, hipStream_t st)
{
    QuantArgs c = D.c;
    if (D.g_out2) c.g_out = D.g_out2;
    const hipError_t e = launch_quantize(c, dt, 0, rounding, block, sf, hw_convert, st);
    return e != hipSuccess ? e : launch_saved_tag(D.tag, D.c.g_out, D.g_out2, st);
}

hipError_t launch_quantize_dual_pair(const DualArgs &x, const DualArgs &w, int dt, int block, int sf, bool hw_convert, hipStream_t st)
{
    if (!(x.slab_r || x.slab_c || w.slab_r || w.slab_c) && small_tensor(dt, x.c, block, sf, hw_convert, SMALL_DUAL) && small_tensor(dt, w.c, block, sf, hw_convert, SMALL_DUAL) &&
        x.c.rows % block == 0 && w.c.rows % block == 0) {
        return launch_quantize_small_dual(x, &w, dt, NVFP4_RTN, NVFP4_SR, block, sf, st);
    }
    const int64_t tiles = ((x.c.rows + 127) / 128) * ((x.c.cols + 255) / 256) + ((w.c.rows + 127) / 128) * ((w.c.cols + 255) / 256);
    const bool nv = block == 16 && sf == NVFP4_SCALE_E4M3, mxf = block == 32 && sf == NVFP4_SCALE_E8M0;
    const bool fused = (nv || mxf) && quantize_dual_fused(dt, x.c.rows, x.c.cols, x.c.ld, block, hw_convert) &&
                       quantize_dual_fused(dt, w.c.rows, w.c.cols, w.c.ld, block, hw_convert);
    const bool slabs = (x.slab_r || x.slab_c) && (w.slab_r || w.slab_c);
    if (fused && dt == NVFP4_BF16 && tiles > PAIR_TILES && tiles < ((int64_t)1 << 31) && (slabs || tiles <= STREAM_ROW_MAJOR_TILES) && streams(x.c) && streams(w.c)) {
        if (nv) launch_dual_stream_pair<16, NVFP4_SCALE_E4M3>(x, w, st);
        else launch_dual_stream_pair<32, NVFP4_SCALE_E8M0>(x, w, st);
        return launch_status();
    }
    if (fused && tiles <= PAIR_TILES) {
        if (dt == NVFP4_BF16 && nv) launch_dual_pair_fmt<NVFP4_BF16, 16, NVFP4_SCALE_E4M3>(x, w, st);
        else if (dt == NVFP4_BF16) launch_dual_pair_fmt<NVFP4_BF16, 32, NVFP4_SCALE_E8M0>(x, w, st);
        else if (nv) launch_dual_pair_fmt<NVFP4_F32, 16, NVFP4_SCALE_E4M3>(x, w, st);
        else launch_dual_pair_fmt<NVFP4_F32, 32, NVFP4_SCALE_E8M0>(x, w, st);
        return launch_status();
    }
    if (!quantize_dual_fused(dt, x.c.rows, x.c.cols, x.c.ld, block, hw_convert) && !quantize_dual_fused(dt, w.c.rows, w.c.cols, w.c.ld, block, hw_convert)) {
        // (wide blocks) the rows of both in one launch, then the columns of each
        if (x.slab_r || x.slab_c || w.slab_r || w.slab_c) return hipErrorInvalidValue;
        hipError_t e = launch_quantize_rows_pair(row_side(x), row_side(w), dt, block, sf, hw_convert, st);
        if (e == hipSuccess) e = launch_column_side(x, dt, NVFP4_SR, block, sf, hw_convert, st);
        return e != hipSuccess ? e : launch_column_side(w, dt, NVFP4_RTN, block, sf, hw_convert, st);
    }
    const hipError_t e = launch_quantize_dual(x, dt, NVFP4_RTN, NVFP4_SR, block, sf, hw_convert, st);
    return e != hipSuccess ? e : launch_quantize_dual(w, dt, NVFP4_RTN, NVFP4_RTN, block, sf, hw_convert, st);
}

template <int DT>
static void launch_rows_pair_dt(const QuantArgs &a, const QuantArgs &b, int block, int sf, unsigned wa, unsigned wb, hipStream_t st)
{
    const dim3 grid(wa + wb), wg(256);
    if (sf == NVFP4_SCALE_E8M0) hipLaunchKernelGGL((quantize_rows_pair_kernel<DT, 32, NVFP4_SCALE_E8M0>), grid, wg, 0, st, a, b, wa);
    else if (block == 16) hipLaunchKernelGGL((quantize_rows_pair_kernel<DT, 16, NVFP4_SCALE_E4M3>), grid, wg, 0, st, a, b, wa);
    else if (block == 32) hipLaunchKernelGGL((quantize_rows_pair_kernel<DT, 32, NVFP4_SCALE_E4M3>), grid, wg, 0, st, a, b, wa);
    else if (block == 64) hipLaunchKernelGGL((quantize_rows_pair_kernel<DT, 64, NVFP4_SCALE_E4M3>), grid, wg, 0, st, a, b, wa);
    else hipLaunchKernelGGL((quantize_rows_pair_kernel<DT, 128, NVFP4_SCALE_E4M3>), grid, wg, 0, st, a, b, wa);
}

hipError_t launch_quantize_rows_pair(const QuantArgs &a, const QuantArgs &b, int dt, int block, int sf, bool hw_convert, hipStream_t st)
{
    if (small_tensor(dt, a, block, sf, hw_convert, SMALL_ROWS) && small_tensor(dt, b, block, sf, hw_convert, SMALL_ROWS))
        return launch_quantize_small_rows(a, &b, dt, NVFP4_RTN, block, sf, st);
    auto wgs = [](const QuantArgs &P) { return (P.rows * (P.cols >> 3) + 256 * ROWS_UNROLL - 1) / (256 * ROWS_UNROLL); };
    if (hw_convert && wgs(a) + wgs(b) < ((int64_t)1 << 31) && (sf == NVFP4_SCALE_E4M3 || block == 32)) {
        const unsigned wa = (unsigned)wgs(a), wb = (unsigned)wgs(b);
        if (dt == NVFP4_BF16) launch_rows_pair_dt<NVFP4_BF16>(a, b, block, sf, wa, wb, st);
        else launch_rows_pair_dt<NVFP4_F32>(a, b, block, sf, wa, wb, st);
        return launch_status();
    }
    const hipError_t e = launch_quantize(a, dt, 1, NVFP4_RTN, block, sf, hw_convert, st);
    return e != hipSuccess ? e : launch_quantize(b, dt, 1, NVFP4_RTN, block, sf, hw_convert, st);
}

bool quantize_dual_fused(int dt, int64_t rows, int64_t cols, int64_t ld, int block, bool hw_convert)
{
    const int64_t esz = dt == NVFP4_BF16 ? 2 : 4;
    return hw_convert && (block == 16 || block == 32) && rows % block == 0 && cols % block == 0 &&
           (ld * esz) % 16 == 0 && cols < (int64_t(1) << 31) && rows < (int64_t(1) << 31);
}

hipError_t launch_quantize_dual(const DualArgs &D, int dt, int rnd_r, int rnd_c, int block, int sf, bool hw_convert,
                                hipStream_t st)
{
    if (!D.slab_r && !D.slab_c && small_tensor(dt, D.c, block, sf, hw_convert, SMALL_DUAL)) return launch_quantize_small_dual(D, nullptr, dt, rnd_r, rnd_c, block, sf, st);
    // (SR rows with RtN columns is a combination no equation asks for: two kernels)
    if (quantize_dual_fused(dt, D.c.rows, D.c.cols, D.c.ld, block, hw_convert) && !(rnd_r == NVFP4_SR && rnd_c == NVFP4_RTN)) {
        if (dt == NVFP4_F32) launch_dual_fmt<NVFP4_F32>(D, rnd_r, rnd_c, block, sf, st);
        else launch_dual_fmt<NVFP4_BF16>(D, rnd_r, rnd_c, block, sf, st);
        return launch_status();
    }
    // other block sizes and ragged shapes: the two single-orientation kernels (they write the plain layout only)
    if (D.slab_r || D.slab_c) return hipErrorInvalidValue;
    const hipError_t e = launch_quantize(row_side(D), dt, 1, rnd_r, block, sf, hw_convert, st);
    return e != hipSuccess ? e : launch_column_side(D, dt, rnd_c, block, sf, hw_convert, st);
}

hipError_t launch_saved_tag(const TagArgs &t, float *g1, float *g2, hipStream_t st)
{
    if (!t.dst && !t.chk) return hipSuccess;
    hipLaunchKernelGGL(saved_tag_kernel, dim3(1), dim3(1), 0, st, t, g1, g2);
    return launch_status();
}

}  // namespace nvfp4
