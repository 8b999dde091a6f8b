// Linear layers of a small network in one launch per call: forward (quantizers of X and W, Eq. 4, and the transposed operands for the
// backward call) and backward on saved operands (both orientations of dY, Eqs. 5-6).
//
// A call of this size is bound by its launches: the host spends 3.4 us on each, the GPU 2 to 3 us before and after the arithmetic, and the
// second one reads what the first has just written.  So every workgroup of a product quantizes the rows (or, for dW, the columns) that its
// tile needs into the LDS stages that gemm_ksplit.hip fills by loads, taking the tensor maximum of the whole tensor like the quantizers for
// small tensors do, and multiplies them there: the same codes and, a K tile per wave, the same sums.  What a forward call leaves for the
// backward one are workgroups of the same launch.  All loads of a workgroup are issued before the first wait (in the order of their use:
// 0.7 us more), and all its waves draw for the columns of dY (the few that hold a block alone: 0.8 us more).
// us, forward and backward, operands handed over, two launches each / one each; GPU time, and as a program calls it:
//     64 x 256 x 128 binary32 NVFP4 16.5 / 13.9 and 20.2 / 14.4, MXFP4 14.6 / 10.1      512 x 64 x 64 NVFP4 18.5 / 15.3 (two in the backward call)
//     160 x 160 x 160 binary32 NVFP4 17.4 / 14.6, MXFP4 15.3 / 10.6                     256 x 256 x 256 bf16 NVFP4 18.9 / 18.1, MXFP4 16.8 / 11.5
#include "gemm_ksplit.h"
#include "quantize_small.h"

namespace nvfp4 {

namespace fs {

constexpr int NT = 512, NW = NT / 64;
constexpr int FOLD = 2 * NT / 16 * 4;                 // LDS bytes of the fold of two maxima
constexpr int MOST_ROWS = 256;                        // of dY in a backward call: its draws are in the LDS
constexpr int MOST_K = 512, TILES = MOST_K / ks::KT;  // contraction: K tiles in the LDS

// A thread's part of a tensor of at most SELF_AMAX_BYTES, for its maximum: all of it in flight at once.
template <int DT>
struct Part {
    static constexpr int U = (int)(SELF_AMAX_BYTES / (DT == NVFP4_BF16 ? 16 : 32) / NT);
    Chunk<DT> v[U];
    __device__ __forceinline__ void load(const void *x, int n)
    {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            v[u].zero();
            if ((int)threadIdx.x + u * NT < (n >> 3)) v[u].template load<false>(x, (int64_t)(threadIdx.x + u * NT) * 8);
        }
    }
    __device__ __forceinline__ uint32_t maximum() const
    {
        float a = 0.0f;
#pragma unroll
        for (int u = 0; u < U; ++u) a = fmaxf(a, chunk_amax(v[u]));
        return f2u(a);
    }
};
// every thread's maxima -> the workgroup's (one barrier)
template <int N>
__device__ __forceinline__ void fold_max(uint32_t (&m)[N], uint32_t *fold)
{
#pragma unroll
    for (int i = 0; i < N; ++i) {
        m[i] = f2u(group_max<16>(u2f(m[i])));
        if ((threadIdx.x & 15) == 0) fold[i * (NT / 16) + (threadIdx.x >> 4)] = m[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int t = 0; t < NT / 16; ++t) m[i] = umax(m[i], fold[i * (NT / 16) + t]);
}

// One block's scale byte into a stage (gemm_ksplit.h): row of the stage, chunk c of 8 elements of the K tile that the block starts with.
template <int B, int SF, int ROWS>
__device__ __forceinline__ void put_scale(uint8_t *scales, int row, int c, uint32_t sbyte)
{
    if constexpr (SF == NVFP4_SCALE_E8M0) scales[row * 4 + (c >> 2)] = (uint8_t)sbyte;
    else if constexpr (B == 16) reinterpret_cast<uint16_t *>(scales)[((c >> 2) * ROWS + row) * 2 + ((c >> 1) & 1)] = (uint16_t)(sbyte << 7);
    else reinterpret_cast<uint32_t *>(scales)[(c >> 2) * ROWS + row] = sbyte * 0x00800080u;
}
__device__ __forceinline__ int code_at(int row, int c) { return row * ks::KTB + ((((c >> 2) & 3) ^ ((row >> 2) & 3)) << 4) + (c & 3) * 4; }

// 32 rows of a dense [rows, K] tensor from `first` on (past the last: the last), as chunks in registers, then as codes in the stages.
template <int DT>
struct Rows {
    static constexpr int U = 32 * MOST_K / 8 / NT;
    Chunk<DT> v[U];
    int64_t first, last;
    int cpr;
    __device__ __forceinline__ int64_t row(int u, uint32_t row_mul, int &r, int &c) const
    {
        const int id = threadIdx.x + u * NT;
        r = (int)__umulhi((uint32_t)id, row_mul);
        c = id - r * cpr;
        return first + r < last ? first + r : last;
    }
    __device__ __forceinline__ void load(const void *x, int64_t first_, int64_t rows, int64_t K, uint32_t row_mul)
    {
        first = first_;
        last = rows - 1;
        cpr = (int)(K >> 3);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            int r, c;
            const int64_t i = row(u, row_mul, r, c);
            v[u].zero();
            if (r < 32) v[u].template load<false>(x, i * K + c * 8);
        }
    }
    template <int B, int SF, int RND, int ROWS, int STAGE>
    __device__ __forceinline__ void put(uint8_t *stages, int row0, float g, float k, uint64_t seed, uint32_t row_mul) const
    {
        constexpr bool MXS = SF == NVFP4_SCALE_E8M0;
        constexpr int LPB = B / 8;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            int r, c;
            const int64_t i = row(u, row_mul, r, c);
            const float a = group_max<LPB>(MXS ? chunk_amax_packed(v[u]) : chunk_amax(v[u]));
            float q;
            const uint32_t sbyte = block_scale<SF, true, false>(a, g, k, &q);
            if (MXS) q = mx_scale_operand(sbyte);
            const uint32_t packed = chunk_codes_hw<DT, RND, MXS>(v[u], q, seed, (uint64_t)(i * cpr + c));
            if (r < 32) {
                uint8_t *const stage = stages + (c >> 4) * STAGE;
                *reinterpret_cast<uint32_t *>(stage + code_at(row0 + r, c & 15)) = packed;
                if ((threadIdx.x & (LPB - 1)) == 0) put_scale<B, SF, ROWS>(stage + ROWS * ks::KTB, row0 + r, c & 15, sbyte);
            }
        }
    }
};

// The scales of the chunks that the last K tile of a ragged contraction lacks: zeros
template <int SF, int ROWS, int STAGE>
__device__ __forceinline__ void put_tail(uint8_t *stages, int nkt, int rem)
{
    uint8_t *const scales = stages + (nkt - 1) * STAGE + ROWS * ks::KTB;
    for (int id = threadIdx.x; id < 4 * ROWS; id += NT) {
        const int j = id / ROWS, row = id - j * ROWS;
        if (j * 32 < rem) continue;
        if constexpr (SF == NVFP4_SCALE_E8M0) scales[row * 4 + j] = 0;
        else reinterpret_cast<uint32_t *>(scales)[j * ROWS + row] = 0;
    }
}

// The K tiles in the stages, dealt to the waves as in gemm_ksplit.hip (the same sums in the same order), and the outputs
template <int SF, int TA, int TB, int OUT_DT>
__device__ __forceinline__ void multiply(const GemmArgs &P, uint8_t *lds, int64_t m0, int64_t n0, int nkt, int rem, float gg)
{
    using G = ks::Geom<SF, TA, TB, NW>;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    ks::float16_t acc[TA][TB];
#pragma unroll
    for (int a = 0; a < TA; ++a)
#pragma unroll
        for (int b = 0; b < TB; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.0f;
    for (int kt = wave; kt < nkt; kt += NW) ksplit_compute<SF, TA, TB, NW>(lds + kt * G::STAGE, kt == nkt - 1 && rem < ks::KT, rem, acc, lane);
    ksplit_finish<SF, TA, TB, NW, OUT_DT>(P, acc, lds, m0, n0, [&]() { return gg; });
}

}  // namespace fs

template <int DT, int B, int SF, int OUT_DT>
__global__ __launch_bounds__(fs::NT) void small_forward_kernel(SmallForward S)
{
    using namespace fs;
    using G = ks::Geom<SF, 1, 1, NW>;
    constexpr bool MX = SF == NVFP4_SCALE_E8M0;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    uint32_t *const aux = reinterpret_cast<uint32_t *>(lds + S.lds_aux);  // fold, or a column job's draws
    if (blockIdx.x >= S.tiles) {
        unsigned wg = blockIdx.x - S.tiles;
        if (wg < S.cx.wgs) cols_small<DT, B, SF, NVFP4_SR>(S.cx.q, wg, aux);
        else cols_small<DT, B, SF, NVFP4_RTN>(S.cw.q, wg - S.cx.wgs, aux);
        return;
    }
    const GemmArgs &P = S.P;
    int ty, tx;
    tile_coords((int)blockIdx.x, (int)((P.N + 31) / 32), (int)((P.M + 31) / 32), ty, tx);
    const int64_t m0 = (int64_t)ty * 32, n0 = (int64_t)tx * 32;
    const int nkt = (int)((P.K + ks::KT - 1) / ks::KT), rem = (int)(P.K - (int64_t)(nkt - 1) * ks::KT);
    Rows<DT> a, b;
    a.load(S.X, m0, P.M, P.K, S.row_mul);
    b.load(S.W, n0, P.N, P.K, S.row_mul);
    float gx = 1.0f, gw = 1.0f;
    if (!MX && S.tensor_scale) {
        Part<DT> x, w;
        x.load(S.X, (int)(P.M * P.K));
        w.load(S.W, (int)(P.N * P.K));
        uint32_t m[2] = {x.maximum(), w.maximum()};
        fold_max<2>(m, aux);
        gx = tensor_scale_from_amax(u2f(m[0]));
        gw = tensor_scale_from_amax(u2f(m[1]));
    }
    a.template put<B, SF, NVFP4_RTN, G::ROWS, G::STAGE>(lds, 0, gx, 1.0f / (6.0f * gx), 0, S.row_mul);
    b.template put<B, SF, NVFP4_RTN, G::ROWS, G::STAGE>(lds, 32, gw, 1.0f / (6.0f * gw), 0, S.row_mul);
    if (rem < ks::KT) put_tail<SF, G::ROWS, G::STAGE>(lds, nkt, rem);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        S.scales[0] = gx;
        S.scales[1] = gw;
        if (S.saved_scales) {
            S.saved_scales[0] = gx;
            S.saved_scales[1] = gw;
        }
        tag_apply(S.tag);
    }
    __syncthreads();
    multiply<SF, 1, 1, OUT_DT>(P, lds, m0, n0, nkt, rem, gx * gw);
}

// A packed row-major operand's 32 rows from `first` on (a chunk of 32 codes a thread), in registers, then as rows row0 .. of the stages
template <int B>
struct Packed {
    uint4 codes;
    uint32_t scales;
    int r, c;
    __device__ __forceinline__ void load(const uint8_t *cp, const uint8_t *sp, int64_t first, int64_t rows, int64_t K)
    {
        static_assert(32 * fs::MOST_K / 32 == fs::NT, "one chunk a thread");
        const int cpr = (int)(K >> 5);
        r = (int)threadIdx.x / cpr;
        c = (int)threadIdx.x - r * cpr;
        if (r >= 32) return;
        const int64_t i = first + r < rows ? first + r : rows - 1;
        codes = *reinterpret_cast<const uint4 *>(cp + i * (K >> 1) + c * 16);
        scales = B == 16 ? *reinterpret_cast<const uint16_t *>(sp + i * (K / B) + 2 * c) : sp[i * (K / B) + c];
    }
    template <int SF, int ROWS, int STAGE>
    __device__ __forceinline__ void put(uint8_t *stages, int row0) const
    {
        if (r >= 32) return;
        uint8_t *const stage = stages + (c >> 2) * STAGE;
        *reinterpret_cast<uint4 *>(stage + fs::code_at(row0 + r, 4 * (c & 3))) = codes;
#pragma unroll
        for (int t = 0; t < 32 / B; ++t) fs::put_scale<B, SF, ROWS>(stage + ROWS * ks::KTB, row0 + r, 4 * (c & 3) + t * (B / 8), (scales >> (8 * t)) & 0xFFu);
    }
};

template <int DT, int B, int SF, int OUT_DT>
__global__ __launch_bounds__(fs::NT) void small_backward_kernel(SmallBackward S)
{
    using namespace fs;
    constexpr bool MX = SF == NVFP4_SCALE_E8M0;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    uint32_t *const aux = reinterpret_cast<uint32_t *>(lds + S.lds_aux);
    const bool first = blockIdx.x < S.tiles;
    const GemmArgs &P = first ? S.dx : S.dw;
    const int nkt = (int)((P.K + ks::KT - 1) / ks::KT), rem = (int)(P.K - (int64_t)(nkt - 1) * ks::KT);
    const int bm = first ? 32 : 64;
    int ty, tx;
    tile_coords((int)(first ? blockIdx.x : blockIdx.x - S.tiles), (int)((P.N + 31) / 32), (int)((P.M + bm - 1) / bm), ty, tx);
    const int64_t m0 = (int64_t)ty * bm, n0 = (int64_t)tx * 32;
    // every load first: B's packed rows, dY's, and all of dY for its maximum
    Packed<B> b;
    b.load(P.B_codes, P.B_scales, n0, P.N, P.K);
    Part<DT> y;
    const bool maximum = !MX && S.tensor_scale;
    auto scale = [&]() {
        if (!maximum) return 1.0f;
        uint32_t m[1] = {y.maximum()};
        fold_max<1>(m, aux);
        return tensor_scale_from_amax(u2f(m[0]));
    };
    // (a `saved` buffer that is not the one this call expects poisons the outputs)
    const float gb = tag_apply(S.tag) ? P.gB[0] : __builtin_nanf("");
    if (first) {
        // dX = Q_SR(dY) Q(W^T)^T
        using G = ks::Geom<SF, 1, 1, NW>;
        Rows<DT> a;
        a.load(S.dY.x, m0, P.M, P.K, S.row_mul);
        if (maximum) y.load(S.dY.x, (int)(S.dY.rows * S.dY.cols));
        b.template put<SF, G::ROWS, G::STAGE>(lds, 32);
        const float g = scale();
        a.template put<B, SF, NVFP4_SR, G::ROWS, G::STAGE>(lds, 0, g, 1.0f / (6.0f * g), S.seed_rows, S.row_mul);
        if (rem < ks::KT) put_tail<SF, G::ROWS, G::STAGE>(lds, nkt, rem);
        __syncthreads();
        multiply<SF, 1, 1, OUT_DT>(P, lds, m0, n0, nkt, rem, g * gb);
    } else {
        // dW = Q_SR(dY^T) Q(X^T)^T: 64 columns of dY, a wave for each of their blocks
        using G = ks::Geom<SF, 2, 1, NW>;
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, row = lane_column<DT>(lane), blocks = (int)(P.K / B);
        uint16_t *const draws = reinterpret_cast<uint16_t *>(lds + S.lds_aux + FOLD);  // [row][column of the 64]
        float v[B];
        load_column<DT, B>(S.dY, (int64_t)wave * B, m0, lane, wave < blocks && m0 + row < P.M, v);
        if (maximum) y.load(S.dY.x, (int)(S.dY.rows * S.dY.cols));
        // (all waves draw, also those without a block)
#pragma unroll
        for (int u = 0; u < MOST_ROWS * 8 / NT; ++u) {
            const int i = (threadIdx.x + u * NT) >> 3, cg = threadIdx.x & 7;
            if (i >= (int)P.K) break;
            const u32x4 d = sr_draw(S.dY.seed, (uint64_t)i * ((uint64_t)S.dY.cols >> 3) + ((uint64_t)m0 >> 3) + cg);
            *reinterpret_cast<uint4 *>(draws + i * 64 + cg * 8) = make_uint4(d.x, d.y, d.z, d.w);
        }
        b.template put<SF, G::ROWS, G::STAGE>(lds, 64);
        const float g = scale();
        if (!maximum) __syncthreads();  // (the draws)
        for (int blk = wave; blk < blocks; blk += NW) {
            if (blk != wave) load_column<DT, B>(S.dY, (int64_t)blk * B, m0, lane, m0 + row < P.M, v);
            uint32_t words[B / 8];
            const uint32_t sbyte = column_block<DT, B, SF, NVFP4_SR>(v, column_max(v), g, 1.0f / (6.0f * g), draws + blk * (B * 64), lane, words);
            const int c = blk * (B / 8);
            uint8_t *const stage = lds + (c >> 4) * G::STAGE;
#pragma unroll
            for (int w = 0; w < B / 8; ++w) *reinterpret_cast<uint32_t *>(stage + code_at(row, (c & 15) + w)) = words[w];
            put_scale<B, SF, G::ROWS>(stage + G::CODES, row, c & 15, sbyte);
        }
        if (rem < ks::KT) put_tail<SF, G::ROWS, G::STAGE>(lds, nkt, rem);
        __syncthreads();
        multiply<SF, 2, 1, OUT_DT>(P, lds, m0, n0, nkt, rem, g * gb);
    }
}

// ------------------------------------------------------------------ host side

static bool small_format(int block, int sf) { return (block == 16 && sf == NVFP4_SCALE_E4M3) || (block == 32 && sf == NVFP4_SCALE_E8M0); }
// Tensors whose maximum every workgroup takes, contractions whose K tiles fit the LDS beside the partial sums.  (The tile rule of a product
// that is not fused is asked, so that its sums are the same: one K tile per wave.)
static bool small_product(int64_t M, int64_t N, int64_t K, int dt, int sf)
{
    const int64_t esz = dt == NVFP4_BF16 ? 2 : 4;
    return K <= fs::MOST_K && M * K * esz <= SELF_AMAX_BYTES && M > 16 && choose_gemm_tile(M, N, K, sf) <= TILE_64x64;
}
static int64_t tiles(int64_t M, int64_t N, int rows) { return (M + rows - 1) / rows * ((N + 31) / 32); }
// The workgroups of one launch repeat each other's work: every one quantizes its rows of X and W (or of dY) anew, and with a tensor scale reads
// all of both tensors for their maxima.  So the rules count workgroups.  With a tensor scale it is those that the CUs hold at once (one per CU
// in bf16, two in binary32), and without saved operands contractions up to 256, beyond which the quantizer's part of a tile is longer than the launch
// it saves.  us, GPU time of a forward call in a graph, separate / one launch (NVFP4, bf16 unless said; + : with saved operands):
//     480 x 512 x 64 (240 workgroups)  7.4 /  7.3   + (248) 8.9 /  7.2      512 x  512 x  64 (256)  7.4 /  7.3   + (264)  9.0 / 10.2
//     576 x 512 x 64 (288)             7.8 / 11.1   + (297) 9.2 / 11.4     1024 x 1024 x  64 (1024) 10.0 / 28.3   +       11.8 / 31.6
//     256 x 256 x 256 (64)             7.7 /  8.5   +       9.4 /  8.5      128 x  128 x 512 (16)   7.7 /  9.4   + (32)   9.3 /  9.4
//     binary32: 512 x 512 x 64 (256)   7.8 /  7.4   + (264) 9.4 /  8.0     1024 x  512 x  32 (512)  8.7 /  9.0   + (518) 10.2 / 11.0
// (as a program calls them the host's work for the second launch, 1 to 2 us, is saved besides: 128 x 128 x 256 8.9 / 8.0, x 512 10.1 / 9.6.)  Without a
// tensor scale: MXFP4 1024 x 640 x 64 (640) 6.8 / 5.9, + 8.9 / 6.4, 1024 x 896 x 32 (896) 6.9 / 7.5, + (904) 9.2 / 7.9, 1024 x 1024 x 32 (1024) + 9.0 / 8.7; E4M3
// 1024 x 512 x 32 bf16 1.05 times as fast, 768 x 768 x 32 0.84, binary32 960 x 768 x 32 1.16, 1024 x 1024 x 32 0.98.
bool small_forward_takes(int64_t M, int64_t N, int64_t K, int dt, int block, int sf, bool tensor_scale, bool saved)
{
    if (!small_format(block, sf) || !small_product(M, N, K, dt, sf) || N * K * (dt == NVFP4_BF16 ? 2 : 4) > SELF_AMAX_BYTES) return false;
    const int64_t product = tiles(M, N, 32), waves = SMALL_NT / 64;
    if (sf == NVFP4_SCALE_E8M0) return product <= (saved ? 960 : 768);
    if (!tensor_scale) return product <= (dt == NVFP4_BF16 ? 512 : 768);
    const int64_t jobs = saved ? (K + 63) / 64 * ((M / block + waves - 1) / waves + (N / block + waves - 1) / waves) : 0;
    return product + jobs <= (dt == NVFP4_BF16 ? 256 : 512) && (saved || K <= 256);
}
// The backward kernel's LDS is one workgroup per CU's.  A second round is worth it for few rows of dY, whose quantization is the shorter part.  us,
// GPU time in a graph, separate / one launch, NVFP4 bf16: 64 x 512 x 800 (250) 12.8 / 8.4, 64 x 512 x 832 (260) 12.9 / 12.6, 64 x 64 x 2880 (270) 12.4 / 13.1,
// 128 x 128 x 1440 (270) 11.4 / 13.7, 256 x 256 x 640 (240) 12.8 / 9.4, x 704 (264) 12.5 / 15.6, x 4096 (1536) 16.0 / 44.7; binary32 64 x 512 x 1024 (320) 13.6 /
// 12.2, 64 x 64 x 3456 (324) 0.99 times as fast; MXFP4 64 x 512 x 1024 11.6 / 10.2, 128 x 128 x 2048 (384) 10.4 / 10.3, 256 x 256 x 704 0.98 times as fast, x
// 4096 13.9 / 30.3; E4M3 without a tensor scale 64 x 512 x 1024 1.20 times as fast, 128 x 128 x 1440 0.95.  (Slower within one round: 256 x 128 x 640
// bf16 (200) 8.6 / 9.1, whose two products share a launch; the host's work again makes up for it.)
bool small_backward_takes(int64_t M, int64_t N, int64_t K, int dt, int block, int sf, bool tensor_scale)
{
    if (!small_format(block, sf) || M > fs::MOST_ROWS || !small_product(M, K, N, dt, sf) || !small_product(N, K, M, dt, sf)) return false;
    const int64_t wgs = tiles(M, K, 32) + tiles(N, K, 64);
    const bool again = sf == NVFP4_SCALE_E8M0 ? M <= 128 : M <= 96 && (!tensor_scale || (dt == NVFP4_F32 && N >= 128));
    return wgs <= (again ? 512 : 256);
}

static uint32_t reciprocal(int64_t d) { return (uint32_t)(((uint64_t)1 << 32) / (uint64_t)d) + 1u; }  // of chunk numbers below 2^13

template <int DT, int B, int SF>
static hipError_t launch_small_forward_fmt(SmallForward &S, int out_dt, hipStream_t st)
{
    using G = ks::Geom<SF, 1, 1, fs::NW>;
    constexpr int STAGES = fs::TILES * G::STAGE, PARTS = fs::NW * G::PARTIAL, MAIN = STAGES > PARTS ? STAGES : PARTS, DRAWS = fs::NW * B * 128;
    constexpr int LDS = MAIN + fs::FOLD + DRAWS;
    S.lds_aux = MAIN;
    S.row_mul = reciprocal(S.P.K >> 3);
    S.tiles = (unsigned)tiles(S.P.M, S.P.N, 32);
    const unsigned wgs = S.tiles + S.cx.wgs + S.cw.wgs;
    if (out_dt == NVFP4_F32) {
        auto k = small_forward_kernel<DT, B, SF, NVFP4_F32>;
        static bool once = ((void)hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, LDS), true);
        (void)once;
        hipLaunchKernelGGL(k, dim3(wgs), dim3(fs::NT), LDS, st, S);
    } else {
        auto k = small_forward_kernel<DT, B, SF, NVFP4_BF16>;
        static bool once = ((void)hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, LDS), true);
        (void)once;
        hipLaunchKernelGGL(k, dim3(wgs), dim3(fs::NT), LDS, st, S);
    }
    return hipGetLastError();
}
hipError_t launch_small_forward(SmallForward S, const QuantArgs *cx, const QuantArgs *cw, int dt, int block, int sf, int out_dt, hipStream_t st)
{
    S.cx = S.cw = SmallJob{};
    if (cx) S.cx = small_job(*cx, 0, NVFP4_SR, block);
    if (cw) S.cw = small_job(*cw, 0, NVFP4_RTN, block);
    if (sf == NVFP4_SCALE_E8M0)
        return dt == NVFP4_BF16 ? launch_small_forward_fmt<NVFP4_BF16, 32, NVFP4_SCALE_E8M0>(S, out_dt, st) : launch_small_forward_fmt<NVFP4_F32, 32, NVFP4_SCALE_E8M0>(S, out_dt, st);
    return dt == NVFP4_BF16 ? launch_small_forward_fmt<NVFP4_BF16, 16, NVFP4_SCALE_E4M3>(S, out_dt, st) : launch_small_forward_fmt<NVFP4_F32, 16, NVFP4_SCALE_E4M3>(S, out_dt, st);
}

template <int DT, int B, int SF>
static hipError_t launch_small_backward_fmt(SmallBackward &S, int out_dt, hipStream_t st)
{
    using G = ks::Geom<SF, 2, 1, fs::NW>;
    constexpr int STAGES = fs::TILES * G::STAGE, PARTS = fs::NW * G::PARTIAL, MAIN = STAGES > PARTS ? STAGES : PARTS, DRAWS = fs::MOST_ROWS * 128;
    constexpr int LDS = MAIN + fs::FOLD + DRAWS;
    S.lds_aux = MAIN;
    S.row_mul = reciprocal(S.dx.K >> 3);
    S.tiles = (unsigned)tiles(S.dx.M, S.dx.N, 32);
    const unsigned wgs = S.tiles + (unsigned)tiles(S.dw.M, S.dw.N, 64);
    if (out_dt == NVFP4_F32) {
        auto k = small_backward_kernel<DT, B, SF, NVFP4_F32>;
        static bool once = ((void)hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, LDS), true);
        (void)once;
        hipLaunchKernelGGL(k, dim3(wgs), dim3(fs::NT), LDS, st, S);
    } else {
        auto k = small_backward_kernel<DT, B, SF, NVFP4_BF16>;
        static bool once = ((void)hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, LDS), true);
        (void)once;
        hipLaunchKernelGGL(k, dim3(wgs), dim3(fs::NT), LDS, st, S);
    }
    return hipGetLastError();
}
hipError_t launch_small_backward(SmallBackward S, int dt, int block, int sf, int out_dt, hipStream_t st)
{
    (void)block;
    if (sf == NVFP4_SCALE_E8M0)
        return dt == NVFP4_BF16 ? launch_small_backward_fmt<NVFP4_BF16, 32, NVFP4_SCALE_E8M0>(S, out_dt, st) : launch_small_backward_fmt<NVFP4_F32, 32, NVFP4_SCALE_E8M0>(S, out_dt, st);
    return dt == NVFP4_BF16 ? launch_small_backward_fmt<NVFP4_BF16, 16, NVFP4_SCALE_E4M3>(S, out_dt, st) : launch_small_backward_fmt<NVFP4_F32, 16, NVFP4_SCALE_E4M3>(S, out_dt, st);
}

}  // namespace nvfp4
