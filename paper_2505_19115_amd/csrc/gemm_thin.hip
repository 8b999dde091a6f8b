// Block-scaled FP4 GEMM for up to 16 rows of A (generation: one token of each of a few sequences against a weight matrix), NVFP4 and MXFP4,
//     out[i, j] = gA gB sum_k cA[i,k] sA[i,k/B] cB[j,k] sB[j,k/B]        ("NT", as in gemm.hip),
// with A packed, or as a tensor that every workgroup quantizes for itself (rows, round to nearest).
//
// Such a product reads B once and does little else: its bound is the time in which the chip can bring B, and with MXFP4 it is reached
// (16 x 11008 x 4096 in slabs: 6.6 us, 24 MB at 5.5 TB/s and 2.3 us that any launch takes).  So there is one workgroup per CU, whose 8 or
// 16 waves divide the K tiles (wave w takes w, w + NW, ...) and request as many of theirs at once as the LDS holds, by direct global -> LDS
// loads, codes and scale bytes alike: with nothing staged in registers the loads in flight are counted, and a wave multiplies a K tile
// when that one is there.  The MFMA tile is 16 x 16: no rows computed that a 16-token call does not have.  The sums of the waves are added
// through the LDS in their order: the bits depend on the number of waves, which follows K and, past 12288 columns, N, and not on how A came
// or on the columns per workgroup otherwise.
// Two neighbouring lanes in a quad fetch two scale pieces of one row: with 16 rows across the lanes a scale load took the vector L1 64
// requests instead of 16 (16 x 11008 x 4096 MXFP4, row-major: 7.8 instead of 6.5 us).
// NVFP4 needs 8 vector instructions per 8 codes of B on top of that, 3 us of a CU's time at 16 x 11008 x 4096, of which 16 waves hide more
// than 8 (8.7 -> 8.0 us; contractions of up to 2048 are over sooner with 8: 16 x 11008 x 1024 4.2 / 3.7; MXFP4 up to 8192: 16 x 11008 x
// 4096 6.7 / 6.6, 16 x 4096 x 11008 7.3 / 7.8).
// us, bf16 outputs, the tile kernels (gemm_ksplit.hip, mostly 32 x 32) / this one:
//                         NVFP4, row-major   MXFP4, B in slabs
//     16 x   256 x 12288     12.2 /  7.5         7.5 /  5.3  (row-major)
//     16 x  4096 x  4096      6.9 /  4.9
//     16 x  4096 x 11008     12.1 /  9.6         8.4 /  7.3
//     16 x  8224 x  1024      5.0 /  3.4
//     16 x 11008 x  4096      9.9 /  8.0         7.2 /  6.6
//     16 x 12288 x 12288     31.5 / 26.4        19.1 / 17.4
//     16 x   256 x   256      3.3 /  2.5
#include "quantize_tile.h"

namespace nvfp4 {

// A that a workgroup quantizes itself: what fits the LDS beside the loads in flight.  us, a call with packed weights, quantizer and product
// in two launches / in one: NVFP4 1 x 4096 x 4096 9.4 / 6.4, 3 x 4096 x 4096 9.0 / 7.5, 1 x 11008 x 4096 10.6 / 10.6 (the product's arithmetic
// cannot begin before A is there), 1 x 4096 x 11008 12.4 / 12.4; MXFP4 1 x 11008 x 4096 8.6 / 7.1.  (All of a 16 x 4096 activation, by eight
// waves more: 17.9 instead of 12.9 for 16 x 11008 x 4096.)
constexpr int THIN_TENSOR_BYTES = 24 * 1024;

namespace thin {

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef int int8v_t __attribute__((ext_vector_type(8)));
typedef float float4v_t __attribute__((ext_vector_type(4)));
typedef float float2v_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

constexpr int KT = 128, KTB = 64;            // contraction elements and code bytes per row of a K tile
constexpr int PIECE = 1024 + 256;            // LDS bytes of 16 rows of a K tile: codes, then a dword of scale bytes per 32 codes
constexpr int PACKED = -1;                   // (in place of A's element type)
// A tensor's bytes; its codes and scale bytes; fold of the maximum and the tensor scale
constexpr int X_BYTES = THIN_TENSOR_BYTES, A_BYTES = 7 * 1024 + 768, MISC = 512;
// K tiles that each of the NW waves has in flight: as many as the LDS holds beside these
template <int DT, int NW, int TN>
constexpr int STAGES = (DT == PACKED ? (NW == 16 ? 8 : 15) : 96 / NW) / (TN + (DT == PACKED ? 1 : 0));

// 8 codes (one dword) of one block -> 8 fp16 values times the block scale (see gemm.hip)
__device__ __forceinline__ half8_t dequant8(uint32_t w, _Float16 s)
{
    const half2_t s2 = {s, s};
    half2_t h0 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 256.0f, 0) * s2;
    half2_t h1 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 256.0f, 1) * s2;
    half2_t h2 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 256.0f, 2) * s2;
    half2_t h3 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 256.0f, 3) * s2;
    half8_t r;
    r[0] = h0[0]; r[1] = h0[1]; r[2] = h1[0]; r[3] = h1[1];
    r[4] = h2[0]; r[5] = h2[1]; r[6] = h3[0]; r[7] = h3[1];
    return r;
}

// a barrier that waits for the LDS and not for loads in flight
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}
template <int N>
__device__ __forceinline__ void wait_loads()
{
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}
// waits until at most `left` K tiles (PER loads each) are outstanding, left <= MOST
template <int PER, int MOST>
__device__ __forceinline__ void wait_tiles(int left)
{
    if constexpr (MOST == 0) {
        wait_loads<0>();
    } else {
        if (left >= MOST) wait_loads<PER * MOST>();
        else wait_tiles<PER, MOST - 1>(left);
    }
}

}  // namespace thin

// A, which the workgroup has in its LDS as it came -> codes [K tile][row][64 bytes, swizzled] and scale bytes [K tile][row][KT / B];
// returns the tensor scale.  The arithmetic is that of the quantizers' row kernels.
template <int DT, int B, int SF, int NT>
__device__ __forceinline__ float thin_quantize(const uint8_t *raw, const int M, const int cpr, const uint32_t row_mul, uint8_t *codes, uint8_t *scales,
                                               uint32_t *fold)
{
    using namespace thin;
    constexpr bool MXS = SF == NVFP4_SCALE_E8M0;
    constexpr int LPB = B / 8, SPT = KT / B, U = (X_BYTES / (DT == NVFP4_BF16 ? 16 : 32) + NT - 1) / NT;
    const int total = M * cpr, tid = threadIdx.x;
    Chunk<DT> v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        v[u].zero();
        if (tid + u * NT < total) v[u].template load<false>(raw, (int64_t)(tid + u * NT) * 8);
    }
    float g = 1.0f, k = 0.0f;
    if (!MXS) {
        float a = 0.0f;
#pragma unroll
        for (int u = 0; u < U; ++u) a = fmaxf(a, chunk_amax(v[u]));
        a = group_max<16>(a);
        if ((tid & 15) == 0) fold[tid >> 4] = f2u(a);
        lds_barrier();
        uint32_t m = 0;
#pragma unroll
        for (int t = 0; t < NT / 16; ++t) m = umax(m, fold[t]);
        g = tensor_scale_from_amax(u2f(m));
        k = 1.0f / (6.0f * g);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int id = tid + u * NT, row = (int)__umulhi((uint32_t)id, row_mul), c = id - row * cpr;
        const float a = group_max<LPB>(MXS ? chunk_amax_packed(v[u]) : chunk_amax(v[u]));
        float q;
        const uint32_t sbyte = block_scale<SF, true, false>(a, g, k, &q);
        if (MXS) q = mx_scale_operand(sbyte);
        const uint32_t packed = chunk_codes_hw<DT, NVFP4_RTN, MXS>(v[u], q, 0, 0);
        if (id < total) {
            const int at = (c >> 4) * M + row;
            *reinterpret_cast<uint32_t *>(codes + at * KTB + ((((c >> 2) & 3) ^ ((row >> 2) & 3)) << 4) + (c & 3) * 4) = packed;
            if ((tid & (LPB - 1)) == 0) scales[at * SPT + (c & 15) / LPB] = (uint8_t)sbyte;
        }
    }
    return g;
}

template <int DT, int B, int SF, int NW, int TN, int OUT_DT>
__global__ __launch_bounds__(64 * NW) void gemm_nt_thin_kernel(GemmArgs P, const void *X, float *g_out, uint32_t row_mul)
{
    using namespace thin;
    constexpr bool MX = SF == NVFP4_SCALE_E8M0, FUSED = DT != PACKED;
    constexpr int G = TN + (FUSED ? 0 : 1), S = STAGES<DT, NW, TN>, RING = S * G * PIECE;  // pieces of a K tile (B's, then A's), ring of a wave
    constexpr int SPT = KT / B, BN = 16 * TN;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    uint8_t *const raw = lds + NW * RING, *const a_codes = raw + X_BYTES;
    uint32_t *const fold = reinterpret_cast<uint32_t *>(a_codes + A_BYTES);

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, h = lane >> 4;
    const int n0 = (int)blockIdx.x * BN;
    const int nkt = (int)((P.K + KT - 1) / KT), rem = (int)(P.K - (int64_t)(nkt - 1) * KT);
    const int M = (int)P.M, N = (int)P.N;
    uint8_t *const a_scales = a_codes + nkt * M * KTB;
    uint8_t *const ring = lds + wave * RING;

    const int64_t Kb = P.K >> 1, Ks = P.K / B;
    constexpr int64_t SB = MX ? SLAB_MX_SCALE_BYTES : SLAB_SCALE_BYTES;
    // ---- addresses, relative to the workgroup's first row of B and the first row of A; rows past the edge are the last row
    const int ch = (lane & 3) ^ ((lane >> 4) & 3);
    uint32_t coff[G], soff[G];
#pragma unroll
    for (int p = 0; p < G; ++p) {
        const bool isA = p == TN, slab = isA ? P.a_slab : P.b_slab;
        const int first = isA ? 0 : n0, rows = isA ? M : N, row0 = isA ? 0 : n0 + 16 * p;
        const int row = row0 + (lane >> 2) < rows ? row0 + (lane >> 2) : rows - 1;
        if (slab) {
            coff[p] = (uint32_t)(((row >> 8) - (first >> 8)) * nkt) * (uint32_t)SLAB_CODE_BYTES + (uint32_t)(slab_row(row & 255) * KTB + ch * 16);
            soff[p] = (uint32_t)(((row >> 8) - (first >> 8)) * nkt) * (uint32_t)SB + (uint32_t)(slab_row(row & 255) * SPT + (lane & 3) * (SPT / 4));
        } else {
            coff[p] = (uint32_t)((row - first) * Kb + ch * 16);
            soff[p] = (uint32_t)((row - first) * Ks + (lane & 3) * (SPT / 4));
        }
    }
    const uint8_t *const cB = P.b_slab ? P.B_codes + (int64_t)(n0 >> 8) * nkt * SLAB_CODE_BYTES : P.B_codes + n0 * Kb;
    const uint8_t *const sB = P.b_slab ? P.B_scales + (int64_t)(n0 >> 8) * nkt * SB : P.B_scales + n0 * Ks;
    const int64_t cstepB = P.b_slab ? SLAB_CODE_BYTES : KTB, sstepB = P.b_slab ? SB : SPT;
    const int64_t cstepA = P.a_slab ? SLAB_CODE_BYTES : KTB, sstepA = P.a_slab ? SB : SPT;
    typedef __attribute__((address_space(3))) void *lds_ptr_t;
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_ptr_t)ring);
    auto uniform_ptr = [](const uint8_t *p) -> const uint8_t * {
        const uint64_t v = reinterpret_cast<uint64_t>(p);
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
        return reinterpret_cast<const uint8_t *>(((uint64_t)hi << 32) | lo);
    };
    // inline assembly for the reason given in gemm.hip: a stage is read only after the counted wait for it.  Five wait states behind a
    // lane read that may have written the address.
    auto dma16 = [&](uint32_t lds_addr, uint32_t voff, const uint8_t *base) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds_addr), "v"(voff), "s"(base) : "memory", "m0");
    };
    // the scale bytes of a lane's 32 codes (two for NVFP4, one for MXFP4), to its dword
    auto dma_scale = [&](uint32_t lds_addr, uint32_t voff, const uint8_t *base) {
        if constexpr (MX) asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tglobal_load_lds_ubyte %1, %2" : : "s"(lds_addr), "v"(voff), "s"(base) : "memory", "m0");
        else asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tglobal_load_lds_ushort %1, %2" : : "s"(lds_addr), "v"(voff), "s"(base) : "memory", "m0");
    };
    auto fetch = [&](int i, int stage) {
        const int kt = wave + i * NW;
        const bool tail = kt == nkt - 1 && rem < KT;
        // a missing chunk of the last tile is replaced by the tile's first (A's is zeroed below)
        const uint32_t cback = tail && ch * 32 >= rem ? (uint32_t)ch * 16 : 0u, sback = tail && (lane & 3) * 32 >= rem ? (uint32_t)(lane & 3) * (SPT / 4) : 0u;
        const uint8_t *const uc = uniform_ptr(cB + kt * cstepB), *const us = uniform_ptr(sB + kt * sstepB);
        const uint32_t dst = lds0 + stage * (G * PIECE);
#pragma unroll
        for (int p = 0; p < TN; ++p) {
            dma16(dst + p * PIECE, coff[p] - cback, uc);
            dma_scale(dst + p * PIECE + 1024, soff[p] - sback, us);
        }
        if (!FUSED) {
            dma16(dst + TN * PIECE, coff[G - 1] - cback, uniform_ptr(P.A_codes + kt * cstepA));
            dma_scale(dst + TN * PIECE + 1024, soff[G - 1] - sback, uniform_ptr(P.A_scales + kt * sstepA));
        }
    };
    float4v_t acc[TN];
#pragma unroll
    for (int p = 0; p < TN; ++p) acc[p] = float4v_t{0, 0, 0, 0};
    const int ar = r < M ? r : M - 1;
    const int slot = r * KTB + ((h ^ ((r >> 2) & 3)) << 4), aslot = ar * KTB + ((h ^ ((ar >> 2) & 3)) << 4);
    auto compute = [&](int i, int stage) {
        const int kt = wave + i * NW;
        const bool none = kt == nkt - 1 && h * 32 >= rem;
        const uint8_t *const s = ring + stage * (G * PIECE);
        uint4 ca, cb[TN];
        uint32_t sa, sb[TN];
        if (FUSED) {
            ca = *reinterpret_cast<const uint4 *>(a_codes + kt * M * KTB + aslot);
            const uint8_t *const as = a_scales + (kt * M + ar) * SPT + h * (SPT / 4);
            sa = MX ? *as : *reinterpret_cast<const uint16_t *>(as);
        } else {
            ca = *reinterpret_cast<const uint4 *>(s + TN * PIECE + slot);
            sa = *reinterpret_cast<const uint32_t *>(s + TN * PIECE + 1024 + (4 * r + h) * 4);
        }
        if (none) {
            ca = make_uint4(0, 0, 0, 0);
            sa = 0;
        }
#pragma unroll
        for (int p = 0; p < TN; ++p) {
            cb[p] = *reinterpret_cast<const uint4 *>(s + p * PIECE + slot);
            sb[p] = *reinterpret_cast<const uint32_t *>(s + p * PIECE + 1024 + (4 * r + h) * 4);
        }
        if constexpr (MX) {
            const int8v_t va = {(int)ca.x, (int)ca.y, (int)ca.z, (int)ca.w, 0, 0, 0, 0};
#pragma unroll
            for (int p = 0; p < TN; ++p) {
                const int8v_t vb = {(int)cb[p].x, (int)cb[p].y, (int)cb[p].z, (int)cb[p].w, 0, 0, 0, 0};
                acc[p] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(vb, va, acc[p], 4, 4, 0, (int)sb[p], 0, (int)sa);
            }
        } else {
            // scale bytes -> fp16(scale * 2^-8) pairs, as in gemm.hip; dword t of the chunk belongs to its block t / 2
            auto pair = [](uint32_t two) { return __builtin_bit_cast(half2_t, __builtin_amdgcn_perm(0, two, 0x0C010C00u) << 7); };
            auto dword = [](const uint4 &w, int t) { return t == 0 ? w.x : t == 1 ? w.y : t == 2 ? w.z : w.w; };
            const half2_t pa = pair(sa);
            half8_t fa[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) fa[t] = dequant8(dword(ca, t), pa[t >> 1]);
#pragma unroll
            for (int p = 0; p < TN; ++p) {
                const half2_t pb = pair(sb[p]);
#pragma unroll
                for (int t = 0; t < 4; ++t) acc[p] = __builtin_amdgcn_mfma_f32_16x16x32_f16(dequant8(dword(cb[p], t), pb[t >> 1]), fa[t], acc[p], 0, 0, 0);
            }
        }
    };

    const int tiles = nkt > wave ? (nkt - wave + NW - 1) / NW : 0;
    float g = 1.0f;
    if constexpr (FUSED) {
        // A first: it is there before any of B's pieces, and is quantized while those arrive
        const int bytes = M * (int)P.K * (DT == NVFP4_BF16 ? 2 : 4);
        const uint32_t raw0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_ptr_t)raw);
#pragma unroll
        for (int u = 0; u < (X_BYTES + 1024 * NW - 1) / (1024 * NW); ++u) {
            // (lanes past the end fetch the last 16 bytes once more)
            const int at = (u * NW + wave) * 1024;
            if (at < bytes) dma16(raw0 + at, (uint32_t)(at + lane * 16 < bytes ? at + lane * 16 : bytes - 16), uniform_ptr(static_cast<const uint8_t *>(X)));
        }
    }
    for (int i = 0; i < S && i < tiles; ++i) fetch(i, i);
    if constexpr (FUSED) {
        wait_tiles<2 * G, S>(tiles < S ? tiles : S);
        lds_barrier();
        g = thin_quantize<DT, B, SF, 64 * NW>(raw, M, (int)(P.K >> 3), row_mul, a_codes, a_scales, fold);
        lds_barrier();
        if (blockIdx.x == 0 && threadIdx.x == 0) *g_out = g;
    }
    int stage = 0;
    for (int i = 0; i < tiles; ++i) {
        wait_tiles<2 * G, S - 1>(tiles - 1 - i);
        compute(i, stage);
        if (i + S < tiles) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // (the stage has been read)
            fetch(i + S, stage);
        }
        stage = stage + 1 == S ? 0 : stage + 1;
    }
    // ---- partial sums: element e of lane (r, h), piece p is row r, column 16 p + 4 h + e
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int p = 0; p < TN; ++p) *reinterpret_cast<float4v_t *>(ring + p * 1024 + lane * 16) = acc[p];
    __syncthreads();
    const int t = threadIdx.x;
    if (t >= 64 * TN) return;
    float4v_t y = {0, 0, 0, 0};
#pragma unroll
    for (int w = 0; w < NW; ++w) y += *reinterpret_cast<const float4v_t *>(lds + w * RING + t * 16);
    const int col = n0 + 16 * (t >> 6) + 4 * h;
    if (r >= M || col >= N) return;
    y *= (FUSED ? g : *P.gA) * *P.gB;
    const bool whole = col + 4 <= N && (P.ldc & 3) == 0;
    if (OUT_DT == NVFP4_F32) {
        float *const dst = reinterpret_cast<float *>(P.out) + r * P.ldc + col;
        if (whole) {
            *reinterpret_cast<float4v_t *>(dst) = y;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (col + e < N) dst[e] = y[e];
        }
    } else {
        const float2v_t lo = {y[0], y[1]}, hi = {y[2], y[3]};
        const uint32_t w0 = __builtin_bit_cast(uint32_t, __builtin_convertvector(lo, bf16x2_t)), w1 = __builtin_bit_cast(uint32_t, __builtin_convertvector(hi, bf16x2_t));
        uint16_t *const dst = reinterpret_cast<uint16_t *>(P.out) + r * P.ldc + col;
        if (whole) {
            *reinterpret_cast<uint2 *>(dst) = make_uint2(w0, w1);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (col + e < N) dst[e] = (uint16_t)((e & 2 ? w1 : w0) >> (16 * (e & 1)));
        }
    }
}

// ------------------------------------------------------------------ host side

bool gemm_is_thin(int64_t M, int64_t N, int64_t K, int block, int sf)
{
    // (512 threads per 64 columns, and those of a launch are counted in 32 bits)
    constexpr int64_t MOST_N = (int64_t)(0xFFFFFFFFu / 512) * 64;
    // one round of workgroups, or a contraction that is worth more (us, the tile kernels / this one: NVFP4 1 x 65536 x 128 5.2 / 8.5, 16 x 65536 x
    // 512 12.9 / 11.8, 16 x 131072 x 1024 36.0 / 29.2; MXFP4 16 x 65536 x 512 7.1 / 9.9, 4 x 131072 x 4096 58.4 / 59.5)
    return M <= 16 && (N <= 64 * 256 || (sf == NVFP4_SCALE_E4M3 && K >= 512 && N <= MOST_N)) && ((block == 16 && sf == NVFP4_SCALE_E4M3) || (block == 32 && sf == NVFP4_SCALE_E8M0));
}
bool thin_takes_tensor(int64_t M, int64_t K, int dt) { return M <= 16 && M * K * (dt == NVFP4_BF16 ? 2 : 4) <= THIN_TENSOR_BYTES; }

template <int DT, int B, int SF, int NW, int TN>
static void launch_thin(const GemmArgs &P, const void *X, float *g_out, int out_dt, hipStream_t st)
{
    using namespace thin;
    constexpr bool FUSED = DT != PACKED;
    constexpr int LDS = NW * STAGES<DT, NW, TN> * (TN + (FUSED ? 0 : 1)) * PIECE + (FUSED ? X_BYTES + A_BYTES + MISC : 0);
    static_assert(LDS <= 160 * 1024, "LDS of a CU");
    const dim3 grid((unsigned)((P.N + 16 * TN - 1) / (16 * TN))), wg(64 * NW);
    const uint32_t row_mul = (uint32_t)(((uint64_t)1 << 32) / (uint64_t)(P.K >> 3)) + 1u;
    if (out_dt == NVFP4_F32) {
        auto k = gemm_nt_thin_kernel<DT, B, SF, NW, TN, NVFP4_F32>;
        static bool once = ((void)hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, LDS), true);
        (void)once;
        hipLaunchKernelGGL(k, grid, wg, LDS, st, P, X, g_out, row_mul);
    } else {
        auto k = gemm_nt_thin_kernel<DT, B, SF, NW, TN, NVFP4_BF16>;
        static bool once = ((void)hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, LDS), true);
        (void)once;
        hipLaunchKernelGGL(k, grid, wg, LDS, st, P, X, g_out, row_mul);
    }
}
template <int DT, int B, int SF>
static hipError_t launch_thin_tile(const GemmArgs &P, const void *X, float *g_out, int out_dt, hipStream_t st)
{
    // the narrowest columns that take one round of the 256 CUs; the lines between 8 and 16 waves: above
    const int64_t pieces = (P.N + 15) / 16;
    if (pieces > 3 * 256) {
        launch_thin<DT, B, SF, 8, 4>(P, X, g_out, out_dt, st);
    } else if (P.K > (SF == NVFP4_SCALE_E4M3 ? 2048 : 8192)) {
        if (pieces <= 256) launch_thin<DT, B, SF, 16, 1>(P, X, g_out, out_dt, st);
        else if (pieces <= 512) launch_thin<DT, B, SF, 16, 2>(P, X, g_out, out_dt, st);
        else launch_thin<DT, B, SF, 16, 3>(P, X, g_out, out_dt, st);
    } else {
        if (pieces <= 256) launch_thin<DT, B, SF, 8, 1>(P, X, g_out, out_dt, st);
        else if (pieces <= 512) launch_thin<DT, B, SF, 8, 2>(P, X, g_out, out_dt, st);
        else launch_thin<DT, B, SF, 8, 3>(P, X, g_out, out_dt, st);
    }
    return hipGetLastError();
}
hipError_t launch_gemm_thin(const GemmArgs &P, int sf, int out_dt, hipStream_t st)
{
    return sf == NVFP4_SCALE_E8M0 ? launch_thin_tile<thin::PACKED, 32, NVFP4_SCALE_E8M0>(P, nullptr, nullptr, out_dt, st)
                                  : launch_thin_tile<thin::PACKED, 16, NVFP4_SCALE_E4M3>(P, nullptr, nullptr, out_dt, st);
}
hipError_t launch_gemm_thin_tensor(const GemmArgs &P, const void *X, int dt, float *g_out, int sf, int out_dt, hipStream_t st)
{
    if (sf == NVFP4_SCALE_E8M0)
        return dt == NVFP4_BF16 ? launch_thin_tile<NVFP4_BF16, 32, NVFP4_SCALE_E8M0>(P, X, g_out, out_dt, st)
                                : launch_thin_tile<NVFP4_F32, 32, NVFP4_SCALE_E8M0>(P, X, g_out, out_dt, st);
    return dt == NVFP4_BF16 ? launch_thin_tile<NVFP4_BF16, 16, NVFP4_SCALE_E4M3>(P, X, g_out, out_dt, st)
                            : launch_thin_tile<NVFP4_F32, 16, NVFP4_SCALE_E4M3>(P, X, g_out, out_dt, st);
}

}  // namespace nvfp4
