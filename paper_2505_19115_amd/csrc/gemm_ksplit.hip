// Block-scaled FP4 GEMM for outputs too small, or contractions too ragged, for the 256 x 256 kernels: few tokens against
// a large weight matrix, layers of a small network, K that is no multiple of 128.
//     out[i, j] = gA gB sum_k cA[i,k] sA[i,k/B] cB[j,k] sB[j,k/B]        ("NT", as in gemm.hip and gemm_mx.hip)
//
// What bounds such a product is not the matrix pipe but how many bytes the chip has in flight and how long one
// workgroup's serial walk along K takes: with one 128 x 128 or 256 x 256 tile per workgroup a 16-token product runs on
// 16 or 86 of the 256 CUs, each waiting for one K tile after the other.  So here the NW waves of a workgroup share one
// small output tile and divide the CONTRACTION: wave w multiplies the 128-wide K tiles w, w + NW, w + 2 NW, ...  A wave
// stages its own K tiles in its own part of the LDS (direct global -> LDS loads, two stages) and reads nothing another
// wave has loaded, so the K loop has no barrier at all; at the end the NW partial tiles are added through the LDS in the
// order of the waves (deterministic), scaled and stored.
//
// Operands: row-major or slab (kernels.h), each for itself.  Rows past the edge are clamped to the last row (their
// products land in outputs that are never stored).  A last K tile of 32, 64 or 96 elements reads a valid chunk in place of
// each missing one and multiplies it by zero: by zero scales (E4M3), or with the A codes zeroed (E8M0).
#include "gemm_ksplit.h"

namespace nvfp4 {

template <int SF, int B, int TA, int TB, int NW, int OUT_DT>
__device__ __forceinline__ void ksplit_tile(const GemmArgs &P, const int wg)
{
    using namespace ks;
    using G = Geom<SF, TA, TB, NW>;
    constexpr bool MX = SF == NVFP4_SCALE_E8M0;
    constexpr int BM = G::BM, BN = G::BN, ROWS = G::ROWS;
    constexpr int SPT = KT / B;                // scale bytes per row and K tile
    constexpr int NI = ROWS / 16;              // direct-to-LDS instructions per stage (16 rows each)
    constexpr int NSR = (ROWS + 63) / 64;      // scale rows per lane
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ntx = (int)((P.N + BN - 1) / BN), nty = (int)((P.M + BM - 1) / BM);
    int ty, tx;
    tile_coords(wg, ntx, nty, ty, tx);
    const int64_t m0 = (int64_t)ty * BM, n0 = (int64_t)tx * BN;
    const int64_t Kb = P.K >> 1, Ks = P.K / B;
    const int nkt = (int)((P.K + KT - 1) / KT);
    const int rem = (int)(P.K - (int64_t)(nkt - 1) * KT);  // elements of the last K tile
    uint8_t *const mine = lds + wave * (2 * G::STAGE);

    float16_t acc[TA][TB];
#pragma unroll
    for (int a = 0; a < TA; ++a)
#pragma unroll
        for (int b = 0; b < TB; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.0f;

    // ---- addresses.  A code instruction fills 1 KB = 16 consecutive tile rows; lane i lands at byte 16 i (row i / 4,
    // slot i % 4) and fetches the chunk the XOR swizzle puts there.  Offsets are relative to the tile's first row (32 bits).
    const int ch = (lane & 3) ^ ((lane >> 4) & 3);
    uint32_t off[NI];
#pragma unroll
    for (int u = 0; u < NI; ++u) {
        const int row = 16 * u + (lane >> 2);
        const bool isA = 16 * u < BM;
        const int64_t base = isA ? m0 : n0, rows = isA ? P.M : P.N;
        const int lrow = isA ? row : row - BM;
        const int64_t lr = base + lrow < rows ? lrow : rows - 1 - base;
        const bool slab = isA ? P.a_slab : P.b_slab;
        off[u] = slab ? (uint32_t)(slab_row((int)(base & 255) + lrow) * 64 + ch * 16) : (uint32_t)(lr * Kb + ch * 16);
    }
    const uint8_t *const baseA = P.a_slab ? P.A_codes + (m0 >> 8) * nkt * SLAB_CODE_BYTES : P.A_codes + m0 * Kb;
    const uint8_t *const baseB = P.b_slab ? P.B_codes + (n0 >> 8) * nkt * SLAB_CODE_BYTES : P.B_codes + n0 * Kb;
    const int64_t stepA = P.a_slab ? SLAB_CODE_BYTES : KTB, stepB = P.b_slab ? SLAB_CODE_BYTES : KTB;
    const uint8_t *sptr[NSR];
    int sstep[NSR];
    bool sgo[NSR];
#pragma unroll
    for (int i = 0; i < NSR; ++i) {
        const int row = lane + 64 * i;
        sgo[i] = row < ROWS;
        const bool isA = row < BM;
        const int64_t base = isA ? m0 : n0, rows = isA ? P.M : P.N;
        const int lrow = isA ? row : row - BM;
        const uint8_t *const s = isA ? P.A_scales : P.B_scales;
        if (isA ? P.a_slab : P.b_slab) {
            constexpr int64_t SB = MX ? SLAB_MX_SCALE_BYTES : SLAB_SCALE_BYTES;
            sptr[i] = s + (base >> 8) * nkt * SB + slab_row(((int)(base & 255) + lrow) & 255) * SPT;
            sstep[i] = (int)SB;
        } else {
            sptr[i] = s + (base + lrow < rows ? base + lrow : rows - 1) * Ks;
            sstep[i] = SPT;
        }
    }

    typedef __attribute__((address_space(3))) void *lds_ptr_t;
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_ptr_t)mine);
    auto uniform_ptr = [](const uint8_t *p) -> const uint8_t * {
        const uint64_t v = reinterpret_cast<uint64_t>(p);
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
        return reinterpret_cast<const uint8_t *>(((uint64_t)hi << 32) | lo);
    };
    // inline assembly for the reason given in gemm.hip: the stage is read only after the explicit wait below
    auto dma16 = [&](uint32_t lds_addr, uint32_t voff, const uint8_t *base) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds_addr), "v"(voff), "s"(base) : "memory", "m0");
    };
    uint64_t gs[NSR];  // the fetched K tile's scale bytes of this lane's rows
    auto fetch = [&](int kt, int stage) {
        const bool tail = kt == nkt - 1 && rem < KT;
#pragma unroll
        for (int i = 0; i < NSR; ++i) {
            if (!sgo[i]) continue;
            const uint8_t *sp = sptr[i] + (int64_t)kt * sstep[i];
            uint64_t v = 0;
            if (!tail) {
                // (row-major scale rows of a ragged K start at any byte)
                if (SPT == 8) __builtin_memcpy(&v, sp, 8);
                else if (SPT == 4) { uint32_t w; __builtin_memcpy(&w, sp, 4); v = w; }
                else if (SPT == 2) { uint16_t w; __builtin_memcpy(&w, sp, 2); v = w; }
                else v = *sp;
            } else {
#pragma unroll
                for (int t = 0; t < SPT; ++t)
                    if (t * B < rem) v |= (uint64_t)sp[t] << (8 * t);
            }
            gs[i] = v;
        }
        const uint8_t *const ua = uniform_ptr(baseA + kt * stepA), *const ub = uniform_ptr(baseB + kt * stepB);
        // a missing chunk of the last tile is replaced by the tile's first
        const uint32_t back = tail && ch * 32 >= rem ? (uint32_t)ch * 16 : 0u;
#pragma unroll
        for (int u = 0; u < NI; ++u) dma16(lds0 + stage * G::STAGE + u * 1024, off[u] - back, 16 * u < BM ? ua : ub);
    };
    auto stash_scales = [&](int stage) {
        uint32_t *const sS = reinterpret_cast<uint32_t *>(mine + stage * G::STAGE + G::CODES);
#pragma unroll
        for (int i = 0; i < NSR; ++i) {
            if (!sgo[i]) continue;
            const uint32_t lo = (uint32_t)gs[i], hi = (uint32_t)(gs[i] >> 32);
            if (MX) {
                sS[lane + 64 * i] = lo;
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) {  // scale bytes -> fp16(scale * 2^-8) pairs, as in gemm.hip
                    const uint32_t sel = 0x0C000C00u | (uint32_t)((32 * j) / B) | ((uint32_t)((32 * j + 16) / B) << 16);
                    sS[j * ROWS + lane + 64 * i] = __builtin_amdgcn_perm(hi, lo, sel) << 7;
                }
            }
        }
    };
    int stage = 0;
    if (wave < nkt) fetch(wave, 0);
    for (int kt = wave; kt < nkt; kt += NW) {
        // this wave's loads of tile kt have landed, and its reads of the other stage (the last trip's) are done before fetch() has
        // that stage overwritten
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        stash_scales(stage);
        if (kt + NW < nkt) fetch(kt + NW, stage ^ 1);
        // (compute() reads scales that other lanes of the wave stored: the LDS keeps a wave's order, and so must the compiler)
        asm volatile("" ::: "memory");
        ksplit_compute<SF, TA, TB, NW>(mine + stage * G::STAGE, kt == nkt - 1 && rem < KT, rem, acc, lane);
        stage ^= 1;
    }

    ksplit_finish<SF, TA, TB, NW, OUT_DT>(P, acc, lds, m0, n0, [&]() { return P.gA[0] * P.gB[0]; });
}

// One product, or two that do not depend on each other (a backward call's dX and dW) in one launch: the first `tiles`
// workgroups take P0.  Products this small are over in one latency: 3.4 us less per backward call of a 64 x 256 x 128 layer.
template <int SF, int B, int TA, int TB, int NW, int OUT_DT>
__global__ __launch_bounds__(64 * NW) void gemm_nt_ksplit_kernel(GemmArgs P0, GemmArgs P1, unsigned tiles)
{
    const bool first = blockIdx.x < tiles;
    ksplit_tile<SF, B, TA, TB, NW, OUT_DT>(first ? P0 : P1, (int)(first ? blockIdx.x : blockIdx.x - tiles));
}

template <int SF, int B, int TA, int TB, int NW>
static void launch_cfg(const GemmArgs &P, const GemmArgs *P1, int out_dt, hipStream_t st)
{
    using G = ks::Geom<SF, TA, TB, NW>;
    auto count = [](const GemmArgs &Q) { return (unsigned)(((Q.N + G::BN - 1) / G::BN) * ((Q.M + G::BM - 1) / G::BM)); };
    const unsigned tiles = count(P), ntiles = tiles + (P1 ? count(*P1) : 0u);
    const GemmArgs &Q = P1 ? *P1 : P;
    if (out_dt == NVFP4_F32) {
        auto k = gemm_nt_ksplit_kernel<SF, B, TA, TB, NW, NVFP4_F32>;
        static bool once = ((void)hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, G::LDS), true);
        (void)once;
        hipLaunchKernelGGL(k, dim3(ntiles), dim3(64 * NW), G::LDS, st, P, Q, tiles);
    } else {
        auto k = gemm_nt_ksplit_kernel<SF, B, TA, TB, NW, NVFP4_BF16>;
        static bool once = ((void)hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, G::LDS), true);
        (void)once;
        hipLaunchKernelGGL(k, dim3(ntiles), dim3(64 * NW), G::LDS, st, P, Q, tiles);
    }
}
template <int SF, int B>
static void launch_tile(const GemmArgs &P, const GemmArgs *P1, GemmTile tile, int out_dt, hipStream_t st)
{
    switch (tile) {
    case TILE_32x32: launch_cfg<SF, B, 1, 1, 8>(P, P1, out_dt, st); break;
    case TILE_32x64: launch_cfg<SF, B, 1, 2, 8>(P, P1, out_dt, st); break;
    case TILE_64x32: launch_cfg<SF, B, 2, 1, 8>(P, P1, out_dt, st); break;
    default: launch_cfg<SF, B, 2, 2, 4>(P, P1, out_dt, st); break;
    }
}

hipError_t launch_gemm_ksplit(const GemmArgs &P, const GemmArgs *P1, GemmTile tile, int block, int sf, int out_dt, hipStream_t st)
{
    if (sf == NVFP4_SCALE_E8M0) {
        launch_tile<NVFP4_SCALE_E8M0, 32>(P, P1, tile, out_dt, st);
        return hipGetLastError();
    }
    switch (block) {
    case 16: launch_tile<NVFP4_SCALE_E4M3, 16>(P, P1, tile, out_dt, st); break;
    case 32: launch_tile<NVFP4_SCALE_E4M3, 32>(P, P1, tile, out_dt, st); break;
    case 64: launch_tile<NVFP4_SCALE_E4M3, 64>(P, P1, tile, out_dt, st); break;
    case 128: launch_tile<NVFP4_SCALE_E4M3, 128>(P, P1, tile, out_dt, st); break;
    default: return hipErrorNotSupported;
    }
    return hipGetLastError();
}

}  // namespace nvfp4
