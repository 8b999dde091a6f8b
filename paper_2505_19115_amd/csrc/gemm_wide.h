// Block-scaled FP4 products with E4M3 scales on four waves of 16 TA x 128 outputs, one wave per SIMD: the products of gemm.hip on
// v_mfma_f32_16x16x32_f16, for workgroup tiles of 256 x 256, 192 x 256, 160 x 256 (2 x 2 waves) and 128 x 256 (two groups of 1 x 2 waves on every
// other K tile).  Operands, layouts and arithmetic are those described there.
//
// What bounds them: the instructions of the one wave a SIMD has, which issues one every 5.8 to 6 cycles, at a clock that the matrix unit's power sets (2.05 to
// 2.3 GHz), and a start and an end of 22000 cycles a tile that nothing covers.  Counted (two lengths of K where there is a K tile's share; instructions
// of all kinds and cycles of a wave for each K tile of its own, of these MFMAs, 16 cycles each):
//     256 x 256                                                       838 instructions  4850 cycles  4096 in MFMAs (pipe busy 53 % of a launch with 16 K tiles, 73 % with 86)
//     128 x 256 in two groups                                         866               5170         4096 (51 % with 32 K tiles, 64 % with 86)
//     160 x 256 (from 32 K tiles, start and end as in the others)     630               3700         2560 (47 % with 32)
// Expanding the operands takes 8 (TA + 8) / (8 TA) vector instructions per MFMA of 16 cycles, 2 for TA = 8 (eight waves of 128 x 64 need 3, shared by
// two waves).  Measured with registers only, operands of quantized normal numbers, all 256 CUs, PFLOP/s:
//     32 x 32 x 16, eight waves of 128 x 64, each convert right before its multiply 1.57, four converts and then four multiplies 1.63
//     the same, four waves of 128 x 128                                             1.68                                          1.74
//     16 x 16 x 32, eight waves of 128 x 64                                         1.63                                          1.66
//     16 x 16 x 32, four waves of 128 x 128                                         1.76                                          1.98
// The 16 x 16 instruction does the same work with less power (the accumulators are read and written once per 32 products, not 16), and
// converts and multiplies in fours leave no instruction waiting for the one before.
// (A header, so that each block size is compiled by itself: gemm_wide16.hip to gemm_wide128.hip.)
#pragma once
#include <type_traits>
#include <utility>

#include "gemm_fold.h"
#include "kernels.h"
#include "nvfp4_math.h"
#include "store_lines.h"

namespace nvfp4 {

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef float float4v_t __attribute__((ext_vector_type(4)));

namespace wide {

constexpr int KT = 128, KTB = 64, TB = 8;  // K tile, bytes of codes per row and K tile, fragments of B per wave

// Written as assembly so that the accumulators stay where they are: with 64 of them the compiler moves the builtin's between the two halves of
// the register file.  What it cannot know about it: an operand must not have been written by the vector ALU in the two instructions before, and
// the result of the last one must not be read for 11 wait states.
__device__ __forceinline__ void mfma_16x16x32(float4v_t &acc, const u32x4_t &b, const u32x4_t &a)
{
    asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(acc) : "v"(b), "v"(a));
}

// f(0), ..., f(N - 1) with the number as a type: 256 MFMAs with all that goes between them are too much for the compiler's own unrolling
template <class F, int... I>
__device__ __forceinline__ void static_for_each(std::integer_sequence<int, I...>, F &&f)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F &&f)
{
    static_for_each(std::make_integer_sequence<int, N>{}, f);
}

template <int WM, int WN, int KG, int TA>
struct Geom {
    static constexpr int NW = WM * WN, NT = 64 * NW, BM = 16 * TA * WM, BN = 16 * TB * WN, ROWS = BM + BN;
    static constexpr int NSR = (ROWS + NT - 1) / NT;                   // scale rows per thread (the last ones may repeat the last row)
    static constexpr int SBLOCKS = WM * ((TA + 3) / 4) + WN * (TB / 4);  // scales in the LDS: 1 KB for each four fragments of a wave
    static constexpr int STAGE = ROWS * KTB + SBLOCKS * 1024;          // codes, then scales
    static constexpr int IN = TA % 2 == 0 ? 2 : 1, S = TA / IN;        // tile rows per strip of the epilogue, strips
    static constexpr int STAGES = KG * 2 * STAGE, PIECES = 4 * 16 * IN * 16 * TB * 4, FOLD = KG == 1 ? 0 : KG / 2 * BM * BN * 4;
    static constexpr int LDS = STAGES > PIECES ? (STAGES > FOLD ? STAGES : FOLD) : (PIECES > FOLD ? PIECES : FOLD);
    static_assert(WM * WN * KG == 4 && LDS <= 160 * 1024, "four waves, the LDS of a CU");
};

}  // namespace wide

// The tile whose first output is (m0, n0)
template <int B, int WM, int WN, int KG, int TA, int OUT_DT, bool KTAIL>
__device__ __forceinline__ void wide_tile(const TileArgs &P, uint8_t *const lds, const int64_t m0, const int64_t n0)
{
    using namespace wide;
    using G = Geom<WM, WN, KG, TA>;
    constexpr int NW = G::NW, NT = G::NT, BM = G::BM, ROWS = G::ROWS, NSR = G::NSR, STAGE = G::STAGE, IN = G::IN, S = G::S;
    constexpr int SPT = KT / B;       // scale bytes per row and K tile in global memory
    constexpr int WINDOW = 8 / SPT;   // row-major scales come 8 bytes at a time: those of so many K tiles
    constexpr bool WINDOWS = KTAIL || WINDOW > 1;
    constexpr int NI = ROWS / 16, CI = (NI + NW - 1) / NW;  // direct loads of a K tile, 16 rows each: A's, then B's; per wave
    constexpr bool EVEN = TA * WM % NW == 0 && TB * WN % NW == 0;  // each wave loads as many of A as the others, and of B
    constexpr int CA = TA * WM / NW, CB = TB * WN / NW;

    const int lane = threadIdx.x & 63;
    const int wave_wg = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int group = KG == 1 ? 0 : wave_wg / NW, wave = wave_wg - group * NW, tid = wave * 64 + lane;  // (inside the group from here on)
    const int wm = wave / WN, wn = wave % WN;
    const int r = lane & 15, g = lane >> 4;
    const int64_t Kb = P.K >> 1, Ks = P.K / B;
    const int nkt = (int)((P.K + KT - 1) / KT);
    const int steps = (nkt + KG - 1) / KG;            // K tiles that every group walks: j KG + group
    const int own = (nkt - group + KG - 1) / KG;      // (of which the last may not be there: its scales are zeros)

    float4v_t acc[S][IN * TB];
#pragma unroll
    for (int a = 0; a < S; ++a)
#pragma unroll
        for (int b = 0; b < IN * TB; ++b) acc[a][b] = float4v_t{0.0f, 0.0f, 0.0f, 0.0f};

    // ---- global -> LDS, codes: lane i of a load lands at byte 16 i (row i / 4, slot i % 4) of 16 rows, so the swizzle is applied by choosing which
    // chunk the lane fetches.  Rows past the edge are clamped to the last one.  A K tail is handled through the scales alone: a chunk past K
    // is replaced by the tile's first one and meets the zeros that follow the row's last scale byte.
    constexpr bool SPAN = 256 % BM != 0;  // A's rows may lie in two slabs
    auto piece = [&](int u) { return !EVEN ? (u * NW + wave < NI ? u * NW + wave : NI - 1) : u < CA ? wave * CA + u : BM / 16 + wave * CB + u - CA; };
    uint32_t off[CI];
    const int ch = (lane & 3) ^ quad_xor(lane >> 4);
#pragma unroll
    for (int u = 0; u < CI; ++u) {
        const int trow = piece(u) * 16 + (lane >> 2);  // row of the tile: A's, then B's
        const bool isA = EVEN ? u < CA : trow < BM;
        const int row = isA ? trow : trow - BM;
        const int64_t base = isA ? m0 : n0, rows = isA ? P.M : P.N;
        const int64_t lr = base + row < rows ? row : rows - 1 - base;  // row inside the tile, clamped
        // (a slab holds all rows of a 256- or 128-row tile: nothing to clamp; one of 96, 160 or 192 rows may reach into the next slab)
        const int srow = (int)(base & 255) + (int)(SPAN && isA ? lr : row);
        const uint32_t slab_off = (uint32_t)(slab_row(SPAN && isA ? srow & 255 : srow) * 64 + ch * 16) +
                                  (SPAN && isA && srow > 255 ? (uint32_t)nkt * (uint32_t)SLAB_CODE_BYTES : 0u);
        off[u] = (isA ? P.a_slab : P.b_slab) ? slab_off : (uint32_t)(lr * Kb + ch * 16);  // (relative to the tile's first row: 32 bits suffice)
    }
    typedef __attribute__((address_space(3))) void *lds_ptr_t;
    uint8_t *const stages = lds + group * (2 * STAGE);
    auto uniform_ptr = [](const uint8_t *p) -> const uint8_t * {
        const uint64_t v = reinterpret_cast<uint64_t>(p);
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
        return reinterpret_cast<const uint8_t *>(((uint64_t)hi << 32) | lo);
    };
    // Inline assembly, since the compiler would wait for a direct load before the next LDS read; in two parts, the destination (m0) and, at
    // least one instruction later, the load.  Load u of the wave: piece(u), 1 KB per piece.
    auto load_dst = [&](auto stc, int u) {
        constexpr int ST = decltype(stc)::value;
        const uint32_t base = (uint32_t)(uintptr_t)(lds_ptr_t)stages + piece(u) * 1024;
        asm volatile("s_add_u32 m0, %0, %1" : : "s"(__builtin_amdgcn_readfirstlane(base)), "n"(ST * STAGE) : "scc", "m0");
    };
    const uint8_t *const firstA = uniform_ptr(P.a_slab ? P.A_codes + (m0 >> 8) * nkt * SLAB_CODE_BYTES : P.A_codes + m0 * Kb);
    const uint8_t *const firstB = uniform_ptr(P.b_slab ? P.B_codes + (n0 >> 8) * nkt * SLAB_CODE_BYTES : P.B_codes + n0 * Kb);
    const uint32_t stepA = (uint32_t)__builtin_amdgcn_readfirstlane(P.a_slab ? (int)SLAB_CODE_BYTES : KTB),
                   stepB = (uint32_t)__builtin_amdgcn_readfirstlane(P.b_slab ? (int)SLAB_CODE_BYTES : KTB);
    const uint8_t *pa = firstA + group * stepA, *pb = firstB + group * stepB;  // of the K tile that is fetched next
    const int rem = KTAIL ? (int)(P.K - (int64_t)(nkt - 1) * KT) : KT;         // elements of the last K tile
    auto load_codes = [&](int u) {
        const bool isA = EVEN ? u < CA : piece(u) < BM / 16;
        asm volatile("global_load_lds_dwordx4 %0, %1" : : "v"(off[u]), "s"(isA ? pa : pb) : "memory");
    };
    // Before the loads of the group's step j: past its own last step every lane fetches the first bytes of A's codes instead (a valid address),
    // and in a K tail the chunks past K are the first ones.
    auto aim = [&](int j) {
        if (KTAIL && j * KG + group == nkt - 1 && ch * 32 >= rem) {
#pragma unroll
            for (int u = 0; u < CI; ++u) off[u] -= (uint32_t)ch * 16;
        }
        if (j >= own) {
            asm volatile("");
#pragma unroll
            for (int u = 0; u < CI; ++u) off[u] = 0;
            pa = pb = firstA;
        }
    };
    auto advance = [&]() {
        pa += KG * stepA;
        pb += KG * stepB;
    };

    // ---- scales: a thread's rows are tid + NT u of the tile's; 8 bytes into registers, then into the stage as fp16 pairs (byte << 7 =
    // fp16(scale * 2^-8), exact for every E4M3 byte), one pair for each chunk of 32 elements, repeated for blocks wider than 16
    const uint8_t *srow_ptr[NSR];
    int srow_step[NSR];
    uint64_t gs[NSR];
#pragma unroll
    for (int u = 0; u < NSR; ++u) {
        const int srow = tid + NT * u < ROWS ? tid + NT * u : ROWS - 1;
        const bool isA = srow < BM;
        int64_t gr = isA ? m0 + srow : n0 + (srow - BM);
        const int64_t nrows = isA ? P.M : P.N;
        gr = gr < nrows ? gr : nrows - 1;
        srow_ptr[u] = (isA ? P.A_scales : P.B_scales) + gr * Ks;
        srow_step[u] = SPT;
        if (!KTAIL && (isA ? P.a_slab : P.b_slab)) {
            const int64_t base = isA ? m0 : n0;
            const int lrow = SPAN && isA ? (int)(gr - base) : isA ? srow : srow - BM;
            const int sr = (int)(base & 255) + lrow;
            const int64_t slab = SPAN ? (base >> 8) + (sr >> 8) : base >> 8;
            srow_ptr[u] = (isA ? P.A_scales : P.B_scales) + slab * nkt * SLAB_SCALE_BYTES + slab_row(SPAN ? sr & 255 : sr) * 8;
            srow_step[u] = (int)SLAB_SCALE_BYTES;
        }
    }
    // first byte of the window that K tile kt lies in: the last one ends with the row, which has eight bytes or more (launch_gemm_wide())
    auto window = [&](int kt) { return kt / WINDOW * 8 + 8 < (int)Ks ? kt / WINDOW * 8 : (int)Ks - 8; };
    auto load_scales = [&](int j, int u) {
        const int kt = j * KG + group < nkt ? j * KG + group : nkt - 1;
        if constexpr (!WINDOWS) {
            gs[u] = *reinterpret_cast<const uint64_t *>(srow_ptr[u] + (int64_t)kt * srow_step[u]);
        } else if (WINDOW == 1 || KG > 1 || j == 0 || kt % WINDOW == 0) {  // (the groups' K tiles lie KG apart: a window each)
            __builtin_memcpy(&gs[u], srow_ptr[u] + window(kt), 8);
        }
    };
    // LDS: 1 KB for four fragments of a wave, [4 chunks][16 rows][4 fragments] dwords, so that a lane reads the scales of all four (of its chunk and
    // row) at once.  Chunks 2 p and 2 p + 1 of row tid + NT u, for step j.
    uint32_t srow_dst[NSR];
#pragma unroll
    for (int u = 0; u < NSR; ++u) {
        const int srow = tid + NT * u < ROWS ? tid + NT * u : ROWS - 1;
        const bool isA = srow < BM;
        const int frag = (isA ? srow : srow - BM) >> 4, per = isA ? TA : TB, blocks = (per + 3) / 4;
        const int w = frag / per, i = frag - w * per;
        srow_dst[u] = (uint32_t)((isA ? 0 : WM * ((TA + 3) / 4) * 1024) + (w * blocks + (i >> 2)) * 1024 + (srow & 15) * 16 + (i & 3) * 4);
    }
    auto stash = [&](int stage, int j, int u, int p) {
        const int kj = j * KG + group;
        // bits of the window in front of the K tile's scales; what follows the row is shifted in as zeros, and all of a K tile past the
        // last one is
        const int at = WINDOWS ? 8 * (kj * SPT - window(kj)) : (KG == 1 || kj < nkt) ? 0 : 64;
        uint64_t w = gs[u];
        if (WINDOWS || KG > 1) w = at < 64 ? w >> at : 0;
        uint32_t *const dst = reinterpret_cast<uint32_t *>(stages + stage * STAGE + ROWS * KTB + srow_dst[u]);
#pragma unroll
        for (int c = 2 * p; c < 2 * p + 2; ++c) {
            const int i0 = (32 * c) / B, i1 = (32 * c + 16) / B;  // (constants after unrolling)
            const uint32_t sel = 0x0C000C00u | (uint32_t)i0 | ((uint32_t)i1 << 16);
            dst[64 * c] = __builtin_amdgcn_perm((uint32_t)(w >> 32), (uint32_t)w, sel) << 7;
        }
    };

    // ---- LDS -> registers: fragment i of an operand is its rows 16 i + r, of which lane group g has chunk g: 32 codes (dword t for MFMA step
    // t of four) and the scales of their two blocks
    u32x4_t ca[TA], cb[TB];
    u32x4_t sa[(TA + 3) / 4], sb[TB / 4];  // of four fragments each
    const uint8_t *const fragA = stages + (wm * 16 * TA + r) * KTB + ((g ^ quad_xor(r >> 2)) << 4);
    const uint8_t *const fragB = stages + (BM + wn * 16 * TB + r) * KTB + ((g ^ quad_xor(r >> 2)) << 4);
    const uint8_t *const scalA = stages + ROWS * KTB + wm * ((TA + 3) / 4 * 1024) + lane * 16;
    const uint8_t *const scalB = stages + ROWS * KTB + (WM * ((TA + 3) / 4) + wn * (TB / 4)) * 1024 + lane * 16;
    auto read_a = [&](int stage, int i) {
        ca[i] = *reinterpret_cast<const u32x4_t *>(fragA + stage * STAGE + i * (16 * KTB));
    };
    auto read_b = [&](int stage, int i) {
        cb[i] = *reinterpret_cast<const u32x4_t *>(fragB + stage * STAGE + i * (16 * KTB));
    };
    auto read_sa = [&](int stage, int q) { sa[q] = *reinterpret_cast<const u32x4_t *>(scalA + stage * STAGE + q * 1024); };
    auto read_sb = [&](int stage, int q) { sb[q] = *reinterpret_cast<const u32x4_t *>(scalB + stage * STAGE + q * 1024); };
    // ---- expansion: 8 instructions per fragment and step, four converts and four multiplies by the scale
    u32x4_t fa[2], fb[2][TB];
    uint32_t ta[4], tb[4];
    auto convert = [](uint32_t w, int q) -> uint32_t {
        return __builtin_bit_cast(uint32_t, q == 0   ? __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 256.0f, 0)
                                            : q == 1 ? __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 256.0f, 1)
                                            : q == 2 ? __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 256.0f, 2)
                                                     : __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 256.0f, 3));
    };
    // (assembly here too: where the tile has a branch the compiler moves such instructions down behind it, right in front of their MFMA)
    auto scaled = [](uint32_t v, uint32_t s, int block) __attribute__((always_inline)) -> uint32_t {
        uint32_t y;
        if (block == 0) asm volatile("v_pk_mul_f16 %0, %1, %2 op_sel_hi:[1,0]" : "=v"(y) : "v"(v), "v"(s));
        else asm volatile("v_pk_mul_f16 %0, %1, %2 op_sel:[0,1]" : "=v"(y) : "v"(v), "v"(s));
        return y;
    };
    // instruction k of A's fragment i for step t into fa[to], of B's into fb[t & 1]
    auto expand_a = [&](int i, int t, int to, int k) {
        if (k < 4) ta[k] = convert(ca[i][t], k);
        else fa[to][k - 4] = scaled(ta[k - 4], sa[i >> 2][i & 3], t >> 1);
    };
    auto expand_b = [&](int i, int t, int k) {
        if (k < 4) tb[k] = convert(cb[i][t], k);
        else fb[t & 1][i][k - 4] = scaled(tb[k - 4], sb[i >> 2][i & 3], t >> 1);
    };

    // ---- start: K tile 0 of the group into stage 0, 1 into stage 1
    aim(0);
#pragma unroll
    for (int u = 0; u < NSR; ++u) load_scales(0, u);
#pragma unroll
    for (int u = 0; u < CI; ++u)
        {
            load_dst(std::integral_constant<int, 0>{}, u);
            asm volatile("s_nop 4");
            load_codes(u);
        }
    advance();
#pragma unroll
    for (int u = 0; u < NSR; ++u)
#pragma unroll
        for (int p = 0; p < 2; ++p) stash(0, 0, u, p);
    aim(1);
#pragma unroll
    for (int u = 0; u < NSR; ++u) load_scales(1, u);
#pragma unroll
    for (int u = 0; u < CI; ++u)
        {
            load_dst(std::integral_constant<int, 1>{}, u);
            asm volatile("s_nop 4");
            load_codes(u);
        }
    advance();
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(CI) : "memory");  // K tile 0 has landed
    __syncthreads();
#pragma unroll
    for (int q = 0; q < TB / 4; ++q) read_sb(0, q);
#pragma unroll
    for (int i = 0; i < TB; ++i) read_b(0, i);
#pragma unroll
    for (int q = 0; q < (TA + 3) / 4; ++q) read_sa(0, q);
#pragma unroll
    for (int i = 0; i < TA; ++i) read_a(0, i);
#pragma unroll
    for (int i = 0; i < TB; ++i)
#pragma unroll
        for (int k = 0; k < 8; ++k) expand_b(i, 0, k);
#pragma unroll
    for (int k = 0; k < 8; ++k) expand_a(0, 0, 0, k);

    // The group's step j, its K tile in registers (stage ST is free at the barrier): four MFMA steps of TA rows of 8 MFMAs.  Under a row's MFMAs the
    // next row's fragment of A is expanded and a share of B's fragments for the next step.  In step 1 the scales of step j + 1 go into the
    // other stage, where its codes are by then, ONE barrier; in step 2 a fragment of B is read again as soon as its last dword has been
    // expanded, in step 3 those of A; in step 2 the loads of step j + 2 are requested.  Scheduling fences pin the order.
    int j = 0;
    auto tile = [&](auto stc) __attribute__((always_inline)) {
        constexpr int NEXT = decltype(stc)::value ^ 1, N = 8 * TA;
        aim(j + 2);
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_nop 1");  // (behind the last expansion before the loop)
        __builtin_amdgcn_sched_barrier(0);
        static_for<4 * N>([&](auto xc) __attribute__((always_inline)) {
            constexpr int t = decltype(xc)::value / N, x = decltype(xc)::value % N, a = x >> 3, b = x & 7;
            // (there and back: from one MFMA to the next one operand of two changes; 8192 x 8192 x 8192 657 -> 651 us, 4096 x 4096 x 11008 220 -> 219)
            constexpr int col = a & 1 ? 7 - b : b;
            mfma_16x16x32(acc[a / IN][a % IN * TB + col], fb[t & 1][col], fa[(t * TA + a) & 1]);
            __builtin_amdgcn_sched_barrier(0);
            // the row's vector instructions: 8 for A's next fragment, then its share of B's 64
            constexpr int lo = 64 * a / TA, hi = 64 * (a + 1) / TA, len = 8 + hi - lo;
            constexpr int an = a + 1 < TA ? a + 1 : 0, tn = a + 1 < TA ? t : (t + 1) & 3;
#pragma unroll
            for (int k = len * b / 8; k < len * (b + 1) / 8; ++k) {
                if (k < 8) expand_a(an, tn, (t * TA + a + 1) & 1, k);
                else expand_b((lo + k - 8) >> 3, (t + 1) & 3, (lo + k - 8) & 7);
            }
            // scales of the next K tile: behind the wait for this wave's loads
            constexpr int FIRST = N - 8 - 2 * NSR;
            if constexpr (t == 1 && x == FIRST) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if constexpr (t == 1 && x >= FIRST && x < FIRST + 2 * NSR) stash(NEXT, j + 1, (x - FIRST) >> 1, (x - FIRST) & 1);
            // reads: fragment i of B behind the row that expands its last dword, the second such fragment of a row after the first; the scales
            // of four behind the last of them
#pragma unroll
            for (int i = 0; i < TB; ++i) {
                const int done = (8 * i + 7) * TA / 64;  // the row of instruction 8 i + 7
                const int slot = i == 0 || (8 * i - 1) * TA / 64 != done ? 0 : 2;
                const bool here = (t == 2 && a == done + 1) || (t == 3 && a == 0 && done == TA - 1);
                if (b == slot && here) read_b(NEXT, i);
                if (b == 4 && here && i % 4 == 3) read_sb(NEXT, i / 4);
            }
            // A's row a has been expanded under row a - 1
            if constexpr (t == 3 && b == 6) read_a(NEXT, a);
            if constexpr (t == 3 && b == 5 && (a % 4 == 3 || a == TA - 1)) read_sa(NEXT, a / 4);
            if constexpr (t == 2 && b == 7 && a < NSR) load_scales(j + 2, a);
            constexpr int GAP = (N - 4) / CI, y = (t - 2) * N + x - 1;
            if constexpr (t >= 2 && y >= 0 && y / GAP < CI) {
                if constexpr (y % GAP == 0) load_dst(stc, y / GAP);
                if constexpr (y % GAP == 2) load_codes(y / GAP);
            }
            if constexpr (t == 3 && x == N - 1) advance();
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (t == 1 && x == N - 1) {
                __syncthreads();
                __builtin_amdgcn_sched_barrier(0);
            }
        });
        ++j;
    };
    while (j + 2 <= steps) {
        tile(std::integral_constant<int, 0>{});
        tile(std::integral_constant<int, 1>{});
    }
    if (j < steps) tile(std::integral_constant<int, 0>{});

    // epilogue.  The MFMA's first operand is the B (N-side) fragment, so a lane holds four consecutive columns of one row.
    asm volatile("s_waitcnt vmcnt(0)\n\ts_nop 15" ::: "memory");
    __syncthreads();  // no load under way, every wave has read its last fragments: the stages may be overwritten
#pragma unroll
    for (int a = 0; a < S; ++a)
#pragma unroll
        for (int b = 0; b < IN * TB; ++b) asm volatile("" : "+a"(acc[a][b]));
    const int64_t row0 = m0 + wm * 16 * TA, col0 = n0 + wn * 16 * TB;
    uint8_t *const mine = lds + wave_wg * (G::PIECES / 4 / (OUT_DT == NVFP4_F32 ? 1 : 2));
    if constexpr (KG == 1) {
        store_lines<OUT_DT, TB>(P, acc, row0, col0, mine, lane);
    } else {
        // each group keeps one half of the strips
        static_assert(KG == 2 && S % 2 == 0, "halves");
        float4v_t half[S / 2][IN * TB];
        fold_groups<S, IN * TB, NW>(acc, half, lds, group, wave, lane);
        store_lines<OUT_DT, TB>(P, half, row0 + group * (8 * TA), col0, mine, lane);
    }
}

template <int B, int WM, int WN, int KG, int TA, int OUT_DT, bool KTAIL>
__global__ __launch_bounds__(256) void gemm_nt_f16_wide_kernel(TileArgs P)
{
    using G = wide::Geom<WM, WN, KG, TA>;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    int ty, tx;
    tile_coords(blockIdx.x, (int)((P.N + G::BN - 1) / G::BN), (int)((P.M + G::BM - 1) / G::BM), ty, tx);
    wide_tile<B, WM, WN, KG, TA, OUT_DT, KTAIL>(P, lds, (int64_t)ty * G::BM, (int64_t)tx * G::BN);
}

// Whole rounds of 256 x 256 tiles and, in the place of a partly filled last round of them, one of smaller tiles (192 x 256, or 128 x 256 in two groups):
// X.first workgroups take the first X.split tile rows or columns of the output, those that follow the rest.
template <int B, int WM, int WN, int KG, int TA, int OUT_DT>
__global__ __launch_bounds__(256) void gemm_nt_f16_wide_mixed_kernel(TileArgs P, WideMix X)
{
    using G = wide::Geom<WM, WN, KG, TA>;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    static_assert(G::BN == 256, "columns of the second part's tiles");
    int64_t m0, n0;
    if (blockIdx.x < X.first) {
        mixed_first(X, blockIdx.x, P.M, P.N, m0, n0);
        wide_tile<B, 2, 2, 1, 8, OUT_DT, false>(P, lds, m0, n0);
    } else {
        mixed_second(X, blockIdx.x, P.M, P.N, G::BM, m0, n0);
        wide_tile<B, WM, WN, KG, TA, OUT_DT, false>(P, lds, m0, n0);
    }
}

template <int B, int WM, int WN, int KG, int TA, bool KTAIL>
static void launch_wide(const TileArgs &P, int out_dt, hipStream_t st)
{
    using G = wide::Geom<WM, WN, KG, TA>;
    const unsigned ntiles = (unsigned)(((P.N + G::BN - 1) / G::BN) * ((P.M + G::BM - 1) / G::BM));
    if (out_dt == NVFP4_F32) {
        auto k = gemm_nt_f16_wide_kernel<B, WM, WN, KG, TA, NVFP4_F32, KTAIL>;
        static bool once = ((void)hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, G::LDS), true);
        (void)once;
        hipLaunchKernelGGL(k, dim3(ntiles), dim3(256), G::LDS, st, P);
    } else {
        auto k = gemm_nt_f16_wide_kernel<B, WM, WN, KG, TA, NVFP4_BF16, KTAIL>;
        static bool once = ((void)hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, G::LDS), true);
        (void)once;
        hipLaunchKernelGGL(k, dim3(ntiles), dim3(256), G::LDS, st, P);
    }
}

template <int B, int WM, int WN, int KG, int TA, int OUT_DT>
static void launch_wide_mixed_as(const TileArgs &P, const WideMix &X, hipStream_t st)
{
    using G = wide::Geom<WM, WN, KG, TA>;
    using G256 = wide::Geom<2, 2, 1, 8>;
    constexpr int LDS = G::LDS > G256::LDS ? G::LDS : G256::LDS;
    auto k = gemm_nt_f16_wide_mixed_kernel<B, WM, WN, KG, TA, OUT_DT>;
    static bool once = ((void)hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, LDS), true);
    (void)once;
    hipLaunchKernelGGL(k, dim3(X.first + X.second), dim3(256), LDS, st, P, X);
}

template <int B>
static void launch_wide_mixed(const TileArgs &P, const WideMix &X, int out_dt, hipStream_t st)
{
    if (X.tile == TILE_192x256) {
        if (out_dt == NVFP4_F32) launch_wide_mixed_as<B, 2, 2, 1, 6, NVFP4_F32>(P, X, st);
        else launch_wide_mixed_as<B, 2, 2, 1, 6, NVFP4_BF16>(P, X, st);
    } else {
        if (out_dt == NVFP4_F32) launch_wide_mixed_as<B, 1, 2, 2, 8, NVFP4_F32>(P, X, st);
        else launch_wide_mixed_as<B, 1, 2, 2, 8, NVFP4_BF16>(P, X, st);
    }
}

// False for a tile that is not one of these
template <int B, bool KTAIL>
static bool launch_wide_tile(const TileArgs &P, GemmTile tile, int out_dt, hipStream_t st)
{
    switch (tile) {
    case TILE_256x256: launch_wide<B, 2, 2, 1, 8, KTAIL>(P, out_dt, st); return true;
    case TILE_192x256: launch_wide<B, 2, 2, 1, 6, KTAIL>(P, out_dt, st); return true;
    case TILE_160x256: launch_wide<B, 2, 2, 1, 5, KTAIL>(P, out_dt, st); return true;
    case TILE_128x256_K2: launch_wide<B, 1, 2, 2, 8, KTAIL>(P, out_dt, st); return true;
    default: return false;
    }
}

}  // namespace nvfp4
