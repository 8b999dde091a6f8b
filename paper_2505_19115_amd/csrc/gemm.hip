// Block-scaled FP4 GEMM for gfx950 ("NT": both operands stored with the contraction axis
// contiguous), the matrix product shared by Eqs. 4-6 of "FP4 All the Way":
//     out[i, j] = gA gB sum_k cA[i,k] sA[i,k/B] cB[j,k] sB[j,k/B].
//
// E4M3 block scales (NVFP4 and its wider-block variants).  The CDNA4 scaled FP4 MFMA applies
// one power-of-two (E8M0) scale per 32 contraction elements, so it cannot apply a 16-wide
// E4M3 scale, and an E2M1 x E4M3 product needs up to 6 significant bits, more than FP8 or FP6
// hold.  The product is exact in fp16 (11 bits; magnitudes 2^-10 .. 2688), so operands travel
// through HBM and LDS as packed 4-bit codes plus scale bytes and are expanded in registers:
//     v_cvt_scalef32_pk_f16_fp4 (code pair -> fp16 pair, times 2^8)  and
//     v_pk_mul_f16 by the block scale written as fp16(scale * 2^-8),
// which is exact for every E4M3 byte, including its subnormals; the MFMA operands themselves
// are always normal fp16 numbers or zero.  The contraction runs on v_mfma_f32_32x32x16_f16 (contractions of more than seven K tiles
// on large tiles: v_mfma_f32_16x16x32_f16, gemm_wide.h) with fp32 accumulation; the tensor scales multiply once in the epilogue.
//
// Operand storage: row-major ([rows, K/2] codes, [rows, K/B] scale bytes), or, for blocks of 16, the slab layout of
// kernels.h, in which the 256 rows x 64 code bytes (and 256 x 8 scale bytes) of a K tile are one contiguous piece.  Only
// addresses differ: per-lane offsets, two base pointers and their step per K tile.
#include "gemm_fold.h"
#include "kernels.h"
#include "nvfp4_math.h"
#include "store_lines.h"

namespace nvfp4 {

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float16_t __attribute__((ext_vector_type(16)));

constexpr int KT = 128;      // contraction elements per LDS tile
constexpr int KTB = KT / 2;  // bytes of codes per row per tile
constexpr int SROW = 16;     // LDS bytes per row for the tile's scales: 8 fp16 values, one per 16 elements

// LDS placement of the codes of one tile row r (64 bytes = 4 chunks of 16): chunk c sits in
// chunk slot c ^ ((r >> 2) & 3).  Rows are 64 bytes apart, so 16 consecutive rows reading the same
// logical chunk (one ds_read_b128 wavefront pass) cover all sixteen 16-byte slots of the 256-byte
// bank period, and a 16-byte store of a whole chunk by 4 consecutive threads per row covers
// contiguous bytes: no conflicts either way.
__device__ __forceinline__ int swz(int r, int c) { return r * KTB + ((c ^ ((r >> 2) & 3)) << 4); }

// 8 codes (one dword) of one block -> 8 fp16 values times the block scale.
// s = fp16 holding scale * 2^-8; the convert multiplies the codes by 2^8.
// FOURS: four converts, then four multiplies, of which none waits for the one before (us, without / with: 1056 x 2080 x 2784 19.5 / 19.0, 2048 x 4096 x 1024
// 18.1 / 17.6, 8192 x 8192 x 256 46.5 / 45.7, 1024 x 1024 x 2048 in blocks of 64 9.3 / 8.9); three more registers, which tiles of 128 x 64 per wave do not have.
template <bool FOURS>
__device__ __forceinline__ half8_t dequant8(uint32_t w, _Float16 s)
{
    const half2_t s2 = {s, s};
    half2_t h0 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 256.0f, 0), h1 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 256.0f, 1);
    half2_t h2 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 256.0f, 2), h3 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 256.0f, 3);
    if (FOURS) asm("" : "+v"(h0), "+v"(h1), "+v"(h2), "+v"(h3));
    h0 *= s2; h1 *= s2; h2 *= s2; h3 *= s2;
    half8_t r;
    r[0] = h0[0]; r[1] = h0[1]; r[2] = h1[0]; r[3] = h1[1];
    r[4] = h2[0]; r[5] = h2[1]; r[6] = h3[0]; r[7] = h3[1];
    return r;
}

// Tile geometry.  A workgroup is KG groups of WM x WN waves; a wave owns (32 TA) x (32 TB) outputs as
// TA x TB MFMA tiles.  The largest shape is 2 x 4 waves of 4 x 2 tiles: 256 x 256 per
// workgroup, 128 accumulator registers per wave, so TWO waves fit on every SIMD.  That is
// the point of the shape: measured on gfx950, one wave alone issues a VALU instruction only
// every ~8 cycles, two waves per SIMD reach the full rate of one per 4 cycles, and the
// operand expansion costs 8 (TA + TB) / (TA TB) = 6 VALU instructions per 32-cycle MFMA.
// KG = 4 serves products with fewer 128 x 128 tiles than CUs, where one workgroup of four waves leaves each SIMD a single wave:
// four groups of 1 x 2 waves multiply every fourth K tile each, with their own stages and the large tile's wave shape, and add
// their sums through the LDS at the end.  1056 x 2080 x 2784: 128 x 128 26.2 us, 96 x 128 with four groups 21.7; 1536 x 1536 x 6144:
// 64 x 64 45.0, 96 x 128 with four groups 34.3.  (256 x 11008 x 4096 stays on 64 x 64: 30.7, the estimates lie 4 % apart, 128 x 128 with
// four groups 28.8.  Two groups of 1 x 4 waves on 128 x 256 were no faster than eight waves of 64 x 64: 4096 x 4096 x 11008 315 and 312 us;
// a chip filled either way is bound by its power, not by the expansion.)
// With blocks of 32 to 128 the 128 x 128 form takes 0.65 to 0.9 of the time of the tile it replaces
// (2164 x 1618 x 11520, blocks of 64, 129.9 -> 94.5 us; blocks of 16 100.7 -> 86.0).
//
// Per 128-wide K tile the 64 code bytes of each operand row sit in LDS as four 16-byte chunks
// and its 8 block scales as fp16 values (scale * 2^-8; for blocks wider than 16 the value is
// repeated).  Lane (r = lane % 32, h = lane / 32) owns chunk 2p + h (p = 0, 1) of its row:
// 32 codes = two 16-element blocks; dword t (0..3) of the chunk feeds one MFMA step and
// belongs to block t / 2.  A and B use the same assignment of contraction indices to (lane
// half, step), which is all the instruction requires.
// (wrow: the wave's first row in the tile)
template <int B, int WM, int WN, int TA, int TB, int KG, int OUT_DT, bool KTAIL, int BM>
__device__ __forceinline__ void f16_tile(const TileArgs &P, const int wrow)
{
    constexpr int NT = 64 * WM * WN;  // threads of a group
    constexpr int BN = 32 * TB * WN;
    constexpr int SPT = KT / B;  // scale bytes per row per tile in global memory
    // A row-major row's scale bytes come 8 at a time: those of WINDOW K tiles.  A request per row costs the vector L1 the same for 1 byte
    // as for 8, and of a K tail the bytes past the row are shifted out below instead of left out one by one, which was a chain of 8
    // loads at the end of the walk.  us, a request per row and K tile / a window: 4096 x 4096 x 11008 blocks of 64 284 / 271, of 32
    // 278 / 267; with a K tail (f32 outputs) 1056 x 2080 x 2784 blocks of 16 25.4 / 21.6, of 32 24.7 / 21.1, 1056 x 2784 x 2080 22.7 / 21.2.
    // (16 bytes, two K tiles, at a time for blocks of 16: a few more registers and branches, 1056 x 2080 x 2816 23.1 instead of 21.4.)
    constexpr int WINDOW = 8 / SPT;
    constexpr bool WINDOWS = KTAIL || WINDOW > 1;  // (without a K tail a window of blocks of 16 is a K tile's 8 bytes, here or in a slab)
    constexpr int VALU_PER_MFMA = (8 * (TA + TB) + TA * TB - 1) / (TA * TB);
    constexpr int A_BYTES = BM * KTB, B_BYTES = BN * KTB, SA_BYTES = BM * SROW, SB_BYTES = BN * SROW;
    constexpr int STAGE = A_BYTES + B_BYTES + SA_BYTES + SB_BYTES;
    // Code loads of a tile, 16 rows each: A's pieces, then B's; CI per wave.  Where they divide evenly a wave takes
    // consecutive pieces of A and of B, else the list is dealt out in turn.
    constexpr int NW = WM * WN, NI = (BM + BN) / 16, CI = (NI + NW - 1) / NW, CA = BM / 16 / NW, CB = BN / 16 / NW;
    constexpr bool EVEN = BM / 16 % NW == 0 && BN / 16 % NW == 0;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];

    const int lane = threadIdx.x & 63;
    const int wave_wg = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int group = KG == 1 ? 0 : wave_wg / NW, wave = wave_wg - group * NW, tid = wave * 64 + lane;  // (inside the group from here on)
    const int wn = wave % WN;
    const int r = lane & 31, h = lane >> 5;
    const int ntx = (int)((P.N + BN - 1) / BN), nty = (int)((P.M + BM - 1) / BM);
    int ty, tx;
    tile_coords(blockIdx.x, ntx, nty, ty, tx);
    const int64_t m0 = (int64_t)ty * BM, n0 = (int64_t)tx * BN;
    const int64_t Kb = P.K >> 1;          // code bytes per row
    const int64_t Ks = P.K / B;           // scale bytes per row
    const int nkt = (int)((P.K + KT - 1) / KT);

    float16_t acc[TA][TB];
#pragma unroll
    for (int a = 0; a < TA; ++a)
#pragma unroll
        for (int b = 0; b < TB; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.0f;

    // ---- global -> LDS staging of one K tile.
    // Rows past the matrix edge are clamped to the last row (their products land in outputs
    // that are never stored), so the code loads carry no predicate.  A K tail (K not a
    // multiple of 128) is handled through the scales alone: a chunk past K is replaced by the
    // tile's first one and meets the zeros that follow the row's last scale byte.
    // The codes go from global memory straight into LDS (global_load_lds, 16
    // bytes per lane): a wave instruction fills 1 KB = 16 consecutive tile rows, lane i landing at
    // byte 16 i (row i / 4, slot i % 4), so the swizzle is applied by choosing WHICH global chunk
    // the lane fetches.  No staging registers, no LDS store instructions for the codes.  (A K tail
    // used to be staged through registers by a 128 x 128 kernel of its own: 4096 x 4128 x 4896 took
    // 539 us, with the direct loads 190.)
    constexpr int NSR = (BM + BN + NT - 1) / NT;  // scale rows per thread
    uint64_t gs[NSR];
    constexpr bool SPAN = 256 % BM != 0;  // A's rows may lie in two slabs
    auto piece = [&](int u) { return !EVEN ? u * NW + wave : u < CA ? wave * CA + u : BM / 16 + wave * CB + u - CA; };
    uint32_t off[CI];  // byte offset of this thread's chunks inside a K tile column
    const int ch = (lane & 3) ^ ((lane >> 4) & 3);
#pragma unroll
    for (int u = 0; u < CI; ++u) {
        const int trow = piece(u) * 16 + (lane >> 2);  // row of the tile: A's, then B's
        const bool isA = EVEN ? u < CA : trow < BM;
        const int row = isA ? trow : trow - BM;
        const int64_t base = isA ? m0 : n0, rows = isA ? P.M : P.N;
        const int64_t lr = base + row < rows ? row : rows - 1 - base;  // row inside the tile, clamped
        // a slab holds all rows of a 256- or 128-row tile: nothing to clamp; one of 96, 160 or 192 rows may reach into the next slab
        const int srow = (int)(base & 255) + (int)(SPAN && isA ? lr : row);
        const uint32_t slab_off = (uint32_t)(slab_row(SPAN && isA ? srow & 255 : srow) * 64 + ch * 16) +
                                  (SPAN && isA && srow > 255 ? (uint32_t)nkt * (uint32_t)SLAB_CODE_BYTES : 0u);
        off[u] = (isA ? P.a_slab : P.b_slab) ? slab_off : (uint32_t)(lr * Kb + ch * 16);  // (relative to the tile's first row: 32 bits suffice)
    }
    typedef __attribute__((address_space(3))) void *lds_ptr_t;
    uint8_t *const stages = lds + group * (2 * STAGE);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr_t)stages;
    // wave-uniform 64-bit value -> scalar registers
    auto uniform_ptr = [](const uint8_t *p) -> const uint8_t * {
        const uint64_t v = reinterpret_cast<uint64_t>(p);
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
        return reinterpret_cast<const uint8_t *>(((uint64_t)hi << 32) | lo);
    };
    // Issued through inline assembly on purpose: the compiler's wait-count pass treats a
    // direct-to-LDS load as a possible writer of every LDS location and would wait for it before
    // the next LDS read.  Here the destination stage is not read before the explicit wait and the
    // barrier in stash().
    auto dma16 = [&](uint32_t lds_addr, uint32_t voff, const uint8_t *base) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds_addr), "v"(voff), "s"(base) : "memory", "m0");
    };
    const uint8_t *srow_ptr[NSR];
    int srow_step[NSR];  // bytes from one K tile's scales of the row to the next
    bool srow_on[NSR];
#pragma unroll
    for (int u = 0; u < NSR; ++u) {
        const int srow = tid + NT * u;
        const bool isA = srow < BM;
        int64_t gr = isA ? m0 + srow : n0 + (srow - BM);
        const int64_t nrows = isA ? P.M : P.N;
        gr = gr < nrows ? gr : nrows - 1;
        srow_on[u] = srow < BM + BN;
        srow_ptr[u] = (isA ? P.A_scales : P.B_scales) + gr * Ks;
        srow_step[u] = SPT;
        if (!KTAIL && (isA ? P.a_slab : P.b_slab) && srow_on[u]) {
            const int64_t base = isA ? m0 : n0;
            const int lrow = SPAN && isA ? (int)(gr - base) : isA ? srow : srow - BM;
            const int sr = (int)(base & 255) + lrow;
            const int64_t slab = SPAN ? (base >> 8) + (sr >> 8) : base >> 8;
            srow_ptr[u] = (isA ? P.A_scales : P.B_scales) + slab * nkt * SLAB_SCALE_BYTES + slab_row(SPAN ? sr & 255 : sr) * 8;
            srow_step[u] = (int)SLAB_SCALE_BYTES;
        }
    }
    // codes of K tile kt: base + kt * step (+ the lane offsets above)
    const uint8_t *baseA = P.a_slab ? P.A_codes + (m0 >> 8) * nkt * SLAB_CODE_BYTES : P.A_codes + m0 * Kb;
    const uint8_t *baseB = P.b_slab ? P.B_codes + (n0 >> 8) * nkt * SLAB_CODE_BYTES : P.B_codes + n0 * Kb;
    const int64_t stepA = P.a_slab ? SLAB_CODE_BYTES : KTB, stepB = P.b_slab ? SLAB_CODE_BYTES : KTB;
    const int rem = KTAIL ? (int)(P.K - (int64_t)(nkt - 1) * KT) : KT;  // elements of the last K tile
    // the group's step j (K tile j KG + group): codes -> LDS stage `stage` (direct); scale bytes -> registers.  A K tile past the
    // last one is the last one again with zero scales: every group takes the same steps and meets the same barriers.
    const int steps = (nkt + KG - 1) / KG;
    // first byte of the window that K tile kt lies in: the last one ends with the row, also if that is shorter
    auto window = [&](int kt) { return kt / WINDOW * 8 + 8 < (int)Ks ? kt / WINDOW * 8 : (int)Ks - 8; };
    auto fetch = [&](int j, int stage) {
        const int kj = j * KG + group;
        const bool absent = KG > 1 && kj >= nkt;
        const int kt = absent ? nkt - 1 : kj;
        const uint8_t *ua = uniform_ptr(baseA + kt * stepA), *ub = uniform_ptr(baseB + kt * stepB);
        const uint32_t dst = __builtin_amdgcn_readfirstlane(lds0 + stage * STAGE);
        const bool tail = KTAIL && kt == nkt - 1;
        const uint32_t back = tail && ch * 32 >= rem ? (uint32_t)ch * 16 : 0u;  // (a chunk past K: the tile's first one)
#pragma unroll
        for (int u = 0; u < CI; ++u) {
            const int i = piece(u);
            if (EVEN || i < NI) dma16(dst + i * 1024, KTAIL ? off[u] - back : off[u], (EVEN ? u < CA : i < BM / 16) ? ua : ub);
        }
#pragma unroll
        for (int u = 0; u < NSR; ++u) {
            if (!srow_on[u]) continue;
            if constexpr (!WINDOWS) {
                gs[u] = *reinterpret_cast<const uint64_t *>(srow_ptr[u] + (int64_t)kt * srow_step[u]);
            } else if (Ks >= 8) {
                // (the groups' K tiles lie KG apart: a window each)
                if (WINDOW == 1 || KG > 1 || j == 0 || kt % WINDOW == 0) __builtin_memcpy(&gs[u], srow_ptr[u] + window(kt), 8);
            } else if (j == 0) {
                gs[u] = 0;
                for (int t = 0; t < (int)Ks; ++t) gs[u] = gs[u] >> 8 | (uint64_t)srow_ptr[u][t] << 56;
            }
        }
    };
    // LDS scale layout: [4 chunks of 32 elements][BM + BN rows] dwords, each dword = the fp16
    // scales (byte << 7 = fp16(scale * 2^-8), exact for normal and subnormal E4M3 bytes alike
    // because fp16's bias is E4M3's plus 8) of the chunk's two 16-element blocks; a wave reads
    // 32 consecutive rows of one chunk.  For blocks wider than 16 the value is repeated.
    auto stash = [&](int stage, int j) {
        uint8_t *base = stages + stage * STAGE;
        const int kj = j * KG + group;
        // bits of the window in front of the K tile's scales; what follows the row is shifted in as zeros, and all of a K tile past the
        // last one is
        const int at = WINDOWS ? 8 * (kj * SPT - window(kj)) : (KG == 1 || kj < nkt) ? 0 : 64;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's direct-to-LDS loads have landed
        uint32_t *sS = reinterpret_cast<uint32_t *>(base + A_BYTES + B_BYTES);
#pragma unroll
        for (int u = 0; u < NSR; ++u) {
            if (!srow_on[u]) continue;
            // (a window of one K tile is not used again: shifted where it is, and only if it has to be)
            if (WINDOW == 1 && at) gs[u] = at < 64 ? gs[u] >> at : 0;
            const uint64_t w = WINDOW == 1 ? gs[u] : at < 64 ? gs[u] >> at : 0;
            const uint32_t lo = (uint32_t)w, hi = (uint32_t)(w >> 32);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                // bytes i0, i1 of the staged scale bytes -> (b0 << 7) | (b1 << 23): one byte permute
                // (b0 into byte 0, b1 into byte 2, zeros between) and one shift
                const int i0 = (32 * c) / B, i1 = (32 * c + 16) / B;  // (constants after unrolling)
                const uint32_t sel = 0x0C000C00u | (uint32_t)i0 | ((uint32_t)i1 << 16);
                sS[c * (BM + BN) + tid + NT * u] = __builtin_amdgcn_perm(hi, lo, sel) << 7;
            }
        }
    };

    // ---- LDS -> registers.  A lane reads chunk 2 p + h (16 bytes = 32 codes = two blocks of 16,
    // four MFMA steps) of rows (frag base + r): its byte offset inside a row is one of two lane
    // constants, the rest are immediates.
    struct Codes {
        uint4 ca[TA], cb[TB];
    };
    struct Scales {  // two fp16 scales (first and second block of the lane's 32-element chunk)
        uint32_t sa[TA], sb[TB];
    };
    int coff[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) coff[p] = swz(r, 2 * p + h);
    const int soff = (h * (BM + BN) + r) * 4;
    auto load_codes = [&](int stage, int p, Codes &Q) {
        const uint8_t *sA = stages + stage * STAGE + coff[p], *sB = sA + A_BYTES;
#pragma unroll
        for (int a = 0; a < TA; ++a)
            Q.ca[a] = *reinterpret_cast<const uint4 *>(sA + (wrow + 32 * a) * KTB);
#pragma unroll
        for (int b = 0; b < TB; ++b)
            Q.cb[b] = *reinterpret_cast<const uint4 *>(sB + (wn * 32 * TB + 32 * b) * KTB);
    };
    auto load_scales = [&](int stage, int p, Scales &S) {
        const uint8_t *sS = stages + stage * STAGE + A_BYTES + B_BYTES + soff + 2 * p * (BM + BN) * 4;
#pragma unroll
        for (int a = 0; a < TA; ++a) S.sa[a] = *reinterpret_cast<const uint32_t *>(sS + (wrow + 32 * a) * 4);
#pragma unroll
        for (int b = 0; b < TB; ++b) S.sb[b] = *reinterpret_cast<const uint32_t *>(sS + (BM + wn * 32 * TB + 32 * b) * 4);
    };
    struct Frags {
        half8_t a[TA], b[TB];
    };
    // operands of MFMA step t (0..3) of a chunk: its dword t, scaled by the scale of the block
    // (t / 2) that dword belongs to
    auto expand = [&](const Codes &Q, const Scales &S, int t, Frags &F) {
        auto dword = [&](const uint4 &v) { return t == 0 ? v.x : t == 1 ? v.y : t == 2 ? v.z : v.w; };
#pragma unroll
        for (int a = 0; a < TA; ++a) {
            const half2_t sp = __builtin_bit_cast(half2_t, S.sa[a]);
            F.a[a] = dequant8<(TA < 4)>(dword(Q.ca[a]), t >= 2 ? sp[1] : sp[0]);
        }
#pragma unroll
        for (int b = 0; b < TB; ++b) {
            const half2_t sp = __builtin_bit_cast(half2_t, S.sb[b]);
            F.b[b] = dequant8<(TA < 4)>(dword(Q.cb[b]), t >= 2 ? sp[1] : sp[0]);
        }
    };
    auto mma = [&](const Frags &F) {
#pragma unroll
        for (int a = 0; a < TA; ++a)
#pragma unroll
            for (int b = 0; b < TB; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(F.b[b], F.a[a], acc[a][b], 0, 0, 0);
    };

    // Software pipeline, continuous across K tiles (8 MFMA steps of TA*TB MFMAs per tile; the
    // operands of step s+1 are expanded under the MFMAs of step s).  On entry to iteration kt
    // the LDS stage kt & 1 holds tile kt; Ca holds the lanes' chunk of its first half, S0 the
    // scales of that half, F0 the operands of its first step.  Within the iteration:
    //   top      global loads of tile kt+1 -> registers; LDS loads of the second half (Cb, S1)
    //   step 6   tile kt+1 -> other LDS stage, ONE barrier, LDS loads of its first half
    //   step 7   already expands the first operands of tile kt+1.
    // After the barrier nobody reads stage kt & 1 again (both halves are in registers), so the
    // next iteration may overwrite it.
    // The scheduling hints pin "one MFMA, then its share of the expansion work" so that VALU
    // work is always queued behind an MFMA that holds the matrix pipe for 32 cycles.
#define NVFP4_INTERLEAVE()                                                  \
    _Pragma("unroll") for (int i = 0; i < TA * TB; ++i) {                   \
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                  \
        __builtin_amdgcn_sched_group_barrier(0x002, VALU_PER_MFMA, 0);      \
    }                                                                       \
    __builtin_amdgcn_sched_barrier(0);
#define NVFP4_STEP(Qn, Sn, tn, Fn, Fc) \
    expand(Qn, Sn, tn, Fn);            \
    mma(Fc);                           \
    NVFP4_INTERLEAVE()

    Codes Ca, Cb;
    Scales S0, S1;
    Frags F0, F1;
    fetch(0, 0);
    stash(0, 0);
    __syncthreads();
    load_codes(0, 0, Ca);
    load_scales(0, 0, S0);
    expand(Ca, S0, 0, F0);
#define NVFP4_TILE(stage, kt)                     \
    {                                             \
        fetch((kt) + 1, (stage) ^ 1);             \
        load_codes(stage, 1, Cb);                 \
        load_scales(stage, 1, S1);                \
        __builtin_amdgcn_sched_barrier(0);        \
        NVFP4_STEP(Ca, S0, 1, F1, F0)             \
        NVFP4_STEP(Ca, S0, 2, F0, F1)             \
        NVFP4_STEP(Ca, S0, 3, F1, F0)             \
        NVFP4_STEP(Cb, S1, 0, F0, F1)             \
        NVFP4_STEP(Cb, S1, 1, F1, F0)             \
        NVFP4_STEP(Cb, S1, 2, F0, F1)             \
        stash((stage) ^ 1, (kt) + 1);             \
        __syncthreads();                          \
        load_codes((stage) ^ 1, 0, Ca);           \
        load_scales((stage) ^ 1, 0, S0);          \
        __builtin_amdgcn_sched_barrier(0);        \
        NVFP4_STEP(Cb, S1, 3, F1, F0)             \
        NVFP4_STEP(Ca, S0, 0, F0, F1)             \
    }
    // two tiles per trip so that the LDS stage (and with it every LDS offset) is a constant
    int kt = 0;
    for (; kt + 2 < steps; kt += 2) {
        NVFP4_TILE(0, kt)
        NVFP4_TILE(1, kt + 1)
    }
    if (kt + 1 < steps) {
        NVFP4_TILE(0, kt)
        ++kt;
    }
#undef NVFP4_TILE
    {
        const int stage = kt & 1;  // the last tile
        load_codes(stage, 1, Cb);
        load_scales(stage, 1, S1);
        __builtin_amdgcn_sched_barrier(0);
        NVFP4_STEP(Ca, S0, 1, F1, F0)
        NVFP4_STEP(Ca, S0, 2, F0, F1)
        NVFP4_STEP(Ca, S0, 3, F1, F0)
        NVFP4_STEP(Cb, S1, 0, F0, F1)
        NVFP4_STEP(Cb, S1, 1, F1, F0)
        NVFP4_STEP(Cb, S1, 2, F0, F1)
        NVFP4_STEP(Cb, S1, 3, F1, F0)
        mma(F1);
    }
#undef NVFP4_STEP
#undef NVFP4_INTERLEAVE

    // epilogue.  The MFMA's first operand is the B (N-side) fragment, so a lane holds four consecutive columns of one row.
    __syncthreads();  // every wave has read the last K tile: the stages may be overwritten
    const int64_t row0 = m0 + wrow, col0 = n0 + wn * 32 * TB;
    uint8_t *const mine = lds + wave_wg * (32 * 32 * TB * (OUT_DT == NVFP4_F32 ? 4 : 2));
    if constexpr (KG == 1) {
        store_lines<OUT_DT, TB>(P, acc, row0, col0, mine, lane);
    } else {
        // the groups' sums over their own K tiles: two groups at a time, each keeping one half of the tile rows
        constexpr int LO = (TA + 1) / 2, HI = TA - LO;
        static_assert(KG == 4 && LO == 2, "four groups, three or four tile rows");
        float16_t half[LO][TB], last[1][TB];
        fold_groups<TA, TB, 2 * NW>(acc, half, lds, group >= 2, (group & 1) * NW + wave, lane);
        fold_groups<LO, TB, 2 * NW>(half, last, lds, group & 1, (group >> 1) * NW + wave, lane);
        // (of three tile rows the last group gets none)
        const int row = (group >> 1) * LO + (group & 1);
        if ((group & 1) < (group >= 2 ? HI : LO)) store_lines<OUT_DT, TB>(P, last, row0 + row * 32, col0, mine, lane);
    }
}

template <int B, int WM, int WN, int TA, int TB, int KG, int OUT_DT, bool KTAIL>
__global__ __launch_bounds__(64 * WM * WN * KG, 2) void gemm_nt_f16_kernel(TileArgs P)
{
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) % (WM * WN);
    f16_tile<B, WM, WN, TA, TB, KG, OUT_DT, KTAIL, 32 * TA * WM>(P, wave / WN * 32 * TA);
}

// 160 x 256: the upper four waves have 96 rows, the lower four 64, one of each on every SIMD, whose matrix unit is thus as busy as with two
// waves of 80.  Expansion of the operands bounds it as in the other tiles (2.06 us a K tile for 160 rows; 192 rows 2.33).  Which code a
// wave runs is uniform over the wave; both halves issue the same number of barriers (one per K tile), loads and stores included.
template <int B, int OUT_DT, bool KTAIL>
__global__ __launch_bounds__(512, 2) void gemm_nt_f16_uneven_kernel(TileArgs P)
{
    if (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) < 4) f16_tile<B, 2, 4, 3, 2, 1, OUT_DT, KTAIL, 160>(P, 0);
    else f16_tile<B, 2, 4, 2, 2, 1, OUT_DT, KTAIL, 160>(P, 96);
}
template <int B, bool KTAIL>
static void launch_f16_uneven(const TileArgs &P, int out_dt, hipStream_t st)
{
    constexpr int LDS_BYTES = 2 * (160 + 256) * (KTB + SROW);
    static_assert(LDS_BYTES >= 8 * 32 * 64 * 4, "the epilogue's pieces");
    const unsigned ntiles = (unsigned)(((P.N + 255) / 256) * ((P.M + 159) / 160));
    if (out_dt == NVFP4_F32) {
        auto k = gemm_nt_f16_uneven_kernel<B, NVFP4_F32, KTAIL>;
        static bool once = ((void)hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES), true);
        (void)once;
        hipLaunchKernelGGL(k, dim3(ntiles), dim3(512), LDS_BYTES, st, P);
    } else {
        auto k = gemm_nt_f16_uneven_kernel<B, NVFP4_BF16, KTAIL>;
        static bool once = ((void)hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES), true);
        (void)once;
        hipLaunchKernelGGL(k, dim3(ntiles), dim3(512), LDS_BYTES, st, P);
    }
}

template <int B, int WM, int WN, int TA, int TB, int KG, bool KTAIL>
static void launch_f16(const TileArgs &P, int out_dt, hipStream_t st)
{
    constexpr int BM = 32 * TA * WM, BN = 32 * TB * WN, NT = 64 * WM * WN * KG;
    // two stages per group, what a fold of the groups exchanges, or the epilogue's pieces (one per wave, 32 rows of fp32)
    constexpr int STAGES = KG * 2 * ((BM + BN) * KTB + (BM + BN) * SROW), PIECES = NT / 64 * 32 * 32 * TB * 4;
    constexpr int FOLD = KG == 1 ? 0 : KG / 2 * BM * BN * 4;
    constexpr int LDS_BYTES = STAGES > PIECES ? (STAGES > FOLD ? STAGES : FOLD) : (PIECES > FOLD ? PIECES : FOLD);
    static_assert(LDS_BYTES <= 160 * 1024, "LDS of a CU");
    const unsigned ntiles = (unsigned)(((P.N + BN - 1) / BN) * ((P.M + BM - 1) / BM));
    if (out_dt == NVFP4_F32) {
        auto k = gemm_nt_f16_kernel<B, WM, WN, TA, TB, KG, NVFP4_F32, KTAIL>;
        static bool once = ((void)hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES), true);
        (void)once;
        hipLaunchKernelGGL(k, dim3(ntiles), dim3(NT), LDS_BYTES, st, P);
    } else {
        auto k = gemm_nt_f16_kernel<B, WM, WN, TA, TB, KG, NVFP4_BF16, KTAIL>;
        static bool once = ((void)hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES), true);
        (void)once;
        hipLaunchKernelGGL(k, dim3(ntiles), dim3(NT), LDS_BYTES, st, P);
    }
}

// Products whose operands the dual quantizer hands over as slabs: large enough for the 256 x 256 tile.
static bool large_tile(int64_t M, int64_t N, int64_t K)
{
    const int64_t big = ((M + 255) / 256) * ((N + 255) / 256);
    return big >= 128 && K % KT == 0;  // (a slab holds whole K tiles)
}

bool gemm_takes_slabs(int64_t M, int64_t N, int64_t K, int block, int sf)
{
    if (sf == NVFP4_SCALE_E8M0) return block == 32 && mxfp4_gemm_takes_slabs(K);
    return sf == NVFP4_SCALE_E4M3 && block == 16 && large_tile(M, N, K);
}

template <int B>
static void launch_f16_tile(const TileArgs &P, GemmTile tile, int out_dt, hipStream_t st)
{
    const bool ktail = (P.K % KT) != 0;
    if (tile == TILE_256x256) {
        if (ktail) launch_f16<B, 2, 4, 4, 2, 1, true>(P, out_dt, st);
        else launch_f16<B, 2, 4, 4, 2, 1, false>(P, out_dt, st);
    } else if (tile == TILE_192x256) {
        if (ktail) launch_f16<B, 2, 4, 3, 2, 1, true>(P, out_dt, st);
        else launch_f16<B, 2, 4, 3, 2, 1, false>(P, out_dt, st);
    } else if (tile == TILE_160x256) {
        if (ktail) launch_f16_uneven<B, true>(P, out_dt, st);
        else launch_f16_uneven<B, false>(P, out_dt, st);
    } else if (tile == TILE_128x256) {
        if (ktail) launch_f16<B, 2, 4, 2, 2, 1, true>(P, out_dt, st);
        else launch_f16<B, 2, 4, 2, 2, 1, false>(P, out_dt, st);
    } else if (tile == TILE_128x128_K4) {
        if (ktail) launch_f16<B, 1, 2, 4, 2, 4, true>(P, out_dt, st);
        else launch_f16<B, 1, 2, 4, 2, 4, false>(P, out_dt, st);
    } else if (tile == TILE_96x128_K4) {
        if (ktail) launch_f16<B, 1, 2, 3, 2, 4, true>(P, out_dt, st);
        else launch_f16<B, 1, 2, 3, 2, 4, false>(P, out_dt, st);
    } else {
        if (ktail) launch_f16<B, 2, 2, 2, 2, 1, true>(P, out_dt, st);
        else launch_f16<B, 2, 2, 2, 2, 1, false>(P, out_dt, st);
    }
}

// Four waves of 128 columns where gemm_wide.h has the tile, but not for short contractions: with one wave per SIMD nothing covers the latencies of a start and an
// end (bf16 outputs, us, the kernels above / those: 2384 x 4096 x 288 11.6 / 12.7, x 512 13.2 / 14.0, x 768 17.0 / 17.4, 777 x 12288 x 512 13.2 / 14.0,
// x 1024 21.3 / 21.2, 320 x 32768 x 512 13.7 / 14.3, x 1024 22.4 / 21.7, 2505 x 3212 x 256 12.7 / 17.7, 3072 x 8192 x 512 29.8 / 31.0, x 1024 50.3 / 48.3,
// 4096 x 11008 x 512 54.3 / 54.5, x 1024 85.7 / 81.4).
// They fetch the scales of a row eight bytes at a time, so a row has to have as many; of more than seven K tiles it has (blocks of 128: K is a multiple
// of 128 too).
static bool wide_contraction(int64_t K) { return K > 7 * KT; }

// Which workgroup tile computes an M x N x K product: the one whose estimated time is least.  With R = the tiles of the
// busiest of the 256 CUs and S = the serial steps of a workgroup (K tiles of 128, divided among its waves or groups of waves),
//     time = fixed + R (tile + step S),      a little more where a CU has only one workgroup (R = 1, `alone` in percent).
// (NVFP4 and MXFP4 products of up to 16 rows have a kernel of their own, gemm_is_thin().)  Small tiles put more workgroups on the chip and walk K in parallel; large ones do less work per product (operand
// expansion, LDS reads).  The constants (nanoseconds) are fitted to every tile timed on 245 shapes from 9 x 162 x 768 to 11008 x 4096 x
// 4096, row-major and in slabs, both output types; those of the tiles that four waves of 128 columns serve from 16 K tiles on stand at wide_cost().  The present
// kernels' times on these shapes are in profiles/gemm_tiles.txt; the choice is 0.9 / 1.3 % (E4M3, bf16 / f32 outputs) and 1.3 / 1.4 % (E8M0) slower than the
// best tile on average.  E4M3, bf16 outputs, us per tile choice:
//                               32x32     64x64  96x128K4   128x128 128x128K4   128x256 128x256K2   160x256   192x256   256x256
//        64 x  4096 x 11008      11.7      26.5      47.3      78.7      58.6     117.9     103.6     143.2     153.3     182.0
//       256 x 11008 x  4096      41.4      30.2      43.7      32.3      27.2      46.2      45.8      57.7      63.6      75.1
//       512 x 11008 x  4096      81.9      57.8      68.2      54.3      56.3      49.0      47.8      59.4      64.5      76.3
//       777 x 12288 x  4096     150.6      96.7      92.9      85.6      86.1     103.2      95.4      65.6      72.6      78.4
//      1056 x  2080 x  2784      29.1      26.5      19.1      23.8      22.6      34.3      33.8      43.9      47.0      54.3
//      2048 x  4096 x  4096     137.9      80.8      73.9      64.6      64.9      61.6      55.4      64.9      67.1      77.5
//      2048 x  4096 x 11008     308.3     205.2     171.2     165.4     154.6     156.7     130.6     160.3     166.8     194.4
//      3072 x  8192 x  4096     378.5     229.3     200.9     182.9     186.7     179.1     159.5     188.9     152.0     144.9
//      4096 x  4096 x  4096     251.5     154.8     141.7     122.6     122.9     119.2     107.8     124.9     137.4      92.5
//      8192 x  8192 x   256     290.8     133.2     140.0      43.4     127.5      51.7         -      53.4      48.6      46.6
//      4096 x 11008 x   512     223.4      97.4      99.0      49.8      90.9      57.0         -      56.6      51.9      48.2
// (128 x 256 in two groups and 160 x 256 are for one round of them: see choose_gemm_tile().)
// (a short contraction wants small tiles: the waves of several workgroups per CU cover each other's epilogues; products that leave
// a 256 x 256 grid short of the 256 CUs, or just past a round of them, take 192 or 128 rows of the same eight waves.)
struct TileCost {
    int bm, bn, kwaves, threads;        // tile, waves that divide the contraction, workgroup size
    int fixed, tile, step, alone;       // ns, ns, ns, percent
};
static const TileCost E4M3_COST[TILES] = {
    {32, 32, 8, 512, 2900, 350, 860, 3},    {32, 64, 8, 512, 1300, 2400, 1430, 0},   {64, 32, 8, 512, 1400, 2300, 1410, 0},
    {64, 64, 4, 256, 3800, 770, 1115, 3},   {96, 128, 4, 512, 2000, 5600, 2600, 0},  {128, 128, 1, 256, 3700, 1200, 890, 8},
    {128, 128, 4, 512, 2300, 5070, 3350, 0}, {128, 256, 1, 512, 500, 3800, 1740, 0}, {128, 256, 2, 512, 2700, 3900, 3080, 0},
    {160, 256, 1, 512, 1500, 4500, 2060, 0}, {192, 256, 1, 512, 2500, 5200, 2330, 0},
    {0, 0, 0, 0, 0, 0, 0, 0},               {256, 256, 1, 512, 0, 8500, 2650, 0}};
static const TileCost E8M0_COST[TILES] = {
    {32, 32, 8, 512, 2700, 410, 585, 0},    {32, 64, 8, 512, 1400, 2140, 930, 0},    {64, 32, 8, 512, 1400, 2100, 935, 0},
    {64, 64, 4, 256, 3200, 910, 685, 0},    {0, 0, 0, 0, 0, 0, 0, 0},                {128, 128, 1, 256, 3200, 1390, 356, 28},
    {0, 0, 0, 0, 0, 0, 0, 0},               {0, 0, 0, 0, 0, 0, 0, 0},                {0, 0, 0, 0, 0, 0, 0, 0},                 {0, 0, 0, 0, 0, 0, 0, 0},
    {0, 0, 0, 0, 0, 0, 0, 0},               {256, 128, 1, 256, 2900, 3150, 556, 30}, {256, 256, 1, 512, 0, 8500, 1000, 0}};

// The same where four waves of 128 columns serve the tile (launch_gemm_wide()), us, estimate / measured: 4096 x 4096 x 1408 35.7 / 35.4, x 11008 226.9 / 226.9;
// 6720 x 1536 x 1408 29.4 / 27.2, 3072 x 4096 x 4096 73.9 / 73.9; 777 x 12288 x 1024 21.2 / 21.2, x 4096 65.8 / 65.9; 2048 x 4096 x 1536 25.0 / 24.4, x 4096 51.6 / 50.2,
// x 11008 123.4 / 123.5; and for the direct-to-LDS kernel in MXFP4: 4096 x 4096 x 4096 33.3 / 33.2, x 16384 111.5 / 111.3.
// From 16 K tiles on (12 in MXFP4); with the fewer of short contractions these estimates favour the large tiles too much (us, the choice without them / with:
// 3953 x 4992 x 960 43.1 / 45.7, 1906 x 9312 x 1056 45.7 / 48.5, 5847 x 3008 x 1472 58.6 / 60.3, 2429 x 7840 x 2016 80.6 / 81.3, 2599 x 1952 x 3008 44.0 / 38.5,
// 1591 x 7328 x 4736 105.9 / 96.9, 5803 x 6368 x 11776 767 / 710; MXFP4 4737 x 2208 x 512 8.6 / 10.1, 3098 x 2592 x 1024 10.7 / 11.8, 4998 x 1664 x 1664 15.6 / 14.5,
// 702 x 11872 x 2048 18.1 / 16.5, 4644 x 11648 x 7552 274 / 229).  Of 8 to 15 K tiles, which are chosen by the costs above and run on four waves, the
// choice is 0.5 / 0.2 % (bf16 / f32 outputs) slower than the best tile on average of 40 products.
static const TileCost *wide_cost(int tile, int64_t K, int sf)
{
    // (a round of several 4 to 7 % above one alone)
    static const TileCost k2 = {128, 256, 2, 512, 2700, 6550, 2765, -4}, r160 = {160, 256, 1, 512, 1500, 5000, 1935, -4},
                          r192 = {192, 256, 1, 512, 1000, 5300, 2205, -4}, r256 = {256, 256, 1, 512, 0, 8000, 2650, -4},
                          direct = {256, 256, 1, 512, 0, 7710, 873, -7};
    if (sf == NVFP4_SCALE_E8M0) return tile == TILE_256x256 && K > 11 * KT && mxfp4_gemm_takes_slabs(K) ? &direct : nullptr;
    if (K <= 15 * KT) return nullptr;
    return tile == TILE_128x256_K2 ? &k2 : tile == TILE_160x256 ? &r160 : tile == TILE_192x256 ? &r192 : tile == TILE_256x256 ? &r256 : nullptr;
}

// Whole rounds of 256 x 256 tiles and one of smaller ones in the place of the last, where the tiles do not fill that: as many tile columns (or rows) of
// 256 as the rounds before it hold, and a smaller tile for the rest, of which the CUs take one round (and the places that the first part leaves
// in its own last one).  Returns the estimated time in nanoseconds, 0 where there is no such division.
// The chip is bound by power, and idle CUs leave theirs to the others: of the 17 % that a round of 192 rows is shorter, a third comes back in a step (six such
// products and all else 2573 / 2553 us), and nothing with 16 K tiles (a backward call of two 607 / 611).  From 18 K tiles on.
// For whole K tiles, and where the rule below would choose 256 x 256, or three rounds or more of 192 x 256 at 4 % more by the estimates (us, without / with:
// 4096 x 11008 x 4096 272.7 / 261.9, 5000 x 5000 x 4096 168.9 / 161.1, 10587 x 3564 x 4224 275.0 / 254.9, 5004 x 7556 x 3584 236.0 / 220.9, 12020 x 3328 x 5504 in
// blocks of 64 335.8 / 302.5, 5714 x 6852 x 7296 with f32 outputs 446.4 / 401.4, 2793 x 10068 x 2560 124.2 / 126.0; in place of 192 x 256
// 9510 x 7272 x 3072 341.4 / 320.8, 7291 x 9712 x 2304 249.9 / 237.5).  Of two rounds of 192 x 256 some are faster and some slower: 2947 x 7552 x 9472 320.8 / 302.2,
// 2731 x 7460 x 5248 183.6 / 189.0, 5407 x 3836 x 2432 98.9 / 102.2; products that the rule gives 128 x 128 are faster there: 5276 x 3676 x 3328 117.2 / 128.8.
static double wide_mix(int64_t M, int64_t N, int64_t K, int sf, WideMix *X)
{
    if (sf != NVFP4_SCALE_E4M3 || K % KT || K <= 17 * KT) return 0;
    const int64_t ny = (M + 255) / 256, nx = (N + 255) / 256, steps = K / KT, full = (ny * nx - 1) / 256 * 256;
    if (full == 0 || ny * nx % 256 == 0 || full > (int64_t)1 << 20) return 0;
    const TileCost &big = *wide_cost(TILE_256x256, K, sf);
    double best = 0;
    for (int tile : {(int)TILE_192x256, (int)TILE_128x256_K2}) {
        const TileCost &c = *wide_cost(tile, K, sf);
        const double time = (double)(full / 256) * (big.tile + (double)big.step * (double)steps) + c.fixed + c.tile + (double)c.step * (double)((steps + c.kwaves - 1) / c.kwaves);
        for (int rows = 0; rows < 2; ++rows) {
            const int64_t across = rows ? nx : ny, split = full / across;
            const int64_t second = rows ? (M - split * 256 + c.bm - 1) / c.bm * nx : (M + c.bm - 1) / c.bm * (nx - split);
            if (split == 0 || second > 256 + full - split * across || (best != 0 && (time > best || (time == best && second >= X->second)))) continue;
            best = time;
            *X = {(unsigned)(split * across), (unsigned)second, (int)split, rows, tile};
        }
    }
    return best;
}

GemmTile choose_gemm_tile(int64_t M, int64_t N, int64_t K, int sf)
{
    const TileCost *const cost = sf == NVFP4_SCALE_E8M0 ? E8M0_COST : E4M3_COST;
    const int64_t nkt = (K + KT - 1) / KT;
    int best = TILE_256x256;
    double best_time = 0;
    for (int t = 0; t < TILES; ++t) {
        const TileCost *const wide = wide_cost(t, K, sf);
        const TileCost &c = wide ? *wide : cost[t];
        if (c.bm == 0) continue;  // (not built)
        const int64_t tiles = ((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn);
        if (tiles * c.threads > 0xFFFFFFFF) continue;  // (the threads of a launch are counted in 32 bits)
        // (the four-group tiles hold a whole CU each: beyond one round of them their times lie up to 12 % below and 23 % above the estimate's
        // other choice.  us, that choice / 96 x 128 with four groups: 1376 x 2432 x 12032, one round of 128 x 128, 99.6 / 81.6; two rounds
        // 6464 x 800 x 9856 139.1 / 127.2, 3072 x 1792 x 8256 102.2 / 121.7, 2377 x 1793 x 7552 with blocks of 64 92.9 / 109.2; three
        // 1280 x 6816 x 5760 103.3 / 118.8, 1381 x 5979 x 8800 167.4 / 202.9)
        if ((t == TILE_96x128_K4 || t == TILE_128x128_K4) && tiles > 256) continue;
        // The 160-row tile is for one round of them in place of one of 192 rows, where it covers the rows with less padding.  us, 192 / 160
        // rows: 777 x 12288 x 4096 74.6 / 65.4, 1600 x 6144 x 4096 69.2 / 64.9, 320 x 32768 x 1024 23.3 / 21.7, 2384 x 4096 x 512 13.3 / 12.5;
        // with as many rows or more there is little in it, and such products have not been moved to it: 960 x 10240 x 8192 126.7 / 123.2, 1281 x 7000 x
        // 1024 22.8 / 22.7.  Contractions of one K tile are slower on it (bf16 / f32 outputs, 192 and 128 rows / 160: 777 x 12288 x 128 6.6 / 7.4 and 10.6 / 11.2,
        // 3307 x 2944 x 128 6.9 / 9.0 and 10.3 / 12.0, 1352 x 7168 x 96 7.2 / 7.9 and 10.9 / 12.1); of two they would be faster (777 x 12288 x 256 10.5 / 9.4 and 14.6 /
        // 12.9, 2505 x 3212 x 256 12.6 / 12.0 and 16.1 / 14.1, 1079 x 9184 x 160 11.9 / 11.3 and 14.4 / 13.9), and have not been moved to it so far.
        if (t == TILE_160x256 && (K <= 256 || tiles > 256 || (M + 159) / 160 * 160 >= (M + 191) / 192 * 192)) continue;
        // 128 x 256 with two groups of two waves of 128 x 128 each, every other K tile (gemm_wide.h, which has it for contractions of more than seven
        // K tiles): 2 vector instructions a MFMA of 16 cycles, where eight waves of 64 x 64 need 8 a MFMA of 32, but one wave per SIMD and a fold at the
        // end, which 12 K tiles pay for.  One round of them, on most of the CUs.  us, one group / two: 2048 x 4096 x 4096 66.6 / 59.1, f32 outputs 65.3 /
        // 57.3, blocks of 64 60.7 / 54.6, 2048 x 4096 x 11008 162.0 / 131.5, 1700 x 4600 x 8192 120.6 / 101.3, 2688 x 2048 x 4096 52.1 / 48.9, 2048 x
        // 4096 x 1536 24.8 / 24.3, x 1280 21.3 / 21.4, x 1024 17.6 / 18.8.
        // Of up to 160 workgroups the estimate would give it some contractions of 1700 to 3300; most would be faster and some slower, and they have
        // not been moved to it so far (the choice / two groups): 908 x 4996 x 3296 55.1 / 47.9, 1664 x 2512 x 2784 43.5 / 39.6, 1302 x 3388 x 2656 36.3 / 38.7,
        // 1966 x 2337 x 2752 43.6 / 42.4.
        if (t == TILE_128x256_K2 && (!wide_contraction(K) || tiles <= 160 || tiles > 256)) continue;
        const int64_t rounds = (tiles + 255) / 256, steps = (nkt + c.kwaves - 1) / c.kwaves;
        double time = (double)rounds * ((double)c.tile + (double)c.step * (double)steps);
        if (rounds == 1) time *= 1.0 + 0.01 * c.alone;
        time += c.fixed;
        if (best_time == 0 || time < best_time) {
            best_time = time;
            best = t;
        }
    }
    WideMix X;
    if (best == TILE_192x256 && ((M + 191) / 192) * ((N + 255) / 256) > 512) {
        const double mixed = wide_mix(M, N, K, sf, &X);
        if (mixed != 0 && mixed < 0.96 * best_time) best = TILE_256x256;
    }
    return (GemmTile)best;
}

bool gemm_mixes_tiles(int64_t M, int64_t N, int64_t K, int sf, WideMix *X)
{
    return choose_gemm_tile(M, N, K, sf) == TILE_256x256 && wide_mix(M, N, K, sf, X) != 0;
}

void gemm_tile_size(GemmTile t, int *rows, int *cols)
{
    const TileCost &c = E4M3_COST[t].bm ? E4M3_COST[t] : E8M0_COST[t];
    *rows = c.bm;
    *cols = c.bn;
}

int gemm_tile_split(GemmTile t) { return E4M3_COST[t].bm ? E4M3_COST[t].kwaves : E8M0_COST[t].kwaves; }

static int g_fp4_rescale_route = 0;  // (measured slower than the fp16 route: opt-in)
void set_fp4_rescale_route(int on) { g_fp4_rescale_route = on; }
int fp4_rescale_route() { return g_fp4_rescale_route; }

bool gemm_reads_slabs(int64_t K, int block, int sf)
{
    return sf == NVFP4_SCALE_E8M0 ? block == 32 && mxfp4_gemm_takes_slabs(K) : block == 16 && K % KT == 0;
}

static hipError_t check_gemm(const GemmArgs &P, int block, int sf)
{
    // lane offsets inside a 256-row tile are 32-bit
    if ((P.K >> 1) * 256 >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
    if ((P.a_slab || P.b_slab) && !gemm_reads_slabs(P.K, block, sf)) return hipErrorInvalidValue;
    if (sf == NVFP4_SCALE_E8M0 && block != 32) return hipErrorNotSupported;
    return hipSuccess;
}

// (one workgroup per CU at most over both: two products that fill the chip by themselves gain nothing from sharing a launch)
bool gemm_pairs(const GemmArgs &P0, const GemmArgs &P1, int sf)
{
    const GemmTile t = choose_gemm_tile(P0.M, P0.N, P0.K, sf);
    if (t > TILE_64x64 || choose_gemm_tile(P1.M, P1.N, P1.K, sf) != t || g_fp4_rescale_route) return false;
    int bm, bn;
    gemm_tile_size(t, &bm, &bn);
    auto tiles = [&](const GemmArgs &P) { return ((P.M + bm - 1) / bm) * ((P.N + bn - 1) / bn); };
    return tiles(P0) + tiles(P1) <= 256;
}

hipError_t launch_gemm_pair(const GemmArgs &P0, const GemmArgs &P1, int block, int sf, int out_dt, hipStream_t st)
{
    hipError_t e = check_gemm(P0, block, sf);
    if (e == hipSuccess) e = check_gemm(P1, block, sf);
    return e != hipSuccess ? e : launch_gemm_ksplit(P0, &P1, choose_gemm_tile(P0.M, P0.N, P0.K, sf), block, sf, out_dt, st);
}

// Outputs up to this size leave by nontemporal stores, which do not wait for a place in the L2 (us, kept / streamed: NVFP4 1024 x 4096 x 4096,
// binary32 outputs, 37.1 / 36.1, bf16 34.4 / 33.7, 2048 x 4096 x 4096 52.7 / 51.1, 4096 x 4096 x 4096 87.0 / 85.2; MXFP4 2048 x 4096 x 4096 28.2 / 26.8,
// 4096 x 4096 x 4096 32.7 / 31.5), and still together with a kernel that reads the output next, but for the first (quantizer 44.2 / 44.5, 41.2 / 40.6, 60.1 / 59.4,
// 101.1 / 100.3; 31.6 / 30.8, 40.4 / 40.1).  Of larger ones the next kernel finds more in the last-level cache: MXFP4 5120 x 4096 x 4096, 40 MB, 62.7 / 62.3, with a
// quantizer behind it 72.6 / 73.2; 4096 x 11008 x 4096, 86 MB, 88.5 / 91.8 and 106.4 / 110.8.  (Weight gradients, which are not read next, of 90 MB, with the
// products of eight waves: the backward half of an MLP of 4096 / 11008 at 2048 tokens 697 / 706, the whole one at 4096 tokens 2872 / 2848: not done.)
// Calls on packed weights, quantizer and product, us, kept / streamed, one by one and from a graph, MXFP4: 2048 x 4096 x 4096 34.0 / 32.9 and 35.0 / 33.5,
// 1024 x 4096 x 4096 with binary32 outputs 31.4 / 29.9 and 30.5 / 29.2, 4096 x 4096 x 2048 (32 MB) 32.3 / 31.3 and 31.8 / 30.6; of 70 random ones with 4 to
// 32 MB 0.97 to 1.10 times as fast (less than 0.99: 3076 x 928 x 928 and 3857 x 928 x 960, NVFP4), 628 x 5888 x 5504 with binary32 outputs 40.8 / 41.0 and
// 39.7 / 38.7 (all with the kernels on 32 x 32 MFMAs).  Rows 32 KB apart are an exception near the line (the product, and with a quantizer of its output): MXFP4
// 1024 x 8192 x 1024 with binary32 outputs 14.3 / 14.7 and 28.4 / 28.9, NVFP4 22.7 / 22.5 and 41.3 / 41.6; MXFP4 896 x 8192 x 1024 12.9 / 11.7 and 25.1 / 24.8,
// 31 KB apart, 1024 x 7936 x 2048, 18.0 / 16.7 and 27.0 / 25.8.
// The rule's answer is an argument of the larger tiles' kernels alone.  As a member of GemmArgs it lengthened the small products' arguments (two of these: 212
// bytes instead of 196), and with them the host's work for a launch: a call of 64 x 4096 x 11008 MXFP4 on packed weights kept the host 8.80 us instead of
// 8.50 (two libraries in turn in one process; on another box 5.45 and 5.41).  Asked in the kernels, from M and ldc, it had the 256 x 256 MXFP4 ones spill
// registers: an MLP of 4096 / 11008 at 4096 tokens, three layers forward and backward, 1128 us instead of 1118.
static bool streamed_output(int64_t rows, int64_t row_bytes)
{
    return rows * row_bytes <= (row_bytes == 32 << 10 ? (int64_t)28 << 20 : (int64_t)32 << 20);
}

// (false: not one of the tiles of gemm_wide.h, or a short contraction)
static bool launch_gemm_wide(const TileArgs &P, GemmTile tile, int block, int out_dt, hipStream_t st)
{
    if (!wide_contraction(P.K) || P.K / block < 8) return false;
    WideMix X;
    if (tile == TILE_256x256 && wide_mix(P.M, P.N, P.K, NVFP4_SCALE_E4M3, &X) != 0) {  // (gemm_mixes_tiles() says the same)
        switch (block) {
        case 16: launch_gemm_wide_mixed16(P, X, out_dt, st); return true;
        case 32: launch_gemm_wide_mixed32(P, X, out_dt, st); return true;
        case 64: launch_gemm_wide_mixed64(P, X, out_dt, st); return true;
        case 128: launch_gemm_wide_mixed128(P, X, out_dt, st); return true;
        }
    }
    switch (block) {
    case 16: return launch_gemm_wide16(P, tile, out_dt, st);
    case 32: return launch_gemm_wide32(P, tile, out_dt, st);
    case 64: return launch_gemm_wide64(P, tile, out_dt, st);
    case 128: return launch_gemm_wide128(P, tile, out_dt, st);
    default: return false;
    }
}

hipError_t launch_gemm(const GemmArgs &P, int block, int sf, int out_dt, hipStream_t st)
{
    const hipError_t e = check_gemm(P, block, sf);
    if (e != hipSuccess) return e;
    const TileArgs T{P, streamed_output(P.M, P.ldc * (out_dt == NVFP4_F32 ? 4 : 2))};
    if (sf == NVFP4_SCALE_E4M3 && g_fp4_rescale_route && fp4_rescale_gemm_applies(P.K, block, P)) return launch_gemm_fp4_rescale(T, block, out_dt, st);
    if (gemm_is_thin(P.M, P.N, P.K, block, sf)) return launch_gemm_thin(P, sf, out_dt, st);
    const GemmTile tile = choose_gemm_tile(P.M, P.N, P.K, sf);
    if (tile <= TILE_64x64) return launch_gemm_ksplit(P, nullptr, tile, block, sf, out_dt, st);
    if (sf == NVFP4_SCALE_E8M0) return launch_gemm_mxfp4(T, tile, out_dt, st);
    if (launch_gemm_wide(T, tile, block, out_dt, st)) return hipGetLastError();
    switch (block) {
    case 16: launch_f16_tile<16>(T, tile, out_dt, st); break;
    case 32: launch_f16_tile<32>(T, tile, out_dt, st); break;
    case 64: launch_f16_tile<64>(T, tile, out_dt, st); break;
    case 128: launch_f16_tile<128>(T, tile, out_dt, st); break;
    default: return hipErrorNotSupported;
    }
    return hipGetLastError();
}

}  // namespace nvfp4
