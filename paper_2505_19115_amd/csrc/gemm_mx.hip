// MXFP4 GEMM on the CDNA4 scaled FP4 MFMA ("NT": both operands stored with the contraction
// axis contiguous).  MXFP4 (Sec. 3 / Table 1 of "FP4 All the Way": E2M1 elements, blocks of 32,
// E8M0 power-of-two scales) is exactly what v_mfma_scale_f32_16x16x128_f8f6f4 (and 32x32x64) consumes: each
// lane supplies 32 consecutive contraction elements (16 bytes of packed codes) of one row plus
// one E8M0 byte for them, so the packed operands go from LDS straight into the instruction with
// no expansion arithmetic at all:
//     out[i, j] = gA gB sum_b 2^(eA[i,b] - 127) 2^(eB[j,b] - 127) sum_{k in b} cA[i,k] cB[j,k].
// Products and the power-of-two scaling are exact; accumulation is fp32.
//
// Geometry of the main kernel and of the rescaling one: 256 threads = 2 x 2 waves, wave tile 128 x 128 (8 x 8 MFMA tiles of 16 x 16 in the main kernel, whose
// 16x16x128 instruction takes less power: 6.95 PFLOP/s in registers against 6.33; 4 x 4 of 32 x 32 in the other; all
// 256 accumulator registers, one wave per SIMD), workgroup tile 256 x 256: with no VALU work in
// the loop what matters is bytes moved per MFMA, hence the largest register tile that fits.  The MFMA's first operand is the B (N-side)
// tile, so a lane's accumulator holds four consecutive output COLUMNS of one row.
#include <type_traits>

#include "kernels.h"
#include "mx_codes.h"
#include "nvfp4_math.h"
#include "store_lines.h"

namespace nvfp4 {

typedef int int8v_t __attribute__((ext_vector_type(8)));
typedef float float16v_t __attribute__((ext_vector_type(16)));
typedef float float4v_t __attribute__((ext_vector_type(4)));

namespace mx {
constexpr int NT = 256, BM = 256, BN = 256, TA = 4, TB = 4;
}

// ---------------------------------------------------------------------------------------------
// E4M3 block scales at blocks of 64 and 128 on the FP4 matrix instruction (the block-size study of Sec. 3.1 / Fig. 2):
// an E4M3 scale has a mantissa, which the instruction's power-of-two scale operand cannot carry, so the blocks are
// multiplied with unit scales and the partial sum of each block is rescaled in binary32:
//     acc[i, j] += P_b[i, j] * (sA[i, b] * sB[j, b]),      P_b = sum_{k in b} cA[i, k] cB[j, k].
// P_b is exact (a multiple of 1/4 below 2^13), the product of two E4M3 values is exact (8 significant bits), and so is
// their product with P_b (<= 23 bits): every term enters the accumulator with the one rounding of the addition, as in
// the other kernels.  One 32 x 32 x 64 MFMA is exactly one block of 64; two chained ones are one block of 128.  The
// cost is on the vector ALU: 16 scale products and 16 multiply-adds per 32 x 32 tile and block.
// K tile 128 = two MFMA steps; step s of lane half g multiplies chunk 2 s + g, so a step covers elements 64 s .. 64 s + 63
// of the tile (one block of 64, half a block of 128).  Two LDS stages, everything staged through registers; the block
// scales are decoded to binary32 when they are staged.  K must be a multiple of 128; rows past the edge are clamped.
namespace mxr {
constexpr int KT = 128, ROWB = 64;
constexpr int CODES = (mx::BM + mx::BN) * ROWB;              // 32 KB
constexpr int STAGE = CODES + 2 * (mx::BM + mx::BN) * 4;     // + decoded scales [2 blocks][512 rows]
constexpr int LDS_BYTES = 2 * STAGE;                         // 72 KB (>= the 64 KB the fp32 epilogue borrows)
}  // namespace mxr

template <int OUT_DT, int B>
__global__ __launch_bounds__(256) void gemm_nt_fp4_rescale_kernel(TileArgs P)
{
    using namespace mx;
    using namespace mxr;
    static_assert(B == 64 || B == 128, "blocks that are whole MFMA steps");
    constexpr int NBLK = KT / B;  // blocks per K tile
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int r = lane & 31, g = lane >> 5;
    const int ntx = (int)((P.N + BN - 1) / BN), nty = (int)((P.M + BM - 1) / BM);
    int ty, tx;
    tile_coords((int)blockIdx.x, ntx, nty, ty, tx);
    const int64_t m0 = (int64_t)ty * BM, n0 = (int64_t)tx * BN;
    const int64_t Kb = P.K >> 1, Ks = P.K / B;
    const int nkt = (int)(P.K / KT);

    float16v_t acc[TA][TB];
#pragma unroll
    for (int a = 0; a < TA; ++a)
#pragma unroll
        for (int b = 0; b < TB; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.0f;

    // ---- global -> registers -> LDS: thread t stages chunks t, t + 256, t + 512, t + 768 (row = chunk / 4) of each operand
    uint4 ga[4], gb[4];
    float gsa[NBLK], gsb[NBLK];
    const uint8_t *pA[4], *pB[4];
    int ldsW[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int qd = tid + NT * u, row = qd >> 2, c = qd & 3;
        const int64_t ar = m0 + row < P.M ? m0 + row : P.M - 1, br = n0 + row < P.N ? n0 + row : P.N - 1;
        pA[u] = P.A_codes + ar * Kb + c * 16;
        pB[u] = P.B_codes + br * Kb + c * 16;
        ldsW[u] = row * ROWB + ((c ^ ((row >> 2) & 3)) << 4);
    }
    const int64_t sar = m0 + tid < P.M ? m0 + tid : P.M - 1, sbr = n0 + tid < P.N ? n0 + tid : P.N - 1;
    auto fetch = [&](int kt) {
        const int64_t kb = (int64_t)kt * ROWB;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            ga[u] = *reinterpret_cast<const uint4 *>(pA[u] + kb);
            gb[u] = *reinterpret_cast<const uint4 *>(pB[u] + kb);
        }
#pragma unroll
        for (int q = 0; q < NBLK; ++q) {
            gsa[q] = e4m3_decode(P.A_scales[sar * Ks + (int64_t)kt * NBLK + q]);
            gsb[q] = e4m3_decode(P.B_scales[sbr * Ks + (int64_t)kt * NBLK + q]);
        }
    };
    auto stash = [&](int stage) {
        uint8_t *base = lds + stage * STAGE;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            *reinterpret_cast<uint4 *>(base + ldsW[u]) = ga[u];
            *reinterpret_cast<uint4 *>(base + BM * ROWB + ldsW[u]) = gb[u];
        }
        float *sS = reinterpret_cast<float *>(base + CODES);
#pragma unroll
        for (int q = 0; q < NBLK; ++q) {
            sS[q * (BM + BN) + tid] = gsa[q];
            sS[q * (BM + BN) + BM + tid] = gsb[q];
        }
    };

    const int sw = (r >> 2) & 3;
    // one K tile: per step the 8 fragments, per block the lane's scales (its row of each A fragment, its 16 columns of
    // each B fragment), then 16 tiles of MFMA (+ MFMA) and rescale
    auto tile = [&](int stage) {
        const uint8_t *cbase = lds + stage * STAGE;
        const float *sS = reinterpret_cast<const float *>(cbase + CODES);
        // the A fragments of both steps stay in registers; B fragments and B scales are fetched per column of tiles
        uint4 fa[2][TA];
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int a = 0; a < TA; ++a)
                fa[s][a] = *reinterpret_cast<const uint4 *>(cbase + (((2 * s + g) ^ sw) << 4) + (wm * 128 + 32 * a + r) * ROWB);
#pragma unroll
        for (int q = 0; q < NBLK; ++q) {
            float sa[TA];
#pragma unroll
            for (int a = 0; a < TA; ++a) sa[a] = sS[q * (BM + BN) + wm * 128 + 32 * a + r];
#pragma unroll
            for (int b = 0; b < TB; ++b) {
                float4 sb[4];
#pragma unroll
                for (int c4 = 0; c4 < 4; ++c4)
                    sb[c4] = *reinterpret_cast<const float4 *>(&sS[q * (BM + BN) + BM + wn * 128 + 32 * b + 8 * c4 + 4 * g]);
                uint4 fb[2];
#pragma unroll
                for (int s = 0; s < 2; ++s)
                    fb[s] = *reinterpret_cast<const uint4 *>(cbase + (((2 * s + g) ^ sw) << 4) + (BM + wn * 128 + 32 * b + r) * ROWB);
#pragma unroll
                for (int a = 0; a < TA; ++a) {
                    float16v_t t;
#pragma unroll
                    for (int v = 0; v < 16; ++v) t[v] = 0.0f;
                    // B = 128: both steps belong to the one block; B = 64: step q is block q
#pragma unroll
                    for (int s = (B == 128 ? 0 : q); s < (B == 128 ? 2 : q + 1); ++s) {
                        const int8v_t va = {(int)fa[s][a].x, (int)fa[s][a].y, (int)fa[s][a].z, (int)fa[s][a].w, 0, 0, 0, 0};
                        const int8v_t vb = {(int)fb[s].x, (int)fb[s].y, (int)fb[s].z, (int)fb[s].w, 0, 0, 0, 0};
                        t = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(vb, va, t, 4, 4, 0, 0x7F7F7F7F, 0, 0x7F7F7F7F);
                    }
#pragma unroll
                    for (int c4 = 0; c4 < 4; ++c4) {
                        acc[a][b][4 * c4 + 0] = __builtin_fmaf(t[4 * c4 + 0], sa[a] * sb[c4].x, acc[a][b][4 * c4 + 0]);
                        acc[a][b][4 * c4 + 1] = __builtin_fmaf(t[4 * c4 + 1], sa[a] * sb[c4].y, acc[a][b][4 * c4 + 1]);
                        acc[a][b][4 * c4 + 2] = __builtin_fmaf(t[4 * c4 + 2], sa[a] * sb[c4].z, acc[a][b][4 * c4 + 2]);
                        acc[a][b][4 * c4 + 3] = __builtin_fmaf(t[4 * c4 + 3], sa[a] * sb[c4].w, acc[a][b][4 * c4 + 3]);
                    }
                }
            }
        }
    };

    fetch(0);
    stash(0);
    __syncthreads();
    for (int kt = 0; kt < nkt; ++kt) {
        const int stage = kt & 1;
        const bool more = kt + 1 < nkt;
        if (more) fetch(kt + 1);
        tile(stage);
        if (more) stash(stage ^ 1);  // the other stage: every wave finished reading it before the previous barrier
        __syncthreads();
    }
    constexpr int PIECE = 32 * 32 * TB * (OUT_DT == NVFP4_F32 ? 4 : 2);  // of the epilogue, per wave
    const int w = __builtin_amdgcn_readfirstlane(wave);
    store_lines<OUT_DT, TB>(P, acc, m0 + (w >> 1) * 128, n0 + (w & 1) * 128, lds + w * PIECE, lane);
}

// ---------------------------------------------------------------------------------------------
// Main kernel (K a multiple of 128 and at least 512, 16-byte aligned codes): four LDS stages of
// 128 contraction elements, every byte written by direct global -> LDS loads, three K tiles in
// flight, one barrier per tile, no VALU work in the loop.
//
// What bounds the loop besides the MFMA pipe is the vector L1: it takes one request (at most 64
// bytes) per clock, and a lane-per-row load costs one request per lane however few bytes it
// fetches.  The codes need 512 requests per tile (64 bytes per row); the scales are therefore
// fetched 16 bytes per row at a time = FOUR tiles' worth in one request, into a double-buffered
// scale area, instead of one dword per row per tile.
//
// LDS: four code stages [512 rows][64 bytes] with the 16-byte chunk c of row r at slot
// c ^ quad_xor(r / 4): the sixteen lanes that the LDS serves at a time cover all sixteen 16-byte
// slots of the 256-byte bank period; two scale buffers [512 rows][16 bytes] (a group of four K
// tiles each); 4 KB that absorbs the filler loads.  Lane group g (16 lanes) of a
// 16x16x128 MFMA multiplies chunk g of its row with scale byte g of the K tile.
//
// An operand in the slab layout (A_SLAB / B_SLAB) brings its scales as slabs too: 256 positions x 4 bytes per K
// tile, contiguous, so ONE instruction of one wave fetches the scales of a whole K tile (wave 0: A, wave 1: B), they
// travel with the codes of their tile through four 1 KB stages (which take the place of that operand's part of the
// first scale buffer), and lane group g reads byte g of its row's dword at position slab_row(row): 16 rows are 16 different banks, and yet each such read
// takes two cycles more (128 per K tile and CU, all that is left of conflicts in the loop).  Row-major scales lie 16 bytes apart in LDS.
//
// Every wave issues the same direct-to-LDS instructions per K tile, which the counted waits rely on: 4 + 4 codes, one slot for a
// row-major scale group where an operand is row-major and one for a scale slab where one comes in slabs; a slot with nothing to fetch
// issues a one-request filler.
//
// The MFMA's first operand is the B (N-side) tile, so a lane's accumulator holds four consecutive
// output COLUMNS of one row: the epilogue is one packed convert pair and one 8-byte (bf16) or
// 16-byte (fp32) store per four outputs.
namespace mxd {
constexpr int KT = 128, ROWB = 64, NS = 4;
constexpr int STAGE = (mx::BM + mx::BN) * ROWB;        // 32 KB of codes
constexpr int SBUF = (mx::BM + mx::BN) * 16;           // 8 KB: the scales of four K tiles
constexpr int SCALES0 = NS * STAGE, DUMP0 = SCALES0 + 2 * SBUF;
constexpr int LDS_BYTES = DUMP0 + 4096;
constexpr int FA = 8, FB = 8;  // fragments of 16 rows of a wave's part of A and of B
}  // namespace mxd

// Written as assembly so that the 64 accumulators stay where they are: through the builtin the compiler moves them between the two halves of
// the register file all the time and spills (some 700 moves per K tile).  What the compiler cannot know about it: an operand must not
// have been written by the vector ALU in the two instructions before (here all come from LDS reads), and the result of the last one
// must not be read for 11 wait states.
__device__ __forceinline__ void mfma_16x16x128(float4v_t &acc, const uint4 &b, const uint4 &a, uint32_t sb, uint32_t sa)
{
    typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
    const u32x4_t vb = {b.x, b.y, b.z, b.w}, va = {a.x, a.y, a.z, a.w};
    asm volatile("v_mfma_scale_f32_16x16x128_f8f6f4 %0, %1, %2, %0, %3, %4 op_sel_hi:[0,0,0] cbsz:4 blgp:4" : "+a"(acc) : "v"(vb), "v"(va), "v"(sb), "v"(sa));
}

template <int OUT_DT, bool A_SLAB, bool B_SLAB>
__global__ __launch_bounds__(256) void gemm_nt_mxfp4_dma_kernel(TileArgs P)
{
    using namespace mx;
    using namespace mxd;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int r = lane & 15, g = lane >> 4;
    const int ntx = (int)((P.N + BN - 1) / BN), nty = (int)((P.M + BM - 1) / BM);
    int ty, tx;
    tile_coords((int)blockIdx.x, ntx, nty, ty, tx);
    const int64_t m0 = (int64_t)ty * BM, n0 = (int64_t)tx * BN;
    const int64_t Kb = P.K >> 1, Ks = P.K >> 5;
    const int nkt = (int)(P.K / KT);

    float4v_t acc[FA / 2][2 * FB];  // (tile rows in pairs, as the epilogue takes them)
#pragma unroll
    for (int a = 0; a < FA / 2; ++a)
#pragma unroll
        for (int b = 0; b < 2 * FB; ++b) acc[a][b] = float4v_t{0.0f, 0.0f, 0.0f, 0.0f};

    // ---- global -> LDS.  A code instruction fills 1 KB = 16 consecutive tile rows, lane i landing
    // at byte 16 i (row i / 4, slot i % 4), so the swizzle is applied by choosing WHICH global chunk
    // the lane fetches.  Rows past the edge are clamped to the last row (their products land in
    // outputs that are never stored).  Lane offsets are relative to the tile's first row, the
    // 64-bit part of the address is wave-uniform (mx_codes.h).
    const int64_t mrows = P.M - m0 < BM ? P.M - m0 : BM, nrows = P.N - n0 < BN ? P.N - n0 : BN;
    MxCodes<A_SLAB> A;
    MxCodes<B_SLAB> B;
    const int c = (lane & 3) ^ quad_xor(lane >> 4);
    A.lane_offsets(wave, lane, c, mrows, Kb);
    B.lane_offsets(wave, lane, c, nrows, Kb);
    const int srow = wave * 64 + lane;
    const uint32_t offSA = (uint32_t)((srow < mrows ? srow : mrows - 1) * Ks);
    const uint32_t offSB = (uint32_t)((srow < nrows ? srow : nrows - 1) * Ks);
    typedef __attribute__((address_space(3))) void *lds_ptr_t;
    auto uniform_ptr = [](const uint8_t *p) -> const uint8_t * {
        const uint64_t v = reinterpret_cast<uint64_t>(p);
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
        return reinterpret_cast<const uint8_t *>(((uint64_t)hi << 32) | lo);
    };
    // Issued through inline assembly on purpose: the compiler's wait-count pass treats a
    // direct-to-LDS load as a possible writer of every LDS location and would wait for ALL of them
    // before the next LDS read.  Here a stage is never read before the explicit counted wait and
    // the barrier that follow its loads.  In two parts: the destination goes into m0 (nothing else here uses it), and the load follows
    // at least one instruction later.
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr_t)lds;
#define NVFP4_MXD_DST(base, more) asm volatile("s_add_u32 m0, %0, %1" : : "s"(base), "n"(more) : "scc", "m0");
#define NVFP4_MXD_LOAD(voff, base, more) asm volatile("global_load_lds_dwordx4 %0, %1 offset:%2" : : "v"(voff), "s"(base), "n"(more) : "memory");
    // part u of four of an operand's codes into stage st.  The constant of a slab's load counts for both of its addresses.
#define NVFP4_MXD_DST_A(st, u) NVFP4_MXD_DST(code_dst, (st) * STAGE + (u) * (1024 - A.more(1)))
#define NVFP4_MXD_DST_B(st, u) NVFP4_MXD_DST(code_dst, (st) * STAGE + BM * ROWB + (u) * (1024 - B.more(1)))
#define NVFP4_MXD_LOAD_A(u) NVFP4_MXD_LOAD(A.off[A_SLAB ? 0 : (u)], A.p, A.more(u))
#define NVFP4_MXD_LOAD_B(u) NVFP4_MXD_LOAD(B.off[B_SLAB ? 0 : (u)], B.p, B.more(u))
    const uint32_t code_dst = __builtin_amdgcn_readfirstlane(lds0 + wave * 4096);
    A.start(uniform_ptr(A_SLAB ? P.A_codes + (int64_t)ty * nkt * SLAB_CODE_BYTES : P.A_codes + m0 * Kb));  // (A.p: K tile kt + 4 in the loop)
    B.start(uniform_ptr(B_SLAB ? P.B_codes + (int64_t)tx * nkt * SLAB_CODE_BYTES : P.B_codes + n0 * Kb));  // (B.p: kt + 3)
    // Scale slabs (one per K tile): wave 0 fetches A's, wave 1 B's, 16 bytes per lane, into stage kt % 4 of that operand's part of the first
    // scale buffer; the other waves (and a wave whose operand is row-major) issue a one-request filler (the first bytes of A's codes: a
    // valid address in both layouts), so that every wave has the same number of loads per tile, which the counted waits rely on.
    constexpr bool SLABS = A_SLAB || B_SLAB, GROUPS = !A_SLAB || !B_SLAB;
    const int wave_s = __builtin_amdgcn_readfirstlane(wave);
    const bool slab_loader = (wave_s == 0 && A_SLAB) || (wave_s == 1 && B_SLAB);
    const uint8_t *slab_ptr = uniform_ptr(!slab_loader ? A.tile
                                          : wave_s == 0   ? P.A_scales + (int64_t)ty * nkt * SLAB_MX_SCALE_BYTES
                                                       : P.B_scales + (int64_t)tx * nkt * SLAB_MX_SCALE_BYTES);
    uint32_t slab_step = __builtin_amdgcn_readfirstlane(slab_loader ? (uint32_t)SLAB_MX_SCALE_BYTES : 0u);
    uint32_t slab_voff = slab_loader ? (uint32_t)lane * 16 : 0u;
    const uint32_t slab_dst = __builtin_amdgcn_readfirstlane(lds0 + (slab_loader ? SCALES0 + wave_s * BM * 16 : DUMP0));
    // Row-major scales.  Group G = the 16 scale bytes of a row that cover K tiles 4 G .. 4 G + 3; the window of the
    // last group is moved back to end with the row (Ks >= 16), so no load passes the end of a row.  Part 0: this wave's 64 A rows, part 1:
    // its 64 B rows.
    const uint8_t *const rowsSA = P.A_scales + m0 * Ks, *const rowsSB = P.B_scales + n0 * Ks;
    const uint32_t scale_dst = __builtin_amdgcn_readfirstlane(lds0 + SCALES0 + wave * 1024), dump_dst = __builtin_amdgcn_readfirstlane(lds0 + DUMP0);
    auto group_start = [&](int G) -> int { return 16 * G + 16 <= Ks ? 16 * G : (int)Ks - 16; };
    auto group_dst = [&](int G, int part, bool real) {
        const uint32_t d = __builtin_amdgcn_readfirstlane(real ? scale_dst + (G & 1) * SBUF + part * (BM * 16) : dump_dst);
        NVFP4_MXD_DST(d, 0)
    };
    // (the compiler selects the address in vector registers and reads the lane back; the load has to come five wait states after that)
    auto group_load = [&](int G, int part, bool real) {
        const uint8_t *const base = uniform_ptr(real ? (part ? rowsSB : rowsSA) + group_start(G) : A.tile);
        const uint32_t off = real ? (part ? offSB : offSA) : 0u;
        asm volatile("s_nop 4\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(off), "s"(base) : "memory");
    };

    // ---- LDS -> registers: fragment i of an operand is its rows 16 i + r, of which lane group g reads the 16-byte chunk g and the
    // scale byte g
    struct Frags {
        uint4 a[FA], b[FB];
        uint32_t sa[FA], sb[FB];
    };
    // (an LDS instruction's constant reaches 64 KB, two stages: a base for each two, hidden from the compiler, which would add them up for
    // each tile)
    const uint8_t *baseA[2], *baseB[2], *baseSA, *baseSB;
    baseA[0] = lds + (wm * 128 + r) * ROWB + ((g ^ quad_xor(r >> 2)) << 4);
    baseB[0] = baseA[0] + (BM + (wn - wm) * 128) * ROWB;
    baseA[1] = baseA[0] + 2 * STAGE;
    baseB[1] = baseB[0] + 2 * STAGE;
    // scale bytes of fragment i (rows 16 i + r of the wave's part): row-major image [row][16 bytes], or the slab
    // image [position][4 bytes] with the row at position slab_row(row) (for row 128 w + 16 i + r that is
    // 128 w + 64 (i / 4) + 8 (r % 8) + 2 (i % 4) + r / 8: a lane part plus a constant per fragment)
    baseSA = lds + SCALES0 + g + (A_SLAB ? slab_row(wm * 128 + r) * 4 : (wm * 128 + r) * 16);
    baseSB = lds + SCALES0 + g + BM * 16 + (B_SLAB ? slab_row(wn * 128 + r) * 4 : (wn * 128 + r) * 16);
#define NVFP4_MXD_HIDE(p) { uint32_t v = (uint32_t)(uintptr_t)(lds_ptr_t)(p); asm volatile("" : "+v"(v)); (p) = (const uint8_t *)(lds_ptr_t)(uintptr_t)v; }
    NVFP4_MXD_HIDE(baseA[0]) NVFP4_MXD_HIDE(baseA[1]) NVFP4_MXD_HIDE(baseB[0]) NVFP4_MXD_HIDE(baseB[1]) NVFP4_MXD_HIDE(baseSA) NVFP4_MXD_HIDE(baseSB)
    auto frag_off = [](bool slab, int i) -> int { return slab ? 256 * (i >> 2) + 8 * (i & 3) : 256 * i; };
    // where in the scale area the dwords of K tile kt, in stage st, start
    auto tile_off = [&](bool slab, int kt, int st) -> int {
        const int G = kt >> 2;
        return slab ? st * 1024 : (G & 1) * SBUF + (4 * kt - group_start(G));
    };
    // half h (fragments 4 h .. 4 h + 3) of an operand of the K tile in stage st, in eight reads, scales (at `scales`) first
    auto read_a = [&](int st, const uint8_t *scales, Frags &F, int h, int i) {
        const int f = 4 * h + (i & 3);
        if (i < 4) F.sa[f] = scales[frag_off(A_SLAB, f)];
        else F.a[f] = *reinterpret_cast<const uint4 *>(baseA[st >> 1] + (st & 1) * STAGE + 16 * f * ROWB);
    };
    auto read_b = [&](int st, const uint8_t *scales, Frags &F, int h, int i) {
        const int f = 4 * h + (i & 3);
        if (i < 4) F.sb[f] = scales[frag_off(B_SLAB, f)];
        else F.b[f] = *reinterpret_cast<const uint4 *>(baseB[st >> 1] + (st & 1) * STAGE + 16 * f * ROWB);
    };
    // one MFMA: output rows of A fragment ia against B fragment ib.  The first MFMA operand is the
    // B tile (its rows become accumulator rows), the second the A tile.
    auto mma = [&](const Frags &F, int ia, int ib) { mfma_16x16x128(acc[ia >> 1][FB * (ia & 1) + ib], F.b[ib], F.a[ia], F.sb[ib], F.sa[ia]); };
    // MFMA j of two quarters -> fragments of A and B inside their halves: there and back, so that one operand of two changes from one MFMA to
    // the next, also from quarter to quarter
    auto there_and_back = [](int j) -> int2 {
        const int row = j >> 2 & 3, i = j & 3;
        return make_int2(j < 16 ? row : 3 - row, row & 1 ? 3 - i : i);
    };
    // wait until at most n direct-to-LDS instructions of this wave are still in flight
#define NVFP4_MXD_WAIT(n) asm volatile("s_waitcnt vmcnt(%0)" : : "n"(n) : "memory");
    constexpr int PER_TILE = 8 + SLABS + GROUPS;  // direct-to-LDS instructions per wave and K tile

    Frags F;
    // (at the end of a tile, the next one's first scales: else the compiler carries them as bytes and masks them again)
    auto keep_scales = [](Frags &F, auto half) {
        __builtin_amdgcn_s_waitcnt(0xC37F);  // lgkmcnt(3): three of the fragments are still under way
#pragma unroll
        for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(F.sa[i]), "+v"(F.sb[4 * decltype(half)::value + i]));
    };
    // K tiles 0 to 2 and A's part of tile 3; scale group 0 rides with tile 0
    if (GROUPS) {
        group_dst(0, 0, !A_SLAB);
        group_load(0, 0, !A_SLAB);
        group_dst(0, 1, !B_SLAB);
        group_load(0, 1, !B_SLAB);
    }
    auto prologue = [&](auto st) {
        constexpr int S = decltype(st)::value;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            NVFP4_MXD_DST_A(S, u)
            asm volatile("s_nop 4");
            NVFP4_MXD_LOAD_A(u)
            if (S < 3) {
                NVFP4_MXD_DST_B(S, u)
                asm volatile("s_nop 4");
                NVFP4_MXD_LOAD_B(u)
            }
        }
        A.advance();
        if (S < 3) {
            B.advance();
            if (SLABS) {
                NVFP4_MXD_DST(slab_dst, S * 1024)
                asm volatile("s_nop 4");
                NVFP4_MXD_LOAD(slab_voff, slab_ptr, 0)
                slab_ptr += slab_step;
            }
            if (GROUPS && S > 0) {
                group_dst(0, 0, false);
                group_load(0, 0, false);
            }
        }
    };
    prologue(std::integral_constant<int, 0>{});
    prologue(std::integral_constant<int, 1>{});
    prologue(std::integral_constant<int, 2>{});
    prologue(std::integral_constant<int, 3>{});
    NVFP4_MXD_WAIT(2 * PER_TILE + 4)  // tile 0 has landed
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        read_a(0, baseSA + tile_off(A_SLAB, 0, 0), F, 0, i);
        read_b(0, baseSB + tile_off(B_SLAB, 0, 0), F, 0, i);
    }
    keep_scales(F, std::integral_constant<int, 0>{});

    // K tile kt (stage kt % 4): a quarter of the wave's 64 MFMAs at a time, halves of A against halves of B, each half overwritten
    // as soon as its last quarter is done.  Of B the half that the tile before ended without comes first (P, then Q):
    //     A0 x P   while Q is read             A0 x Q   while A1 is read
    //     wait for this wave's loads of tile kt + 1 (two and a half tiles old; those of the two tiles behind it stay in flight), ONE
    //     barrier, which also says that every wave has read all of tile kt's stage
    //     A1 x Q   while A0 of kt + 1 is read  A1 x P   while Q of kt + 1 is read, the next tile's P
    // In the first half B's codes and the scales of tile kt + 3 are requested (into the stage that tile kt - 1 left at its barrier), in the
    // second A's codes of tile kt + 4.
    // A wave has its SIMD to itself and issues an instruction every 8 cycles or so; a MFMA takes 16.  So what bounds a K tile (1160 cycles, 1024 of them its
    // MFMAs, at 1.9 to 2.1 GHz by their power), is the number of instructions beyond one per MFMA: stages and with them all LDS addresses are constants (four tiles a trip),
    // pointers advance in scalar registers, the load's destination is one addition, and one LDS read, load or destination follows each MFMA
    // (scheduling fences pin that order).  4096 x 4096 x 16384: 195 instructions a K tile 125.2 us, 135 111.3;
    // 4096 x 11008 x 4096 100.0 and 88.0.
    // Every tile runs the same code: past the end the loads become one-request fillers (lane
    // offsets zero, the codes' from their own operand's first tile, landing in the free stage) that keep the counted wait exact, and
    // the barrier / reads of the tile after the last one are harmless.
    int kt = 0;
    auto tile = [&](auto stage) {
        constexpr int ST = decltype(stage)::value, BEFORE = (ST + 3) & 3, NEXT = (ST + 1) & 3, Pb = ST & 1, Qb = Pb ^ 1;
        if (kt + 4 >= nkt) {
            asm volatile("");
            A.past_end();
            if (kt + 3 >= nkt) {
                asm volatile("");
                B.past_end();
                slab_voff = 0;
                slab_ptr = A.tile;
                slab_step = 0;
            }
        }
        const uint8_t *sa = baseSA + tile_off(A_SLAB, kt, ST), *sb = baseSB + tile_off(B_SLAB, kt, ST);
        const int Gn = (kt >> 2) + 1, part = kt & 1;
        const bool real = GROUPS && (kt & 3) < 2 && 4 * Gn < nkt && !(part ? B_SLAB : A_SLAB);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 32; ++j) {
            mma(F, there_and_back(j).x, 4 * (j < 16 ? Pb : Qb) + there_and_back(j).y);
            __builtin_amdgcn_sched_barrier(0);
            const int q = j & 15, i = q % 3 != 2 && q < 12 ? q / 3 * 2 + q % 3 : -1;  // reads behind MFMAs 0, 1, 3, 4, 6, 7, 9, 10 of a quarter
            if (i >= 0 && j < 16) read_b(ST, sb, F, Qb, i);
            if (i >= 0 && j >= 16) read_a(ST, sa, F, 1, i);
            // the loads' two parts behind the others: B's codes, a scale slab, a scale group
            if (j == 2) NVFP4_MXD_DST_B(BEFORE, 0)
            if (j == 5) NVFP4_MXD_LOAD_B(0)
            if (j == 8) NVFP4_MXD_DST_B(BEFORE, 1)
            if (j == 11) NVFP4_MXD_LOAD_B(1)
            if (j == 12) NVFP4_MXD_DST_B(BEFORE, 2)
            if (j == 13) NVFP4_MXD_LOAD_B(2)
            if (j == 14) NVFP4_MXD_DST_B(BEFORE, 3)
            if (j == 15) NVFP4_MXD_LOAD_B(3)
            if (SLABS && j == 18) NVFP4_MXD_DST(slab_dst, BEFORE * 1024)
            if (SLABS && j == 21) NVFP4_MXD_LOAD(slab_voff, slab_ptr, 0)
            if (GROUPS && j == 24) group_dst(Gn, part, real);
            if (GROUPS && j == 27) group_load(Gn, part, real);
            if (j == 28) B.advance();
            if (SLABS && j == 29) slab_ptr += slab_step;
            __builtin_amdgcn_sched_barrier(0);
        }
        NVFP4_MXD_WAIT(2 * PER_TILE)
        __syncthreads();
        sa = baseSA + tile_off(A_SLAB, kt + 1, NEXT);
        sb = baseSB + tile_off(B_SLAB, kt + 1, NEXT);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 32; ++j) {
            mma(F, 4 + there_and_back(j).x, 4 * (j < 16 ? Qb : Pb) + there_and_back(j).y);
            __builtin_amdgcn_sched_barrier(0);
            const int q = j & 15, i = q % 3 != 2 && q < 12 ? q / 3 * 2 + q % 3 : -1;
            if (i >= 0 && j < 16) read_a(NEXT, sa, F, 0, i);
            if (i >= 0 && j >= 16) read_b(NEXT, sb, F, Qb, i);
            if (j == 2) NVFP4_MXD_DST_A(ST, 0)
            if (j == 5) NVFP4_MXD_LOAD_A(0)
            if (j == 8) NVFP4_MXD_DST_A(ST, 1)
            if (j == 11) NVFP4_MXD_LOAD_A(1)
            if (j == 18) NVFP4_MXD_DST_A(ST, 2)
            if (j == 21) NVFP4_MXD_LOAD_A(2)
            if (j == 24) NVFP4_MXD_DST_A(ST, 3)
            if (j == 27) NVFP4_MXD_LOAD_A(3)
            if (j == 28) A.advance();
            __builtin_amdgcn_sched_barrier(0);
        }
        keep_scales(F, std::integral_constant<int, Qb>{});
        ++kt;
    };
    while (kt + 4 <= nkt) {
        tile(std::integral_constant<int, 0>{});
        tile(std::integral_constant<int, 1>{});
        tile(std::integral_constant<int, 2>{});
        tile(std::integral_constant<int, 3>{});
    }
    if (kt < nkt) {
        tile(std::integral_constant<int, 0>{});
        if (kt < nkt) {
            tile(std::integral_constant<int, 1>{});
            if (kt < nkt) tile(std::integral_constant<int, 2>{});
        }
    }
#undef NVFP4_MXD_WAIT
#undef NVFP4_MXD_HIDE
#undef NVFP4_MXD_DST
#undef NVFP4_MXD_LOAD
#undef NVFP4_MXD_DST_A
#undef NVFP4_MXD_DST_B
#undef NVFP4_MXD_LOAD_A
#undef NVFP4_MXD_LOAD_B

    // every load of every wave has landed and every fragment has been read: stage 0 is free for
    // the epilogue's line buffers
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    asm volatile("s_nop 15" ::: "memory");
#pragma unroll
    for (int a = 0; a < FA / 2; ++a)
#pragma unroll
        for (int b = 0; b < 2 * FB; ++b) asm volatile("" : "+a"(acc[a][b]));
    constexpr int PIECE = 32 * 32 * TB * (OUT_DT == NVFP4_F32 ? 4 : 2);  // of the epilogue, per wave
    store_lines<OUT_DT, FB>(P, acc, m0 + (wave_s >> 1) * 128, n0 + (wave_s & 1) * 128, lds + wave_s * PIECE, lane);
}

// ---------------------------------------------------------------------------------------------
// Tile kernel for the products the kernel above does not serve well: any K that is a multiple of 32, any operand layout, outputs
// that 256 x 256 tiles cannot spread over the 256 CUs.  WM x WN waves of TA x TB MFMA tiles each; built as 128 x 128 (2 x 2 waves
// of 2 x 2), 256 x 128 (2 x 2 of 4 x 2) and 256 x 256 (2 x 4 of 4 x 2), so that two waves share a SIMD and cover each other's
// waits (two workgroups per CU, or one of eight waves).
// What bounds it: LDS reads, (TA + TB) / (TA TB) KB per MFMA, i.e. 1 KB (128 x 128) or 3/4 KB against the 1 KB the LDS delivers
// per 32-cycle MFMA and SIMD.
// Pipeline: three LDS stages of K = 128; the direct loads of tile kt + 2 are requested when tile kt starts and waited for
// (counted) in the middle of tile kt + 1; ONE barrier per tile; step 1's fragments are read under step 0's MFMAs and the next
// tile's first ones under step 1's.
// Scales: E8M0 bytes of a row-major ragged operand start at any byte, which a direct load cannot fetch, and one request per
// row and K tile would cost the vector L1 as much as the codes: so a thread loads 16 bytes of its row = four K tiles at once
// into registers (slabs: four dwords) and stores one dword per K tile into that tile's stage.
// Measured (us; the register-staged 256 x 256 kernel that served a ragged K before -> this one): 4096 x 4128 x 4896 287 -> 84,
// 1056 x 2080 x 2784 75 -> 16.6, 8480 x 9440 x 640 (whole K tiles, ragged edges) 100 -> 63.
namespace mxt {
constexpr int KT = 128, ROWB = 64, NS = 3;
template <int WM, int WN, int TA, int TB>
struct Geom {
    static constexpr int BM = 32 * TA * WM, BN = 32 * TB * WN, ROWS = BM + BN, NT = 64 * WM * WN;
    static constexpr int STAGE = ROWS * ROWB + ROWS * 4;  // codes, then one dword (four E8M0 bytes) per row
    static constexpr int LDS = NS * STAGE > NT * 128 ? NS * STAGE : NT * 128;
};
}  // namespace mxt

template <int OUT_DT, int WM, int WN, int TA, int TB>
__global__ __launch_bounds__(64 * WM * WN, 2) void gemm_nt_mxfp4_tile_kernel(TileArgs P)
{
    using namespace mxt;
    using G = Geom<WM, WN, TA, TB>;
    constexpr int BM = G::BM, BN = G::BN, ROWS = G::ROWS, NT = G::NT, NW = WM * WN;
    constexpr int CA = BM / 16 / NW, CB = BN / 16 / NW;  // direct-to-LDS instructions per wave and K tile (16 rows each)
    constexpr int PW = CA + CB;
    constexpr int NSR = (ROWS + NT - 1) / NT;            // scale rows per thread
    static_assert(BM % (16 * NW) == 0 && BN % (16 * NW) == 0, "whole instructions per wave");
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int r = lane & 31, g = lane >> 5;
    const int ntx = (int)((P.N + BN - 1) / BN), nty = (int)((P.M + BM - 1) / BM);
    int ty, tx;
    tile_coords((int)blockIdx.x, ntx, nty, ty, tx);
    const int64_t m0 = (int64_t)ty * BM, n0 = (int64_t)tx * BN;
    const int64_t Kb = P.K >> 1, Ks = P.K >> 5;
    const int nkt = (int)((P.K + KT - 1) / KT);
    const int rem = (int)(P.K - (int64_t)(nkt - 1) * KT);
    const int ktail = rem < KT ? nkt - 1 : -1;  // the K tile that is not whole

    float16v_t acc[TA][TB];
#pragma unroll
    for (int a = 0; a < TA; ++a)
#pragma unroll
        for (int b = 0; b < TB; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.0f;

    // ---- codes: addresses as in the kernels above
    const int ch = (lane & 3) ^ ((lane >> 4) & 3);
    uint32_t offA[CA], offB[CB];
#pragma unroll
    for (int u = 0; u < CA; ++u) {
        const int row = (wave * CA + u) * 16 + (lane >> 2);
        const int64_t lr = m0 + row < P.M ? row : P.M - 1 - m0;
        offA[u] = P.a_slab ? (uint32_t)(slab_row((int)(m0 & 255) + row) * 64 + ch * 16) : (uint32_t)(lr * Kb + ch * 16);
    }
#pragma unroll
    for (int u = 0; u < CB; ++u) {
        const int row = (wave * CB + u) * 16 + (lane >> 2);
        const int64_t lr = n0 + row < P.N ? row : P.N - 1 - n0;
        offB[u] = P.b_slab ? (uint32_t)(slab_row((int)(n0 & 255) + row) * 64 + ch * 16) : (uint32_t)(lr * Kb + ch * 16);
    }
    const uint8_t *const baseA = P.a_slab ? P.A_codes + (m0 >> 8) * nkt * SLAB_CODE_BYTES : P.A_codes + m0 * Kb;
    const uint8_t *const baseB = P.b_slab ? P.B_codes + (n0 >> 8) * nkt * SLAB_CODE_BYTES : P.B_codes + n0 * Kb;
    const int64_t stepA = P.a_slab ? SLAB_CODE_BYTES : ROWB, stepB = P.b_slab ? SLAB_CODE_BYTES : ROWB;
    typedef __attribute__((address_space(3))) void *lds_ptr_t;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr_t)lds;
    auto uniform_ptr = [](const uint8_t *p) -> const uint8_t * {
        const uint64_t v = reinterpret_cast<uint64_t>(p);
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
        return reinterpret_cast<const uint8_t *>(((uint64_t)hi << 32) | lo);
    };
    auto dma16 = [&](uint32_t lds_addr, uint32_t voff, const uint8_t *base) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds_addr), "v"(voff), "s"(base) : "memory", "m0");
    };
    auto dma_codes = [&](int kt, uint32_t stage) {
        const uint8_t *const pa = uniform_ptr(baseA + kt * stepA), *const pb = uniform_ptr(baseB + kt * stepB);
        const uint32_t dst = __builtin_amdgcn_readfirstlane(lds0 + stage);
        const uint32_t back = kt == ktail && ch * 32 >= rem ? (uint32_t)ch * 16 : 0u;  // (a missing chunk: the tile's first)
#pragma unroll
        for (int u = 0; u < CA; ++u) dma16(dst + (wave * CA + u) * 1024, offA[u] - back, pa);
#pragma unroll
        for (int u = 0; u < CB; ++u) dma16(dst + BM * ROWB + (wave * CB + u) * 1024, offB[u] - back, pb);
    };
    // ---- scales: four K tiles of a row at a time, 16 bytes (row-major, any alignment) or one dword per slab
    static_assert(BM % 64 == 0 && BN % 64 == 0, "a wave's scale rows belong to one operand");
    const uint8_t *sptr[NSR];
#pragma unroll
    for (int i = 0; i < NSR; ++i) {
        const int wrow = 64 * wave + NT * i, row = wrow + lane;
        const bool isA = wrow < BM;
        const int64_t base = isA ? m0 : n0, rows = isA ? P.M : P.N;
        const int lrow = isA ? row : row - BM;
        const uint8_t *const s = isA ? P.A_scales : P.B_scales;
        sptr[i] = (isA ? P.a_slab : P.b_slab) ? s + (base >> 8) * nkt * SLAB_MX_SCALE_BYTES + slab_row(((int)(base & 255) + lrow) & 255) * 4
                                              : s + (base + lrow < rows ? base + lrow : rows - 1) * Ks;
    }
    struct Group {
        uint32_t w[NSR][4];
    };
    auto load_group = [&](int grp, Group &q) {
#pragma unroll
        for (int i = 0; i < NSR; ++i) {
            const int wrow = 64 * wave + NT * i;
            if (wrow >= ROWS) continue;
            const bool slab = wrow < BM ? P.a_slab : P.b_slab;
            if (Ks < 4) {
                // (less than one K tile: a row's one to three bytes)
                uint32_t v = 0;
                for (int t = 0; t < (int)Ks; ++t) v |= (uint32_t)sptr[i][t] << (8 * t);
#pragma unroll
                for (int t = 0; t < 4; ++t) q.w[i][t] = v;
            } else if (!slab && 16 * grp + 16 <= Ks) {
                __builtin_memcpy(q.w[i], sptr[i] + 16 * grp, 16);
            } else {
                // a dword per K tile; the last one of a row is read so that it ends with the row
                const int step = slab ? (int)SLAB_MX_SCALE_BYTES : 4, last = slab ? (nkt - 1) * step : (int)Ks - 4;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int want = (4 * grp + t) * step, at = want < last ? want : last;
                    uint32_t v;
                    __builtin_memcpy(&v, sptr[i] + at, 4);
                    q.w[i][t] = v >> (8 * ((want - at) & 3));
                }
            }
        }
    };
    auto stash = [&](uint32_t stage, const Group &q, int t) {
        uint32_t *const s = reinterpret_cast<uint32_t *>(lds + stage + ROWS * ROWB);
#pragma unroll
        for (int i = 0; i < NSR; ++i)
            if (64 * wave + NT * i < ROWS) s[tid + NT * i] = q.w[i][t];
    };

    // ---- LDS -> registers
    struct Frags {
        uint4 a[TA], b[TB];
    };
    struct Scales {
        uint32_t a[TA], b[TB];
    };
    const int sw = (r >> 2) & 3;
    const int rdA = (wm * 32 * TA + r) * ROWB, rdB = (BM + wn * 32 * TB + r) * ROWB;
    const int rdS = ROWS * ROWB + (wm * 32 * TA + r) * 4, rdT = ROWS * ROWB + (BM + wn * 32 * TB + r) * 4;
    auto load_frags = [&](uint32_t stage, int s, Frags &F) {
        const uint8_t *p = lds + stage + (((2 * g + s) ^ sw) << 4);
#pragma unroll
        for (int b = 0; b < TB; ++b) F.b[b] = *reinterpret_cast<const uint4 *>(p + rdB + 32 * b * ROWB);
#pragma unroll
        for (int a = 0; a < TA; ++a) F.a[a] = *reinterpret_cast<const uint4 *>(p + rdA + 32 * a * ROWB);
    };
    auto load_scales = [&](uint32_t stage, Scales &S) {
#pragma unroll
        for (int b = 0; b < TB; ++b) S.b[b] = *reinterpret_cast<const uint32_t *>(lds + stage + rdT + 128 * b);
#pragma unroll
        for (int a = 0; a < TA; ++a) S.a[a] = *reinterpret_cast<const uint32_t *>(lds + stage + rdS + 128 * a);
    };
    auto shift = [&](Scales &S) {
#pragma unroll
        for (int a = 0; a < TA; ++a) S.a[a] >>= 16 * g;
#pragma unroll
        for (int b = 0; b < TB; ++b) S.b[b] >>= 16 * g;
    };
    auto zero_tail = [&](Frags &F, int s) {
        if ((2 * g + s) * 32 >= rem) {
#pragma unroll
            for (int a = 0; a < TA; ++a) F.a[a] = make_uint4(0, 0, 0, 0);
        }
    };
#define NVFP4_MXT_MMA(F, S, s)                                                                                     \
    _Pragma("unroll") for (int a = 0; a < TA; ++a) _Pragma("unroll") for (int b = 0; b < TB; ++b)                  \
    {                                                                                                              \
        const int8v_t va = {(int)F.a[a].x, (int)F.a[a].y, (int)F.a[a].z, (int)F.a[a].w, 0, 0, 0, 0};               \
        const int8v_t vb = {(int)F.b[b].x, (int)F.b[b].y, (int)F.b[b].z, (int)F.b[b].w, 0, 0, 0, 0};               \
        acc[a][b] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(vb, va, acc[a][b], 4, 4, s, (int)S.b[b], s, (int)S.a[a]); \
    }

    Frags F0, F1;
    Scales S, R;
    Group gc, gn;
    uint32_t s_cur = 0, s_nxt = G::STAGE, s_new = 2 * G::STAGE;
    load_group(0, gc);
    gn = gc;
    dma_codes(0, s_cur);
    stash(s_cur, gc, 0);
    if (nkt > 1) dma_codes(1, s_nxt);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    load_frags(s_cur, 0, F0);
    load_scales(s_cur, R);

    // K tile kt (kt % 4 == j): on entry F0 and R hold the first fragments and the scales of the tile, the direct loads of tile
    // kt + 1 are in flight.
    auto tile = [&](int kt, auto jc) {
        constexpr int j = decltype(jc)::value;
        if (kt + 1 < nkt) stash(s_nxt, j == 3 ? gn : gc, (j + 1) & 3);
        if (j == 3) gc = gn;
        const bool more = kt + 2 < nkt;
        if (more) dma_codes(kt + 2, s_new);
        S = R;
        shift(S);
        if (kt == ktail) zero_tail(F0, 0);
        __builtin_amdgcn_sched_barrier(0);
        load_frags(s_cur, 1, F1);
        NVFP4_MXT_MMA(F0, S, 0)
#pragma unroll
        for (int i = 0; i < TA + TB; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (more)
            asm volatile("s_waitcnt vmcnt(%0)" : : "n"(PW) : "memory");
        else
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (j == 0 && 4 * (kt / 4 + 1) < nkt) load_group(kt / 4 + 1, gn);
        if (kt == ktail) zero_tail(F1, 1);
        __builtin_amdgcn_sched_barrier(0);
        load_frags(s_nxt, 0, F0);
        load_scales(s_nxt, R);
        NVFP4_MXT_MMA(F1, S, 1)
#pragma unroll
        for (int i = 0; i < TA + TB; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        const uint32_t t = s_cur;
        s_cur = s_nxt;
        s_nxt = s_new;
        s_new = t;
    };
    for (int kt = 0;; kt += 4) {
        tile(kt, std::integral_constant<int, 0>{});
        if (kt + 1 >= nkt) break;
        tile(kt + 1, std::integral_constant<int, 1>{});
        if (kt + 2 >= nkt) break;
        tile(kt + 2, std::integral_constant<int, 2>{});
        if (kt + 3 >= nkt) break;
        tile(kt + 3, std::integral_constant<int, 3>{});
        if (kt + 4 >= nkt) break;
    }
#undef NVFP4_MXT_MMA

    __syncthreads();
    static_assert(NW * 32 * 32 * TB * 4 <= G::LDS, "the epilogue's pieces");
    store_lines<OUT_DT, TB>(P, acc, m0 + wm * 32 * TA, n0 + wn * 32 * TB, lds + wave * (32 * 32 * TB * (OUT_DT == NVFP4_F32 ? 4 : 2)), lane);
}

template <int WM, int WN, int TA, int TB>
static void launch_mx_tile(const TileArgs &P, int out_dt, hipStream_t st)
{
    using G = mxt::Geom<WM, WN, TA, TB>;
    const unsigned ntiles = (unsigned)(((P.N + G::BN - 1) / G::BN) * ((P.M + G::BM - 1) / G::BM));
    if (out_dt == NVFP4_F32) {
        auto k = gemm_nt_mxfp4_tile_kernel<NVFP4_F32, WM, WN, TA, TB>;
        static bool once = ((void)hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, G::LDS), true);
        (void)once;
        hipLaunchKernelGGL(k, dim3(ntiles), dim3(G::NT), G::LDS, st, P);
    } else {
        auto k = gemm_nt_mxfp4_tile_kernel<NVFP4_BF16, WM, WN, TA, TB>;
        static bool once = ((void)hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, G::LDS), true);
        (void)once;
        hipLaunchKernelGGL(k, dim3(ntiles), dim3(G::NT), G::LDS, st, P);
    }
}

template <int OUT_DT, bool A_SLAB, bool B_SLAB>
static void launch_mx_dma_as(const TileArgs &P, hipStream_t st)
{
    const unsigned ntiles = (unsigned)(((P.N + mx::BN - 1) / mx::BN) * ((P.M + mx::BM - 1) / mx::BM));
    auto k = gemm_nt_mxfp4_dma_kernel<OUT_DT, A_SLAB, B_SLAB>;
    static bool once = ((void)hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, mxd::LDS_BYTES), true);
    (void)once;
    hipLaunchKernelGGL(k, dim3(ntiles), dim3(256), mxd::LDS_BYTES, st, P);
}

template <int OUT_DT>
static void launch_mx_dma_out(const TileArgs &P, hipStream_t st)
{
    if (P.a_slab && P.b_slab) launch_mx_dma_as<OUT_DT, true, true>(P, st);
    else if (P.a_slab) launch_mx_dma_as<OUT_DT, true, false>(P, st);
    else if (P.b_slab) launch_mx_dma_as<OUT_DT, false, true>(P, st);
    else launch_mx_dma_as<OUT_DT, false, false>(P, st);
}

static void launch_mx_dma(const TileArgs &P, int out_dt, hipStream_t st)
{
    if (out_dt == NVFP4_F32)
        launch_mx_dma_out<NVFP4_F32>(P, st);
    else
        launch_mx_dma_out<NVFP4_BF16>(P, st);
}

template <int B>
static void launch_rescale(const TileArgs &P, int out_dt, hipStream_t st)
{
    const unsigned ntiles = (unsigned)(((P.N + mx::BN - 1) / mx::BN) * ((P.M + mx::BM - 1) / mx::BM));
    if (out_dt == NVFP4_F32) {
        auto k = gemm_nt_fp4_rescale_kernel<NVFP4_F32, B>;
        static bool once = ((void)hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, mxr::LDS_BYTES), true);
        (void)once;
        hipLaunchKernelGGL(k, dim3(ntiles), dim3(256), mxr::LDS_BYTES, st, P);
    } else {
        auto k = gemm_nt_fp4_rescale_kernel<NVFP4_BF16, B>;
        static bool once = ((void)hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, mxr::LDS_BYTES), true);
        (void)once;
        hipLaunchKernelGGL(k, dim3(ntiles), dim3(256), mxr::LDS_BYTES, st, P);
    }
}

// E4M3 scales at blocks of 64 / 128 on the FP4 matrix instruction with binary32 rescaling of the block sums.
bool fp4_rescale_gemm_applies(int64_t K, int block, const GemmArgs &P)
{
    const uintptr_t codes = reinterpret_cast<uintptr_t>(P.A_codes) | reinterpret_cast<uintptr_t>(P.B_codes);
    return (block == 64 || block == 128) && K % 128 == 0 && (codes & 15) == 0 && !P.a_slab && !P.b_slab;
}

hipError_t launch_gemm_fp4_rescale(const TileArgs &P, int block, int out_dt, hipStream_t st)
{
    if (block == 64)
        launch_rescale<64>(P, out_dt, st);
    else
        launch_rescale<128>(P, out_dt, st);
    return hipGetLastError();
}

// The contractions whose operands come as slabs: those that the four-stage direct-to-LDS kernel, which they were made for, can walk
// (with 16-byte aligned codes and 4-byte aligned scales).  The other tiles read them too.
bool mxfp4_gemm_takes_slabs(int64_t K)
{
    // lane offsets of the direct-to-LDS loads are 32-bit and relative to the tile's first row
    const bool offsets_fit = (K >> 1) * 256 < ((int64_t)1 << 31);
    return K % 128 == 0 && K >= 512 && offsets_fit;
}

hipError_t launch_gemm_mxfp4(const TileArgs &P, GemmTile tile, int out_dt, hipStream_t st)
{
    const uintptr_t codes = reinterpret_cast<uintptr_t>(P.A_codes) | reinterpret_cast<uintptr_t>(P.B_codes);
    const uintptr_t scales = reinterpret_cast<uintptr_t>(P.A_scales) | reinterpret_cast<uintptr_t>(P.B_scales);
    if (tile == TILE_256x256 && mxfp4_gemm_takes_slabs(P.K) && (codes & 15) == 0 && (scales & 3) == 0)
        launch_mx_dma(P, out_dt, st);
    else if (tile == TILE_256x256)
        launch_mx_tile<2, 4, 4, 2>(P, out_dt, st);
    else if (tile == TILE_256x128)
        launch_mx_tile<2, 2, 4, 2>(P, out_dt, st);
    else
        launch_mx_tile<2, 2, 2, 2>(P, out_dt, st);
    return hipGetLastError();
}

}  // namespace nvfp4
