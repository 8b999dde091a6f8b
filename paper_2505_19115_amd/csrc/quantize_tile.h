// Device code that the quantizer kernels share: loads and stores, block maxima, scales, the converts, the row-blocked tile.
#pragma once
#include "kernels.h"
#include "nvfp4_math.h"

namespace nvfp4 {

// ------------------------------------------------------------------ small device helpers

template <int CTRL>
__device__ __forceinline__ float dpp_max(float a)
{
    // a >= 0: unsigned order of the bit patterns is the float order
    int o = __builtin_amdgcn_update_dpp(0, (int)f2u(a), CTRL, 0xF, 0xF, false);
    uint32_t ou = (uint32_t)o;
    return u2f(umax(f2u(a), ou));
}

// Maximum over groups of L adjacent lanes (L = 1, 2, 4, 8, 16; groups aligned to L).
template <int L>
__device__ __forceinline__ float group_max(float a)
{
    if (L >= 2) a = dpp_max<0xB1>(a);   // quad_perm [1,0,3,2]  : lane ^ 1
    if (L >= 4) a = dpp_max<0x4E>(a);   // quad_perm [2,3,0,1]  : lane ^ 2
    if (L >= 8) a = dpp_max<0x141>(a);  // row_half_mirror      : swaps the two quads of 8 lanes
    if (L >= 16) a = dpp_max<0x140>(a); // row_mirror           : swaps the two halves of 16 lanes
    return a;
}

// Maximum of the two lanes D apart (lane ^ D; D = 8, 16 or 32), a >= 0.
template <int D>
__device__ __forceinline__ float lane_pair_max(float a)
{
    static_assert(D == 8 || D == 16 || D == 32, "");
    if constexpr (D == 8) return dpp_max<0x128>(a);  // row_ror:8
    const uint32_t u = f2u(a);
    if constexpr (D == 16) {
        const auto p = __builtin_amdgcn_permlane16_swap(u, u, false, false);
        return u2f(umax(p[0], p[1]));
    } else {
        const auto p = __builtin_amdgcn_permlane32_swap(u, u, false, false);
        return u2f(umax(p[0], p[1]));
    }
}

// The quantizer streams: every input byte is read once and every output byte written once, so
// loads and stores carry the nontemporal hint (measured on gfx950 with the quantizer's 16 B in /
// 4 B out shape: 6.1-6.2 TB/s with the hint against 5.4 TB/s without).  STREAM = false keeps a
// tensor in the last-level cache for a second pass.
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
template <bool STREAM>
__device__ __forceinline__ uint4 load16(const void *p)
{
    if (STREAM) {
        const u32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(p));
        return make_uint4(v.x, v.y, v.z, v.w);
    }
    return *reinterpret_cast<const uint4 *>(p);
}
__device__ __forceinline__ void store4_stream(void *p, uint32_t v) { __builtin_nontemporal_store(v, reinterpret_cast<uint32_t *>(p)); }
__device__ __forceinline__ void store8_stream(void *p, uint32_t a, uint32_t b)
{
    const u32x2_t v = {a, b};
    __builtin_nontemporal_store(v, reinterpret_cast<u32x2_t *>(p));
}

template <int DT>
struct Chunk;  // 8 consecutive elements as loaded from memory

template <>
struct Chunk<NVFP4_BF16> {
    uint4 raw;
    template <bool STREAM = true>
    __device__ __forceinline__ void load(const void *x, int64_t off)
    {
        raw = load16<STREAM>(reinterpret_cast<const uint16_t *>(x) + off);
    }
    // (from any element on)
    __device__ __forceinline__ void load_unaligned(const void *x, int64_t off) { __builtin_memcpy(&raw, reinterpret_cast<const uint16_t *>(x) + off, 16); }
    __device__ __forceinline__ void load_partial(const void *x, int64_t off, int n)
    {
        const uint16_t *p = reinterpret_cast<const uint16_t *>(x) + off;
        uint32_t w[4] = {0, 0, 0, 0};
        for (int t = 0; t < n; ++t) w[t >> 1] |= (uint32_t)p[t] << (16 * (t & 1));
        raw = make_uint4(w[0], w[1], w[2], w[3]);
    }
    __device__ __forceinline__ void zero() { raw = make_uint4(0, 0, 0, 0); }
    __device__ __forceinline__ void store(void *x, int64_t off) const
    {
        *reinterpret_cast<uint4 *>(reinterpret_cast<uint16_t *>(x) + off) = raw;
    }
    // 8 binary32 values rounded to bf16 (nearest even) and packed
    __device__ __forceinline__ void set(const float (&f)[8])
    {
        typedef float f2_t __attribute__((ext_vector_type(2)));
        typedef __bf16 b2_t __attribute__((ext_vector_type(2)));
        uint32_t w[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const f2_t p = {f[2 * t], f[2 * t + 1]};
            const b2_t b = __builtin_convertvector(p, b2_t);
            w[t] = __builtin_bit_cast(uint32_t, b);
        }
        raw = make_uint4(w[0], w[1], w[2], w[3]);
    }
    __device__ __forceinline__ void launder() { asm volatile("" : "+v"(raw.x), "+v"(raw.y), "+v"(raw.z), "+v"(raw.w)); }
    // elements 2i (low half) and 2i + 1 (high half) as stored
    __device__ __forceinline__ uint32_t word(int i) const { return i == 0 ? raw.x : i == 1 ? raw.y : i == 2 ? raw.z : raw.w; }
    __device__ __forceinline__ float get(int t) const
    {
        uint32_t w = t < 2 ? raw.x : t < 4 ? raw.y : t < 6 ? raw.z : raw.w;
        return (t & 1) ? u2f(w & 0xFFFF0000u) : u2f(w << 16);
    }
};

template <>
struct Chunk<NVFP4_F32> {
    float4 lo, hi;
    template <bool STREAM = true>
    __device__ __forceinline__ void load(const void *x, int64_t off)
    {
        const float *p = reinterpret_cast<const float *>(x) + off;
        const uint4 a = load16<STREAM>(p), b = load16<STREAM>(p + 4);
        lo = make_float4(u2f(a.x), u2f(a.y), u2f(a.z), u2f(a.w));
        hi = make_float4(u2f(b.x), u2f(b.y), u2f(b.z), u2f(b.w));
    }
    __device__ __forceinline__ void load_unaligned(const void *x, int64_t off)
    {
        const float *p = reinterpret_cast<const float *>(x) + off;
        __builtin_memcpy(&lo, p, 16);
        __builtin_memcpy(&hi, p + 4, 16);
    }
    __device__ __forceinline__ void load_partial(const void *x, int64_t off, int n)
    {
        const float *p = reinterpret_cast<const float *>(x) + off;
        float v[8];
        for (int t = 0; t < 8; ++t) v[t] = t < n ? p[t] : 0.0f;
        lo = make_float4(v[0], v[1], v[2], v[3]);
        hi = make_float4(v[4], v[5], v[6], v[7]);
    }
    __device__ __forceinline__ void zero()
    {
        lo = make_float4(0, 0, 0, 0);
        hi = lo;
    }
    __device__ __forceinline__ void set(const float (&f)[8])
    {
        lo = make_float4(f[0], f[1], f[2], f[3]);
        hi = make_float4(f[4], f[5], f[6], f[7]);
    }
    __device__ __forceinline__ void store(void *x, int64_t off) const
    {
        float *p = reinterpret_cast<float *>(x) + off;
        *reinterpret_cast<float4 *>(p) = lo;
        *reinterpret_cast<float4 *>(p + 4) = hi;
    }
    __device__ __forceinline__ void launder() {}
    __device__ __forceinline__ uint32_t word(int) const { return 0; }  // (bf16 chunks only)
    __device__ __forceinline__ float get(int t) const
    {
        switch (t) {
        case 0: return lo.x;
        case 1: return lo.y;
        case 2: return lo.z;
        case 3: return lo.w;
        case 4: return hi.x;
        case 5: return hi.y;
        case 6: return hi.z;
        default: return hi.w;
        }
    }
};

template <int DT>
__device__ __forceinline__ float chunk_amax(const Chunk<DT> &c)
{
    float a = 0.0f;
#pragma unroll
    for (int t = 0; t < 8; ++t) a = fmaxf(a, fabsf(c.get(t)));
    return a;
}

// The same on a bf16 chunk as stored: magnitudes of finite bf16 values order like their bit patterns, so the
// maximum is taken on packed 16-bit integers, two elements per instruction, and widened once at the end.
typedef uint16_t u16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pk_umax16(uint32_t a, uint32_t b)
{
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2_t, a), __builtin_bit_cast(u16x2_t, b)));
}
// the two halves of a packed maximum as binary32 (even element, odd element)
__device__ __forceinline__ float pk_even(uint32_t m) { return u2f(m << 16); }
__device__ __forceinline__ float pk_odd(uint32_t m) { return u2f(m & 0xFFFF0000u); }
template <int DT>
__device__ __forceinline__ float chunk_amax_packed(const Chunk<DT> &c)
{
    if constexpr (DT == NVFP4_BF16) {
        const uint32_t m = pk_umax16(pk_umax16(c.word(0) & 0x7FFF7FFFu, c.word(1) & 0x7FFF7FFFu),
                                     pk_umax16(c.word(2) & 0x7FFF7FFFu, c.word(3) & 0x7FFF7FFFu));
        return u2f(umax(m << 16, m & 0xFFFF0000u));
    } else {
        return chunk_amax(c);
    }
}

// Per-tensor scale as the kernels see it: none, preset in memory, or the bit pattern of the
// tensor maximum left by the amax kernel.
// With n_partials > 0 the tensor maximum arrives as that many per-workgroup maxima and every
// workgroup (NT threads, all of them must call this) folds them for itself: 2 KB from the L2 per
// workgroup instead of a separate one-workgroup kernel between the maximum pass and the quantizer.
// n_partials < 0: a small dense tensor (SELF_AMAX_BYTES), whose maximum every workgroup takes for itself.
// SELF = false leaves that form out, in kernels that no such tensor reaches: beside a lane tile of 16 rows its loads in flight cost
// the registers of a whole wave per SIMD (129 instead of 126: a columns pass of one tile per workgroup, bf16 SR, over 4096 x 8192 30.1 us instead of 25.8, over
// 8192 x 8192 53.0 instead of 51.6; 4096 x 11008, 1376 tiles, 1.8 rounds of three
// workgroups per CU or 1.3 of four, took 41.9 instead of 43.7).  Binary32 chunks, twice the size, are four at a time, and kernels for E8M0 scales, whose formats have no tensor
// scale, do without; neither changed a time (MXFP4 rows, bf16 SR, 4096 x 11008: 20.8 us both ways).
template <int DT, int NT = 256, bool SELF = true>
__device__ __forceinline__ float resolve_g(const QuantArgs &P)
{
    if (P.g_mode == G_NONE) return 1.0f;
    if (P.g_mode == G_PRESET) {
        float g = *P.g_src;
        return g < tensor_scale_floor() ? tensor_scale_floor() : g;
    }
    const uint32_t *bits = reinterpret_cast<const uint32_t *>(P.g_src);
    if (P.n_partials == 0) return tensor_scale_from_amax(u2f(*bits));
    __shared__ uint32_t fold[NT / 16];
    uint32_t m = 0;
    if (SELF && P.n_partials < 0) {
        constexpr int U = DT == NVFP4_F32 ? 4 : 8;
        const int n = (int)(P.rows * P.cols), nchunk = n >> 3;
        float a = 0.0f;
        for (int base = threadIdx.x; base < nchunk; base += U * NT) {
            Chunk<DT> v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (base + u * NT < nchunk)
                    v[u].template load<false>(P.x, (int64_t)(base + u * NT) * 8);
                else
                    v[u].zero();
            }
#pragma unroll
            for (int u = 0; u < U; ++u) a = fmaxf(a, chunk_amax(v[u]));
        }
        if (threadIdx.x == 0 && (n & 7)) {
            Chunk<DT> t;
            t.load_partial(P.x, (int64_t)nchunk * 8, n & 7);
            a = fmaxf(a, chunk_amax(t));
        }
        m = f2u(a);
    }
    for (int i = threadIdx.x; i < P.n_partials; i += NT) m = umax(m, bits[i]);
    m = f2u(group_max<16>(u2f(m)));
    if ((threadIdx.x & 15) == 0) fold[threadIdx.x >> 4] = m;
    __syncthreads();
#pragma unroll
    for (int t = 0; t < NT / 16; ++t) m = umax(m, fold[t]);
    return tensor_scale_from_amax(u2f(m));
}

// Block scale byte and the multiplier q that maps the block onto the E2M1 range.
// With E4M3 scales q = 0 for a block whose magnitudes are all zero.
// HW: the E4M3 byte and its value come from the gfx950 FP8 converts (OCP E4M3, round to nearest
// even; the input is clamped to 448 first, as in the software encode, so the convert never sees
// an out-of-range value).  Checked against e4m3_encode / e4m3_decode on every non-negative fp32
// up to 512: identical bytes and values.  The software formulation costs ~15 instructions per block.
// With E4M3 scales and a per-tensor g the multiplier q = 1 / (s * g) is a function of the scale byte alone: a
// workgroup evaluates it once for each of the 127 finite bytes (the same multiply and correctly rounded division
// every block would do) and the blocks then look it up, which takes ~12 instructions out of every block's path.
// All threads of the workgroup (128 or more) must call this (it ends in a barrier).  Returns false where no table applies.
__shared__ float qtab[128];
template <int SF, bool HW>
__device__ __forceinline__ bool build_qtab(float g)
{
    if (SF != NVFP4_SCALE_E4M3 || !HW) return false;
    if (threadIdx.x < 128) {
        const uint32_t byte = threadIdx.x;
        const float s = __builtin_amdgcn_cvt_f32_fp8((int)byte, 0);
        const float d = byte == 0 ? 1.0f : s * g;
        const float r = 1.0f / d;
        qtab[byte] = byte == 0 ? 0.0f : r;
    }
    __syncthreads();
    return true;
}

// TAB: look q up in the workgroup's table (build_qtab() must have run) instead of dividing.
template <int SF, bool HW = false, bool TAB = false>
__device__ __forceinline__ uint32_t block_scale(float a, float g, float k, float *q)
{
    if (SF == NVFP4_SCALE_E4M3) {
        float s;
        uint32_t byte;
        if (HW) {
            const float r = a * k;
            const float rc = r < 448.0f ? r : 448.0f;
            byte = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(rc, 0.0f, 0, false) & 0xFFu;
            if (TAB) {
                *q = qtab[byte];
                return byte;
            }
            s = __builtin_amdgcn_cvt_f32_fp8((int)byte, 0);
        } else {
            byte = e4m3_encode(a * k, &s);
        }
        // (no branch around the division: a zero scale byte divides by 1 and is then replaced)
        const bool zero = byte == 0;
        const float d = zero ? 1.0f : s * g;
        const float r = 1.0f / d;
        *q = zero ? 0.0f : r;
        return byte;
    } else {
        // (an all-zero block: byte 0, and its zeros times any finite q are zeros of the same sign)
        return e8m0_encode(a, q);
    }
}

// One element: sign | magnitude code.
template <int RND>
__device__ __forceinline__ uint32_t quant_elem(float x, float q, uint32_t u16)
{
    float m = fabsf(x * q);
    m = m < 6.0f ? m : 6.0f;
    uint32_t mag = RND == NVFP4_RTN ? round_rtn(m) : round_sr(m, u16);
    return mag | ((f2u(x) >> 28) & 8u);
}

// Two adjacent elements -> one byte via the gfx950 convert (RNE, saturating at +-6, sign
// kept on zero), low nibble = first element; the byte replaces byte BYTE of acc, the others stay.
template <int BYTE>
__device__ __forceinline__ uint32_t quant_pair_hw(uint32_t acc, float x0, float x1, float q)
{
    return __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(acc, x0 * q, x1 * q, 1.0f, BYTE);
}

// Stochastic rounding of one element through the gfx950 convert, which takes a pair: the
// element sits in slot SLOT (0: low nibble, random bits seed[31:10]; 1: high nibble, seed[30:9]),
// the other slot holds +0 (never rounded up: code 0).  Byte BYTE of acc is replaced and the
// other bytes kept, so two accumulators (one per slot) are filled and OR-ed.  Saturation at
// +-6 and the sign (also of a zero) are the convert's own.
// Written as inline assembly with the accumulator tied to the destination: the compiler's
// builtin for this instruction does not tie its "old" operand, which loses the other bytes.
template <int SLOT, int BYTE>
__device__ __forceinline__ uint32_t sr_elem_hw(uint32_t acc, float y, uint32_t u16)
{
    typedef float float2_t __attribute__((ext_vector_type(2)));
    const float2_t v = SLOT == 0 ? float2_t{y, 0.0f} : float2_t{0.0f, y};
    const uint32_t seed = SLOT == 0 ? sr_seed_first(u16) : sr_seed_second(u16);
    if (BYTE == 0) asm("v_cvt_scalef32_sr_pk_fp4_f32 %0, %1, %2, 1.0" : "+v"(acc) : "v"(v), "v"(seed));
    if (BYTE == 1) asm("v_cvt_scalef32_sr_pk_fp4_f32 %0, %1, %2, 1.0 op_sel:[0,0,1,0]" : "+v"(acc) : "v"(v), "v"(seed));
    if (BYTE == 2) asm("v_cvt_scalef32_sr_pk_fp4_f32 %0, %1, %2, 1.0 op_sel:[0,0,0,1]" : "+v"(acc) : "v"(v), "v"(seed));
    if (BYTE == 3) asm("v_cvt_scalef32_sr_pk_fp4_f32 %0, %1, %2, 1.0 op_sel:[0,0,1,1]" : "+v"(acc) : "v"(v), "v"(seed));
    return acc;
}

// The same through slot 0 only, with the seed word taken straight from a draw word: nw is the COMPLEMENT of the
// Philox word that holds the element's 16 bits in its low (HALF 0) or high (HALF 1) half, and
// sr_seed_first(u16) = ((~u16 & 0xFFFF) << 16) | 0x8000 becomes one shift-or or one and-or.  An element that
// belongs in the high nibble of its byte is converted into the low nibble of a second accumulator, which the
// caller shifts by 4 once per word.
__device__ __forceinline__ uint32_t sr_seed0(uint32_t nw, int half)
{
    return half ? ((nw & 0xFFFF0000u) | 0x8000u) : ((nw << 16) | 0x8000u);
}
template <int BYTE>
__device__ __forceinline__ uint32_t sr_elem0(uint32_t acc, float y, uint32_t seed)
{
    typedef float float2_t __attribute__((ext_vector_type(2)));
    const float2_t v = float2_t{y, 0.0f};
    if (BYTE == 0) asm("v_cvt_scalef32_sr_pk_fp4_f32 %0, %1, %2, 1.0" : "+v"(acc) : "v"(v), "v"(seed));
    if (BYTE == 1) asm("v_cvt_scalef32_sr_pk_fp4_f32 %0, %1, %2, 1.0 op_sel:[0,0,1,0]" : "+v"(acc) : "v"(v), "v"(seed));
    if (BYTE == 2) asm("v_cvt_scalef32_sr_pk_fp4_f32 %0, %1, %2, 1.0 op_sel:[0,0,0,1]" : "+v"(acc) : "v"(v), "v"(seed));
    if (BYTE == 3) asm("v_cvt_scalef32_sr_pk_fp4_f32 %0, %1, %2, 1.0 op_sel:[0,0,1,1]" : "+v"(acc) : "v"(v), "v"(seed));
    return acc;
}
// the same with the convert's scale operand (1: none)
template <int BYTE>
__device__ __forceinline__ uint32_t sr_scaled(uint32_t acc, float y, uint32_t seed, float sc)
{
    typedef float float2_t __attribute__((ext_vector_type(2)));
    const float2_t v = float2_t{y, 0.0f};
    if (BYTE == 0) asm("v_cvt_scalef32_sr_pk_fp4_f32 %0, %1, %2, %3" : "+v"(acc) : "v"(v), "v"(seed), "v"(sc));
    if (BYTE == 1) asm("v_cvt_scalef32_sr_pk_fp4_f32 %0, %1, %2, %3 op_sel:[0,0,1,0]" : "+v"(acc) : "v"(v), "v"(seed), "v"(sc));
    if (BYTE == 2) asm("v_cvt_scalef32_sr_pk_fp4_f32 %0, %1, %2, %3 op_sel:[0,0,0,1]" : "+v"(acc) : "v"(v), "v"(seed), "v"(sc));
    if (BYTE == 3) asm("v_cvt_scalef32_sr_pk_fp4_f32 %0, %1, %2, %3 op_sel:[0,0,1,1]" : "+v"(acc) : "v"(v), "v"(seed), "v"(sc));
    return acc;
}
// 8 consecutive elements of a row (chunk v, multiplier q, their draw d) -> 8 codes in one word
template <int DT>
__device__ __forceinline__ uint32_t sr_chunk_hw(const Chunk<DT> &v, float q, const u32x4 &d)
{
    const uint32_t n0 = ~d.x, n1 = ~d.y, n2 = ~d.z, n3 = ~d.w;
    uint32_t lo = 0, hi = 0;
    lo = sr_elem0<0>(lo, v.get(0) * q, sr_seed0(n0, 0));
    hi = sr_elem0<0>(hi, v.get(1) * q, sr_seed0(n0, 1));
    lo = sr_elem0<1>(lo, v.get(2) * q, sr_seed0(n1, 0));
    hi = sr_elem0<1>(hi, v.get(3) * q, sr_seed0(n1, 1));
    lo = sr_elem0<2>(lo, v.get(4) * q, sr_seed0(n2, 0));
    hi = sr_elem0<2>(hi, v.get(5) * q, sr_seed0(n2, 1));
    lo = sr_elem0<3>(lo, v.get(6) * q, sr_seed0(n3, 0));
    hi = sr_elem0<3>(hi, v.get(7) * q, sr_seed0(n3, 1));
    return lo | (hi << 4);
}

// ---- MXFP4 through the converts' own scale operand.
// The gfx950 FP4 converts divide the source by a power of two taken from the exponent field of a binary32 "scale"
// operand before rounding.  An E8M0 block scale byte b is exactly such a power (2^(b - 127), also for b = 0), so
// the operand is b << 23 and the element needs no multiply; a bf16 source goes in as stored, two elements per
// register, with no unpacking either.  (With E4M3 block scales the multiplier 1 / (s g) is no power of two and
// the elements are multiplied in binary32 first, as above.)
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float mx_scale_operand(uint32_t byte) { return u2f(byte << 23); }

template <int BYTE>
__device__ __forceinline__ uint32_t mx_pair_bf16(uint32_t acc, uint32_t w, float sc)
{
    return __builtin_amdgcn_cvt_scalef32_pk_fp4_bf16(acc, __builtin_bit_cast(bf16x2_t, w), sc, BYTE);
}
// elements 2 BYTE and 2 BYTE + 1 of a chunk -> byte BYTE of acc, round to nearest
template <int DT, int BYTE>
__device__ __forceinline__ uint32_t mx_rtn_pair(uint32_t acc, const Chunk<DT> &v, float sc)
{
    if constexpr (DT == NVFP4_BF16)
        return mx_pair_bf16<BYTE>(acc, v.word(BYTE), sc);
    else
        return __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(acc, v.get(2 * BYTE), v.get(2 * BYTE + 1), sc, BYTE);
}
// rows R and R + 1 of column c of a lane tile -> byte BYTE of acc, round to nearest
template <int DT, int BYTE>
__device__ __forceinline__ uint32_t mx_rtn_rows(uint32_t acc, const Chunk<DT> &top, const Chunk<DT> &bot, int c, float sc)
{
    if constexpr (DT == NVFP4_BF16) {
        const uint32_t w = __builtin_amdgcn_perm(bot.word(c >> 1), top.word(c >> 1), (c & 1) ? 0x07060302u : 0x05040100u);
        return mx_pair_bf16<BYTE>(acc, w, sc);
    } else {
        return __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(acc, top.get(c), bot.get(c), sc, BYTE);
    }
}
// Stochastic rounding of element t of a chunk through slot 0 of the convert (see sr_elem0) -> low nibble of byte
// BYTE of acc.  (Inline assembly for the same reason as above: the accumulator must be tied to the destination.)
// Always the binary32-source convert: the bf16-source form of the stochastic convert does not consume the 16
// random bits the way the binary32 form does (measured: 0.6 % of the codes of a bf16 tensor differ, all of them
// elements that land between 0 and 0.5), so a bf16 element is widened first; only the multiply is saved.
template <int DT, int BYTE>
__device__ __forceinline__ uint32_t mx_sr_elem0(uint32_t acc, const Chunk<DT> &v, int t, uint32_t seed, float sc)
{
    typedef float float2_t __attribute__((ext_vector_type(2)));
    const float2_t p = float2_t{v.get(t), 0.0f};
    if (BYTE == 0) asm("v_cvt_scalef32_sr_pk_fp4_f32 %0, %1, %2, %3" : "+v"(acc) : "v"(p), "v"(seed), "v"(sc));
    if (BYTE == 1) asm("v_cvt_scalef32_sr_pk_fp4_f32 %0, %1, %2, %3 op_sel:[0,0,1,0]" : "+v"(acc) : "v"(p), "v"(seed), "v"(sc));
    if (BYTE == 2) asm("v_cvt_scalef32_sr_pk_fp4_f32 %0, %1, %2, %3 op_sel:[0,0,0,1]" : "+v"(acc) : "v"(p), "v"(seed), "v"(sc));
    if (BYTE == 3) asm("v_cvt_scalef32_sr_pk_fp4_f32 %0, %1, %2, %3 op_sel:[0,0,1,1]" : "+v"(acc) : "v"(p), "v"(seed), "v"(sc));
    return acc;
}
template <int DT>
__device__ __forceinline__ uint32_t mx_sr_chunk(const Chunk<DT> &v, float sc, const u32x4 &d)
{
    const uint32_t n0 = ~d.x, n1 = ~d.y, n2 = ~d.z, n3 = ~d.w;
    uint32_t lo = 0, hi = 0;
    lo = mx_sr_elem0<DT, 0>(lo, v, 0, sr_seed0(n0, 0), sc);
    hi = mx_sr_elem0<DT, 0>(hi, v, 1, sr_seed0(n0, 1), sc);
    lo = mx_sr_elem0<DT, 1>(lo, v, 2, sr_seed0(n1, 0), sc);
    hi = mx_sr_elem0<DT, 1>(hi, v, 3, sr_seed0(n1, 1), sc);
    lo = mx_sr_elem0<DT, 2>(lo, v, 4, sr_seed0(n2, 0), sc);
    hi = mx_sr_elem0<DT, 2>(hi, v, 5, sr_seed0(n2, 1), sc);
    lo = mx_sr_elem0<DT, 3>(lo, v, 6, sr_seed0(n3, 0), sc);
    hi = mx_sr_elem0<DT, 3>(hi, v, 7, sr_seed0(n3, 1), sc);
    return lo | (hi << 4);
}
// 8 elements of a row, rounding RND, MX (scale operand) or multiplier form
template <int DT, int RND, bool MXS>
__device__ __forceinline__ uint32_t chunk_codes_hw(const Chunk<DT> &v, float q, uint32_t seed, uint64_t ctr)
{
    uint32_t packed = 0;
    if constexpr (RND == NVFP4_RTN && MXS) {
        packed = mx_rtn_pair<DT, 0>(packed, v, q);
        packed = mx_rtn_pair<DT, 1>(packed, v, q);
        packed = mx_rtn_pair<DT, 2>(packed, v, q);
        packed = mx_rtn_pair<DT, 3>(packed, v, q);
    } else if constexpr (RND == NVFP4_RTN) {
        packed = quant_pair_hw<0>(packed, v.get(0), v.get(1), q);
        packed = quant_pair_hw<1>(packed, v.get(2), v.get(3), q);
        packed = quant_pair_hw<2>(packed, v.get(4), v.get(5), q);
        packed = quant_pair_hw<3>(packed, v.get(6), v.get(7), q);
    } else if constexpr (MXS) {
        packed = mx_sr_chunk(v, q, sr_draw(seed, ctr));
    } else {
        packed = sr_chunk_hw(v, q, sr_draw(seed, ctr));
    }
    return packed;
}

// ------------------------------------------------------------------ row-blocked tile

constexpr int ROWS_UNROLL = 4;  // chunks per thread

// (one chunk per thread: the multiplier is divided out per block, a table would cost more than it saves)
template <int DT, int B, int SF, int RND, bool HW, int NT = 256, int UNROLL = ROWS_UNROLL>
__device__ __forceinline__ float rows_tile(const QuantArgs &P, const int64_t wg)
{
    constexpr int LPB = B / 8;  // lanes per block
    constexpr bool MXS = HW && SF == NVFP4_SCALE_E8M0;  // block scale as the convert's scale operand
    constexpr bool TAB = HW && SF == NVFP4_SCALE_E4M3 && UNROLL > 1;
    const int64_t cpr = P.cols >> 3;
    const int64_t total = P.rows * cpr;
    const int64_t base = wg * (NT * UNROLL) + threadIdx.x;
    const bool dense = P.ld == P.cols;
    Chunk<DT> v[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
        const int64_t id = base + u * NT;
        if (id < total) {
            int64_t off = id * 8;
            if (!dense) {
                // (a 64-bit division per chunk costs more than the chunk's arithmetic)
                const int64_t i = total <= 0xFFFFFFFF ? (int64_t)((uint32_t)id / (uint32_t)cpr) : id / cpr;
                off += i * (P.ld - P.cols);
            }
            v[u].template load<true>(P.x, off);
        } else {
            v[u].zero();
        }
    }
    // (after the loads are issued: folding the partial maxima then overlaps their latency)
    const float g = resolve_g<DT, NT, SF == NVFP4_SCALE_E4M3>(P);
    const float k = 1.0f / (6.0f * g);
    if (TAB) build_qtab<SF, HW>(g);
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
        const int64_t id = base + u * NT;
        // a whole block is in or out of range together, so the lanes exchanged below are
        // either all live or all holding zeros
        const float a = group_max<LPB>(MXS ? chunk_amax_packed(v[u]) : chunk_amax(v[u]));
        float q;
        const uint32_t sbyte = block_scale<SF, HW, TAB>(a, g, k, &q);
        uint32_t packed = 0;
        if (HW) {
            if (MXS) q = mx_scale_operand(sbyte);
            packed = chunk_codes_hw<DT, RND, MXS>(v[u], q, P.seed, (uint64_t)id);  // element index = 8*id + t
        } else {
            u32x4 d = {0, 0, 0, 0};
            if (RND == NVFP4_SR) d = sr_draw(P.seed, (uint64_t)id);  // element index = 8*id + t
#pragma unroll
            for (int t = 0; t < 8; ++t)
                packed |= quant_elem<RND>(v[u].get(t), q, sr_bits_of(d, t)) << (4 * t);
        }
        // scale bytes: lanes that start a block hold them; up to four neighbouring blocks are
        // merged into one 4-byte store
        constexpr int GATHER = LPB <= 4 ? 4 : 1;  // blocks merged per store
        uint32_t sw = sbyte;
        if (GATHER == 4) {
            sw |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)sw, 0x100 + LPB, 0xF, 0xF, true) << 8;       // lane + LPB
            sw |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)sw, 0x100 + 2 * LPB, 0xF, 0xF, true) << 16;  // lane + 2 LPB
        }
        if (id < total) {
            store4_stream(reinterpret_cast<uint32_t *>(P.codes) + id, packed);
            const int64_t blk = id / LPB;
            if (GATHER == 4 && blk + 4 <= total / LPB) {
                if ((threadIdx.x & (4 * LPB - 1)) == 0) store4_stream(P.scales + blk, sw);
            } else if ((threadIdx.x & (LPB - 1)) == 0) {
                P.scales[blk] = (uint8_t)sbyte;  // last (partial) group of four, or wide blocks
            }
        }
    }
    return g;
}

}  // namespace nvfp4
