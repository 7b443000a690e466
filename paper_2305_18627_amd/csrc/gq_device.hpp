// Device-side building blocks of the Global-QSGD hot path for gfx950 (wave64).
// Internal to the library; the public surface is include/gqsgd.h.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

namespace gq {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef short i16x4 __attribute__((ext_vector_type(4)));

constexpr int kBlock = 256;          // threads per workgroup: four wave64

// f(integral_constant<int, BEGIN>), ..., f(integral_constant<int, END - 1>): a loop whose index is a compile-time
// constant in the body, so that it is unrolled by the language and not at the optimizer's discretion.
template <int BEGIN, int END, typename F> __device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (BEGIN < END) {
        f(std::integral_constant<int, BEGIN>{});
        static_for<BEGIN + 1, END>(f);
    }
}
constexpr int kMaxWorkers = 64;

// Per-worker device pointers, passed to the kernels by value.  A kernel takes no more of them than it can use: launching
// one with 1.5 KB of arguments costs the host 1.4 us more than one with a few words (5.1 against 3.7 us).
template <int N> struct GradPtrsN { const float *x[N]; };
typedef GradPtrsN<kMaxWorkers> GradPtrs;
template <int KT> using GradPtrsFor = GradPtrsN<(KT > 0 ? KT : kMaxWorkers)>;       // KT: compile-time worker count, 0 = run-time
template <int KT> static inline GradPtrsFor<KT> pointers_for(const GradPtrs &P)
{
    GradPtrsFor<KT> r;
    for (int i = 0; i < (KT > 0 ? KT : kMaxWorkers); i++) r.x[i] = P.x[i];
    return r;
}
struct LevelPtrs { void *lv[kMaxWorkers]; uint32_t *sp[kMaxWorkers]; };
struct LevelCPtrs { const void *lv[kMaxWorkers]; const uint32_t *sp[kMaxWorkers]; };
struct CodePtrs { const void *lv[kMaxWorkers]; };                                    // codes without sign planes
struct NoPtrs {};

// ---------------------------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11).  The 32x32->64 products map to v_mad_u64_u32, the two
// three-way xors of a round to v_bitop3_b32; the key schedule depends on the seed only and stays in
// scalar registers.  What an instruction costs on gfx950 (cycles a wave, eight waves per SIMD): adds, xors, ands, ors, right
// shifts, moves and binary32 adds, products and fused multiply-adds 2.3 to 2.6; products of integers (64-bit results
// included), left shifts, byte permutes, bit-field operations, conversions, minima, compares, packed 16-bit operations 4.3 to 4.6.
// ---------------------------------------------------------------------------------------------
struct Words4 { uint32_t w[4]; };

// a ^ b ^ c in one instruction: gfx950's three-input bitwise op with truth table 0x96
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

template <bool SCALAR_START = true>
__device__ __forceinline__ Words4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                                uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; r++) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
        // Where c1 and c2 are the same for all lanes, half of the words of the first three rounds are too: written as
        // plain xors, with the uniform operands together, they stay on the scalar unit (the three-input instruction
        // exists on the vector unit only, and would take the next product there with it).  Where few waves hide each other's
        // latency, the scalar products' is the longer one: SCALAR_START off.
        const uint32_t n0 = SCALAR_START && r < 3 ? (uint32_t)(p1 >> 32) ^ (c1 ^ k0) : xor3((uint32_t)(p1 >> 32), c1, k0);
        const uint32_t n2 = SCALAR_START && r < 3 ? (uint32_t)(p0 >> 32) ^ (c3 ^ k1) : xor3((uint32_t)(p0 >> 32), c3, k1);
        c1 = (uint32_t)p1;
        c3 = (uint32_t)p0;
        c0 = n0;
        c2 = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    Words4 o;
    o.w[0] = c0; o.w[1] = c1; o.w[2] = c2; o.w[3] = c3;
    return o;
}

// The four random words of the coordinates 4*call .. 4*call+3 of one worker (Eq. (2) draws).
__device__ __forceinline__ Words4 random_words(uint64_t seed, uint32_t worker, uint64_t call)
{
    return philox4x32_10((uint32_t)call, (uint32_t)(call >> 32), worker, 0u,
                         (uint32_t)seed, (uint32_t)(seed >> 32));
}

// ---------------------------------------------------------------------------------------------
// Per-call constants derived from the norm on the device (Algorithm 1's normalisation, y = |x| / norm).
// ---------------------------------------------------------------------------------------------
struct Scale {
    float scale;   // s / norm (linear) or 2^(s-1) / norm (exponential); 0 if the norm is unusable
    float top;     // s (linear) or 2^(s-1) (exponential) as a float
    float full;    // the norm: |x| >= full is y = 1, the top level with certainty; NaN (never reached) if the norm is unusable
};

template <int SCHEME>
__device__ __forceinline__ Scale make_scale(float norm, int s)
{
    Scale sc;
    sc.top = SCHEME == 0 ? (float)s : __uint_as_float((uint32_t)(127 + s - 1) << 23);
    const float q = sc.top / norm;                          // correctly rounded division
    const bool ok = (norm > 0.0f) && (norm <= 3.402823466e+38f) && (q <= 3.402823466e+38f);
    sc.scale = ok ? q : 0.0f;                               // zero / non-finite norm => every code is 0
    sc.full = ok ? norm : __builtin_nanf("");
    return sc;
}

// ---------------------------------------------------------------------------------------------
// Definition 1 / Eq. (2) for one coordinate.  `magnitude` is the integer value of the code without its sign, as a float
// whose integer conversion is exact; with the sign of x it is what is added to the sum.
// ---------------------------------------------------------------------------------------------
template <int SCHEME> struct Round;

// min(t, top) for t >= -0, and 0 for a NaN t (a NaN or Inf coordinate times a zero scale, or a NaN
// coordinate): v_med3_f32 returns the smallest of its non-NaN operands when one operand is a NaN, so the
// clamp at the top level and the "a NaN rounds to code 0" rule cost one instruction together.
__device__ __forceinline__ float clamp_nan_to_zero(float t, float top)
{
    return __builtin_amdgcn_fmed3f(t, 0.0f, top);
}

// Linear grid l_u = (s-u)/s: t = y*s lies between h and h+1; the upper one is taken iff U' < t-h.
template <> struct Round<0> {
    static __device__ __forceinline__ float magnitude(float x, const Scale &sc, uint32_t r)
    {
        const float u = (float)r * 0x1.fffffep-33f;                       // U' in [0,1)
        const float ax = __builtin_fabsf(x);
        const float v = __builtin_fmaf(ax, sc.scale, -u);                 // t - U', one rounding
        const float c = clamp_nan_to_zero(__builtin_ceilf(v), sc.top);   // clamp at the top level
        return ax >= sc.full ? sc.top : c;                                // y = 1 sits on the top level
    }
    // magnitude(x, sc, r) != 0 for s >= 2, without the clamp: ceil(v) > 0 iff v > 0 (false for a NaN).  At the norm
    // |x| scale >= s (1 - 2^-21) > U' anyway; for s = 1 the caller adds |x| >= sc.full.
    static __device__ __forceinline__ bool nonzero(float x, const Scale &sc, uint32_t r)
    {
        const float u = (float)r * 0x1.fffffep-33f;
        const float ax = __builtin_fabsf(x);
        return __builtin_fmaf(ax, sc.scale, -u) > 0.0f;
    }
};

// Exponential grid {0} u {2^-j}: z = y*2^(s-1); a binary32 z >= 1 is rounded to a neighbouring power of
// two by adding 23 random bits to its mantissa; z < 1 is first moved to 1+z in [1,2).
template <> struct Round<1> {
    // bits of the rounded w = z (+ one) and one = (z < 1)
    struct Rounded { uint32_t b; float one; };
    static __device__ __forceinline__ Rounded rounded(float x, const Scale &sc, uint32_t r)
    {
        const float ax = __builtin_fabsf(x);
        const float z = ax >= sc.full ? sc.top : clamp_nan_to_zero(ax * sc.scale, sc.top);   // y = 1 sits on the top level
        // z < 1 ? 1 : 0, as 2^25 (1 - z) clamped to [0, 1] (exact: it is 0 or below for z >= 1, and 2 or more for z < 1):
        // the clamp is part of the fma, a compare and a select cost 2.6 times as much
        const float one = __builtin_amdgcn_fmed3f(__builtin_fmaf(z, -0x1p25f, 0x1p25f), 0.0f, 1.0f);
        return {__float_as_uint(z + one) + (r >> 9), one};
    }
    static __device__ __forceinline__ float magnitude(const Rounded &t) { return __uint_as_float(t.b & 0x7F800000u) - t.one; }   // 0, 1, 2, 4, ..
    // The code k of magnitude 2^(k-1), 0 for 0.  w has the exponent field k + 126 for z >= 1 and k + 127 for z < 1; the bits of
    // 0.5 or 1.0 take that out.
    static __device__ __forceinline__ uint32_t code(const Rounded &t) { return (t.b - (__float_as_uint(t.one) | 0x3F000000u)) >> 23; }
    static __device__ __forceinline__ float magnitude(float x, const Scale &sc, uint32_t r) { return magnitude(rounded(x, sc, r)); }
    // magnitude(x, sc, r) != 0 for s >= 2: z < 1 iff the rounded 1 + z reaches 2, z >= 1 always, and then 1 + z >= 2; a NaN
    // z counts as 0.  At the norm z >= top (1 - 2^-21) >= 1 anyway; for s = 1 the caller adds |x| >= sc.full.
    static __device__ __forceinline__ bool nonzero(float x, const Scale &sc, uint32_t r)
    {
        const float ax = __builtin_fabsf(x);
        const float z = clamp_nan_to_zero(ax * sc.scale, sc.top);
        return __float_as_uint(z + 1.0f) + (r >> 9) >= 0x40000000u;
    }
};

// Four coordinates rounded: m the magnitudes, v the signed values; exponential grid: k the codes without sign.  What a kernel
// does not use is not computed.  The kernels that store codes are bound by instruction issue as much as by HBM, hence the
// care about which instructions form the fields.  gq_quantize of 67.1e6 coordinates, against packing by shifts and
// selects: linear 4 bits + planes 55.9 -> 49.0 us, exponential 4 bits + planes 64 -> 54, exponential int8 57.1 -> 55.2,
// packed int4 54.9 -> 52.9 (short draws 51.3 -> 48.1).
template <int SCHEME> struct Quad4 {
    float m[4], v[4];
    uint32_t k[4], xbits[4];
    __device__ __forceinline__ Quad4(const f32x4 &x, const Scale &sc, const uint32_t *draw)
    {
        const float c[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int j = 0; j < 4; j++) {
            if constexpr (SCHEME == 0) {
                m[j] = Round<0>::magnitude(c[j], sc, draw[j]);
            } else {
                const auto t = Round<1>::rounded(c[j], sc, draw[j]);
                m[j] = Round<1>::magnitude(t);
                k[j] = Round<1>::code(t);
                xbits[j] = __float_as_uint(c[j]);
            }
            v[j] = __builtin_copysignf(m[j], c[j]);
        }
    }
    __device__ __forceinline__ uint32_t exp_signed_code(int j) const
    {
        const uint32_t s = (uint32_t)((int)xbits[j] >> 31);
        return (k[j] ^ s) - s;
    }
    // The four codes as bytes or nibbles of one word, coordinate j in field j: two's complement, or magnitudes alone.
    // Linear codes are put together as floats (exact below 2^24) and converted together: fused multiply-adds issue in half
    // the time of conversions, shifts and byte permutes.  A bias of half the field's range in every field keeps the sum
    // non-negative; flipping the fields' top bits takes it out again.
    __device__ __forceinline__ uint32_t signed_bytes() const
    {
        if (SCHEME == 0) {
            const uint32_t lo = (uint32_t)__builtin_fmaf(v[1], 256.0f, v[0] + 32896.0f);
            const uint32_t hi = (uint32_t)__builtin_fmaf(v[3], 256.0f, v[2] + 32896.0f);
            return (lo | (hi << 16)) ^ 0x80808080u;
        }
        const uint32_t t = (((exp_signed_code(3) << 8) + exp_signed_code(2)) << 8) + exp_signed_code(1);
        return ((t << 8) + exp_signed_code(0) + 0x80808080u) ^ 0x80808080u;
    }
    __device__ __forceinline__ uint32_t signed_nibbles() const
    {
        if (SCHEME == 0)
            return (uint32_t)__builtin_fmaf(v[3], 4096.0f, __builtin_fmaf(v[2], 256.0f, __builtin_fmaf(v[1], 16.0f, v[0] + 34952.0f))) ^ 0x8888u;
        const uint32_t t = (((exp_signed_code(3) << 4) + exp_signed_code(2)) << 4) + exp_signed_code(1);
        return ((t << 4) + exp_signed_code(0) + 0x8888u) ^ 0x8888u;
    }
    __device__ __forceinline__ uint32_t magnitude_bytes() const
    {
        if (SCHEME == 0) {
            const uint32_t lo = (uint32_t)__builtin_fmaf(m[1], 256.0f, m[0]), hi = (uint32_t)__builtin_fmaf(m[3], 256.0f, m[2]);
            return lo | (hi << 16);
        }
        return k[0] | (k[1] << 8) | (k[2] << 16) | (k[3] << 24);
    }
    __device__ __forceinline__ uint32_t magnitude_nibbles() const
    {
        if (SCHEME == 0) return (uint32_t)__builtin_fmaf(m[3], 4096.0f, __builtin_fmaf(m[2], 256.0f, __builtin_fmaf(m[1], 16.0f, m[0])));
        return k[0] | (k[1] << 4) | (k[2] << 8) | (k[3] << 12);
    }
    // bit j = 1 iff code j is negative: -2 v clamped to [0, 1] (a value is 0 or at least 1 in magnitude)
    __device__ __forceinline__ uint32_t sign_nibble() const
    {
        float n[4];
#pragma unroll
        for (int j = 0; j < 4; j++) n[j] = __builtin_amdgcn_fmed3f(v[j] * -2.0f, 0.0f, 1.0f);
        return (uint32_t)__builtin_fmaf(n[3], 8.0f, __builtin_fmaf(n[2], 4.0f, __builtin_fmaf(n[1], 2.0f, n[0])));
    }
};

// Four consecutive coordinates of a gradient (vector v); nvalid < 4 of them exist at the ragged end, zeros beyond.
__device__ __forceinline__ f32x4 load_coords(const float *x, int64_t v, int nvalid)
{
    if (nvalid == 4) return __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(x) + v);
    f32x4 a = {0.0f, 0.0f, 0.0f, 0.0f};
    const float *t = x + (v << 2);
    if (nvalid > 0) a.x = t[0];
    if (nvalid > 1) a.y = t[1];
    if (nvalid > 2) a.z = t[2];
    return a;
}

// The same without a branch per lane, for launches whose time is latency: vector `li` counted from a workgroup's first (`x`),
// whose last existing coordinate is x[last].  Every lane loads, past the end the last coordinate again; behind a branch each
// load would wait for the one before it.  all_asked_for() behind a batch of such loads keeps the scheduler from putting
// the first one's use before the last one; existing() then zeroes what is past the end.
__device__ __forceinline__ f32x4 load_clamped(const float *x, uint32_t li, uint32_t last)
{
    f32x4 a;
#pragma unroll
    for (uint32_t i = 0; i < 4; i++) {
        const uint32_t c = 4 * li + i;
        a[i] = x[c < last ? c : last];
    }
    return a;
}
__device__ __forceinline__ void all_asked_for() { __builtin_amdgcn_sched_barrier(0); }
__device__ __forceinline__ f32x4 existing(f32x4 a, uint32_t li, uint32_t last)
{
#pragma unroll
    for (uint32_t i = 0; i < 4; i++) a[i] = 4 * li + i <= last ? a[i] : 0.0f;
    return a;
}
// the last existing coordinate counted from the first of a workgroup that begins at vector vb of d coordinates, as far as 32 bits
// reach (no workgroup has so many)
__device__ __forceinline__ uint32_t last_coord(int64_t vb, int64_t d)
{
    const int64_t n = d - 1 - (vb << 2);
    return n < 0x7FFFFFFF ? (uint32_t)n : 0x7FFFFFFFu;
}

// Short draws: coordinate j of a vector takes the low (j even) or high (j odd) half of word j / 2 of the vector's pair
// of Philox words, moved to the top of a 32-bit word with zeros below.
__device__ __forceinline__ uint32_t short_draw(const uint32_t *pair, int j)
{
    return (j & 1) ? (pair[j >> 1] & 0xFFFF0000u) : (pair[j >> 1] << 16);
}

// ---------------------------------------------------------------------------------------------
// Wave reductions for the norm: DPP inside a row of 16 lanes (quad permutes, then the two mirror
// patterns), ds_swizzle across the two rows of a half wave, readlane across the halves.
// Every lane of the wave must be active.  The result is uniform.
// ---------------------------------------------------------------------------------------------
template <int CTRL> __device__ __forceinline__ uint32_t dpp32(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false);
}
template <int CTRL> __device__ __forceinline__ double dpp64(double v)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = dpp32<CTRL>((uint32_t)b), hi = dpp32<CTRL>((uint32_t)(b >> 32));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
__device__ __forceinline__ uint32_t swizzle_xor16(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, 0x401F);   // bit-mask mode: lane ^ 16
}
constexpr int kDppQuadXor1 = 0xB1;     // quad_perm:[1,0,3,2]
constexpr int kDppQuadXor2 = 0x4E;     // quad_perm:[2,3,0,1]
constexpr int kDppHalfMirror = 0x141;  // row_half_mirror: lane i <-> 7-i of each 8
constexpr int kDppMirror = 0x140;      // row_mirror:      lane i <-> 15-i of each 16

// Short draws (16 random bits per coordinate): one Philox call serves the eight coordinates of two
// neighbouring vectors 2c and 2c+1.  To keep every load and store of a wave contiguous, a wave takes 128
// consecutive vectors and lane l owns vectors l ("A") and 64 + l ("B") of them.  Even lane 2i runs the call
// of vectors 2i, 2i+1 of the A half, odd lane 2i+1 the call of vectors 2i, 2i+1 of the B half, and the two
// lanes swap the half of the words the other needs (one DPP exchange of two registers).  Afterwards
// word pair `a` rounds the lane's A vector and `b` its B vector; coordinate j of a vector takes the low
// (j even) or high (j odd) half of word j / 2 of its pair, moved to the top of a 32-bit word with zeros
// below, so that the rounding rules apply unchanged.  Every lane of the wave must be active.
struct ShortDraws { uint32_t a[2], b[2]; };
__device__ __forceinline__ ShortDraws share_short_draws(const Words4 &r, bool odd)
{
    const uint32_t got0 = dpp32<kDppQuadXor1>(odd ? r.w[0] : r.w[2]);
    const uint32_t got1 = dpp32<kDppQuadXor1>(odd ? r.w[1] : r.w[3]);
    ShortDraws o;
    o.a[0] = odd ? got0 : r.w[0]; o.a[1] = odd ? got1 : r.w[1];
    o.b[0] = odd ? r.w[2] : got0; o.b[1] = odd ? r.w[3] : got1;
    return o;
}

__device__ __forceinline__ double wave_sum(double v)
{
    v += dpp64<kDppQuadXor1>(v);
    v += dpp64<kDppQuadXor2>(v);
    v += dpp64<kDppHalfMirror>(v);
    v += dpp64<kDppMirror>(v);
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = swizzle_xor16((uint32_t)b), hi = swizzle_xor16((uint32_t)(b >> 32));
    v += __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
    const uint64_t t = (uint64_t)__double_as_longlong(v);
    const uint32_t lo0 = __builtin_amdgcn_readlane((int)(uint32_t)t, 0), hi0 = __builtin_amdgcn_readlane((int)(uint32_t)(t >> 32), 0);
    const uint32_t lo1 = __builtin_amdgcn_readlane((int)(uint32_t)t, 32), hi1 = __builtin_amdgcn_readlane((int)(uint32_t)(t >> 32), 32);
    return __longlong_as_double((long long)(((uint64_t)hi0 << 32) | lo0)) +
           __longlong_as_double((long long)(((uint64_t)hi1 << 32) | lo1));
}
__device__ __forceinline__ uint32_t wave_max(uint32_t v)
{
    v = max(v, dpp32<kDppQuadXor1>(v));
    v = max(v, dpp32<kDppQuadXor2>(v));
    v = max(v, dpp32<kDppHalfMirror>(v));
    v = max(v, dpp32<kDppMirror>(v));
    v = max(v, swizzle_xor16(v));
    return max((uint32_t)__builtin_amdgcn_readlane((int)v, 0), (uint32_t)__builtin_amdgcn_readlane((int)v, 32));
}

}  // namespace gq
