// Algorithm 1's aggregation step and Eq. (1) on MI355X (gfx950): the integer sum of stored codes and its
// dequantisation.  The contract of the entry points is stated in include/gqsgd.h.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include "gqsgd.h"
#include "gq_device.hpp"
#include "gq_host.hpp"

namespace gq {

// =============================================================================================
// Algorithm 1's aggregation step on stored codes.  Same ownership as the fused kernel: a lane owns four
// coordinates, i.e. one 32-bit (8-bit codes) or 16-bit (4-bit codes) word of every worker's level
// buffer and a nibble of its sign words; loads and the 128-bit stores of a wave are contiguous.
// =============================================================================================
constexpr int kAggBlock = 128;

// the pointers that a format has
template <int PACK> using CodesOf = typename std::conditional<(PACK >= GQ_PACK_U8_SIGNPLANE), LevelCPtrs, CodePtrs>::type;
template <int PACK> static inline CodesOf<PACK> codes_of_format(const LevelCPtrs &L)
{
    if constexpr (PACK >= GQ_PACK_U8_SIGNPLANE) return L;
    else {
        CodePtrs r;
        for (int i = 0; i < kMaxWorkers; i++) r.lv[i] = L.lv[i];
        return r;
    }
}

template <int SCHEME, int PACK>
__global__ void __launch_bounds__(kAggBlock)
int_aggregate_kernel(CodesOf<PACK> L, int K, int64_t d, int64_t v_begin, void *__restrict__ agg_out, int agg_fmt)
{
    constexpr bool kNibble = (PACK == GQ_PACK_I4 || PACK == GQ_PACK_U4_SIGNPLANE);
    constexpr bool kPlane = (PACK == GQ_PACK_U8_SIGNPLANE || PACK == GQ_PACK_U4_SIGNPLANE);
    // Packed two's-complement nibbles are decoded through a 256-entry LDS table indexed by a byte: the
    // entry holds the integer values of both nibbles, each biased by 128, in its two 16-bit halves, so
    // that one 32-bit add accumulates two coordinates (K * 192 < 2^16, no carry between the halves).
    constexpr bool kLut = (PACK == GQ_PACK_I4);
    constexpr int kBias = 128;
    __shared__ uint32_t lut[kLut ? 256 : 1];
    if (kLut) {
        for (int b = threadIdx.x; b < 256; b += kAggBlock) {
            uint32_t e = 0;
            for (int h = 0; h < 2; h++) {
                const int q = ((int)((uint32_t)b << (28 - 4 * h))) >> 28;
                const int mag = (int)((1u << abs(q)) >> 1);
                const int val = SCHEME == 0 ? q : (q < 0 ? -mag : mag);
                e |= (uint32_t)(val + kBias) << (16 * h);
            }
            lut[b] = e;
        }
        __syncthreads();
    }
    const int64_t v = v_begin + (int64_t)blockIdx.x * kAggBlock + threadIdx.x;     // v_begin is a multiple of 8
    const int64_t nfull = d >> 2;
    const int nvalid = v < nfull ? 4 : (v == nfull ? (int)(d & 3) : 0);
    if (nvalid == 0) return;

    struct Unit { uint32_t codes, signs; };
    auto fetch = [&](int w) {
        Unit t;
        if (!kNibble) {
            if (nvalid == 4) {
                t.codes = __builtin_nontemporal_load(reinterpret_cast<const uint32_t *>(L.lv[w]) + v);
            } else {
                const uint8_t *b = reinterpret_cast<const uint8_t *>(L.lv[w]) + (v << 2);
                t.codes = 0;
                for (int i = 0; i < nvalid; i++) t.codes |= (uint32_t)b[i] << (8 * i);
            }
        } else {
            if (nvalid == 4) {
                t.codes = __builtin_nontemporal_load(reinterpret_cast<const uint16_t *>(L.lv[w]) + v);
            } else {
                const uint8_t *b = reinterpret_cast<const uint8_t *>(L.lv[w]) + (v << 1);
                t.codes = b[0];
                if (nvalid == 3) t.codes |= (uint32_t)b[1] << 8;
            }
        }
        t.signs = 0u;
        if constexpr (kPlane) t.signs = (L.sp[w][v >> 3] >> (4 * (int)(v & 7))) & 15u;
        return t;
    };
    int a0 = 0, a1 = 0, a2 = 0, a3 = 0;
    auto value = [&](const Unit &t, int i) {
        int q;
        if (PACK == GQ_PACK_I8)      q = (int)(int8_t)(t.codes >> (8 * i));
        else if (PACK == GQ_PACK_I4) q = ((int)(t.codes << (28 - 4 * i))) >> 28;
        else if (PACK == GQ_PACK_U8_SIGNPLANE) q = (int)((t.codes >> (8 * i)) & 255u);
        else                         q = (int)((t.codes >> (4 * i)) & 15u);
        if (SCHEME == 0) return (kPlane && ((t.signs >> i) & 1u)) ? -q : q;
        const bool neg = kPlane ? (((t.signs >> i) & 1u) != 0u) : (q < 0);
        const int mag = (int)((1u << abs(q)) >> 1);                  // 2^(k-1), 0 for k = 0
        return neg ? -mag : mag;
    };
    uint32_t s01 = 0, s23 = 0;
    auto add = [&](const Unit &t) {
        if (kLut) {
            s01 += lut[t.codes & 255u];
            s23 += lut[(t.codes >> 8) & 255u];
        } else {
            a0 += value(t, 0); a1 += value(t, 1); a2 += value(t, 2); a3 += value(t, 3);
        }
    };
    // eight workers' loads are issued before the first is consumed
    int w = 0;
    for (; w + 8 <= K; w += 8) {
        Unit t[8];
#pragma unroll
        for (int j = 0; j < 8; j++) t[j] = fetch(w + j);
#pragma unroll
        for (int j = 0; j < 8; j++) add(t[j]);
    }
    for (; w + 2 <= K; w += 2) {
        const Unit t0 = fetch(w), t1 = fetch(w + 1);
        add(t0); add(t1);
    }
    for (; w < K; w++) add(fetch(w));
    if (kLut) {
        a0 = (int)(s01 & 0xFFFFu) - K * kBias; a1 = (int)(s01 >> 16) - K * kBias;
        a2 = (int)(s23 & 0xFFFFu) - K * kBias; a3 = (int)(s23 >> 16) - K * kBias;
    }

    if (agg_fmt == GQ_AGG_I32) {
        if (nvalid == 4) {
            const i32x4 o = {a0, a1, a2, a3};
            __builtin_nontemporal_store(o, reinterpret_cast<i32x4 *>(agg_out) + v);
        } else {
            int *o = reinterpret_cast<int *>(agg_out) + (v << 2);
            o[0] = a0;
            if (nvalid > 1) o[1] = a1;
            if (nvalid > 2) o[2] = a2;
        }
    } else {
        if (nvalid == 4) {
            const i16x4 o = {(short)a0, (short)a1, (short)a2, (short)a3};
            __builtin_nontemporal_store(o, reinterpret_cast<i16x4 *>(agg_out) + v);
        } else {
            short *o = reinterpret_cast<short *>(agg_out) + (v << 2);
            o[0] = (short)a0;
            if (nvalid > 1) o[1] = (short)a1;
            if (nvalid > 2) o[2] = (short)a2;
        }
    }
}

// =============================================================================================
// Algorithm 1's aggregation step on packed 4-bit codes, for workgroups that lie wholly inside the buffer.  The
// one-vector-per-lane kernel above moves two bytes per lane and load, which leaves it bound by
// instruction issue, not by HBM.  Here a lane owns EIGHT coordinates: one 32-bit load of codes (and one
// byte of sign bits) per worker.
//   TABLE      every byte of codes, together with its two sign bits in the sign-plane format, indexes an LDS table whose
//       entry holds the integer values of both coordinates, each biased to be non-negative, in its two 16-bit halves: one
//       table read and one 32-bit add accumulate two coordinates (the biased sums stay below 2^16 for K <= 64: at most
//       (64 + 128) * 64 resp. (15 + 16) * 64).
//   otherwise  (two's complement, fewer than kNibTableFrom workers) no table to fill and to wait for: the even and the odd
//       nibbles of the word are four bytes each.  Linear: a nibble with its top bit flipped is the value + 8, and the
//       workers' sum fits a byte (at most 15 * 15).  Exponential: a byte permute looks up value + 128 in eight
//       positive and eight negative values, a third one picks by the nibble's top bit, and the bytes go to 16-bit sums.
// 32-bit sums are staged in LDS so that the workgroup writes two contiguous runs of 16 bytes per thread;
// 16-bit sums are 16 bytes per lane already.  Not for the exponential grid in the sign-plane format
// (values up to 2^14 do not fit the halves): that combination keeps the kernel above.
// =============================================================================================
constexpr int kNibBlock = 128;
constexpr int kNibCoords = 8;
// Two's complement codes: workers from which the table is no slower.  100e6 coordinates, us without / with it: 16-bit sums
// K = 4 65 / 68, 8 94.5 / 103 (linear 94 / 100.5), 12 126.5 / 135, 16 163.5 / 163, 24 231.5 / 230, 32 301 / 300; at 350e6 x 32
// 1080 / 1070 (linear 1087 / 1066); 32-bit sums are equal everywhere (memory).
constexpr int kNibTableFrom = 16;
constexpr int nibble_entries(bool plane, bool table) { return !table ? 1 : (plane ? 1024 : 256); }
constexpr unsigned nibble_lds(bool plane, bool table) { return 4u * (kNibBlock * kNibCoords + nibble_entries(plane, table)); }

// value + 128 of four two's complement nibbles (bits 0..3 of every byte of n) on the exponential grid
__device__ __forceinline__ uint32_t exp_nibble_values(uint32_t n)
{
    const uint32_t which = n & 0x07070707u;
    const uint32_t pos = __builtin_amdgcn_perm(0xC0A09088u, 0x84828180u, which);       // 64 32 16 8 | 4 2 1 0
    const uint32_t neg = __builtin_amdgcn_perm(0x7F7E7C78u, 0x70604000u, which);       // -1 -2 -4 -8 | -16 -32 -64 -128
    return __builtin_amdgcn_perm(neg, pos, ((n >> 1) & 0x04040404u) | 0x03020100u);
}

// Workgroups per compute unit (of 16), from kNibLimitFrom coordinates on.  us without a limit / with it, in turn in one process, 100e6
// coordinates: 32-bit sums K = 4 97.3 / 95.5, 8 134.6 / 128.5, 16 201.0 / 193.1, 32 358.6 / 340.4, 64 665 / 638; with planes K = 8
// 148.7 / 142.2, 16 221.2 / 220.2, 32 459 / 455, 64 880 / 873; 16-bit sums K = 16 164.9 / 159.2, 32 315.7 / 303.7, 64 609 / 583.  At 12e6
// to 25.6e6 coordinates it may lose 2 % (K = 12 22.0 / 22.4, with planes K = 32 104.3 / 106.2).  The others lose: planes K = 4, 16-bit
// sums K = 8 138.9 / 140.2 (150e6), with planes 108.5 / 114.3, 32-bit sums K = 1 79 / 88, 2 82 / 86 (they write more than they read).
constexpr int64_t kNibLimitFrom = 10000000;
static inline int nibble_workgroups(const gq_params *p, int K, int64_t d)
{
    if (d < kNibLimitFrom || K < 4) return 0;
    const bool plane = p->pack == GQ_PACK_U4_SIGNPLANE;
    if (p->agg == GQ_AGG_I16) return !plane && K >= kNibTableFrom ? 12 : 0;
    return plane ? (K >= 8 ? 12 : 0) : (K >= 8 ? 11 : 12);
}

template <int SCHEME, bool PLANE, bool TABLE>
__global__ void __launch_bounds__(kNibBlock)
int_aggregate_nibble_kernel(CodesOf<PLANE ? GQ_PACK_U4_SIGNPLANE : GQ_PACK_I4> L, int K, void *__restrict__ agg_out, int agg_fmt)
{
    static_assert(!(SCHEME == 1 && PLANE), "exponential sign-plane values do not fit 16-bit halves");
    static_assert(TABLE || !PLANE, "magnitudes and their sign bits meet in the table");
    constexpr int kEntries = nibble_entries(PLANE, TABLE);
    constexpr int kBias = PLANE ? 16 : (!TABLE && SCHEME == 0 ? 8 : 128);
    __shared__ uint32_t lut[kEntries];
    __shared__ int stage[kNibBlock * kNibCoords];
    if (TABLE) {
        for (int e = threadIdx.x; e < kEntries; e += kNibBlock) {
            uint32_t entry = 0;
            for (int h = 0; h < 2; h++) {
                const int nibble = (e >> (4 * h)) & 15;
                int val;
                if (PLANE) {
                    val = nibble;                                         // linear magnitude
                    if ((e >> (8 + h)) & 1) val = -val;
                } else {
                    const int q = (nibble ^ 8) - 8;                       // two's complement nibble
                    const int mag = (int)((1u << abs(q)) >> 1);           // 2^(k-1), 0 for k = 0
                    val = SCHEME == 0 ? q : (q < 0 ? -mag : mag);
                }
                entry |= (uint32_t)(val + kBias) << (16 * h);
            }
            lut[e] = entry;
        }
        __syncthreads();
    }
    const int64_t ub = (int64_t)blockIdx.x * kNibBlock;                   // scalar
    const int64_t u = ub + threadIdx.x;                                   // eight coordinates 8u .. 8u+7

    // biased sums in 16-bit halves: TABLE coordinates (0,1) (2,3) (4,5) (6,7), else (0,4) (1,5) (2,6) (3,7)
    uint32_t s0 = 0, s1 = 0, s2 = 0, s3 = 0;
    uint32_t even = 0, odd = 0;                                           // no table, linear: byte sums
    auto add = [&](uint32_t c, uint32_t sb) {
        if constexpr (PLANE) {
            s0 += lut[(c & 255u) | ((sb & 3u) << 8)];
            s1 += lut[((c >> 8) & 255u) | ((sb & 12u) << 6)];
            s2 += lut[((c >> 16) & 255u) | ((sb & 48u) << 4)];
            s3 += lut[(c >> 24) | ((sb & 192u) << 2)];
        } else if constexpr (TABLE) {
            s0 += lut[c & 255u];
            s1 += lut[(c >> 8) & 255u];
            s2 += lut[(c >> 16) & 255u];
            s3 += lut[c >> 24];
        } else if constexpr (SCHEME == 0) {
            even += (c & 0x0F0F0F0Fu) ^ 0x08080808u;
            odd += ((c >> 4) & 0x0F0F0F0Fu) ^ 0x08080808u;
        } else {
            const uint32_t e = exp_nibble_values(c), o = exp_nibble_values(c >> 4);
            s0 += e & 0x00FF00FFu; s2 += (e >> 8) & 0x00FF00FFu;
            s1 += o & 0x00FF00FFu; s3 += (o >> 8) & 0x00FF00FFu;
        }
    };
    auto codes_of = [&](int w) { return __builtin_nontemporal_load(reinterpret_cast<const uint32_t *>(L.lv[w]) + ub + threadIdx.x); };
    auto signs_of = [&](int w) -> uint32_t {
        if constexpr (PLANE) return reinterpret_cast<const uint8_t *>(L.sp[w])[ub + threadIdx.x];
        else return 0u;
    };
    int w = 0;
    for (; w + 8 <= K; w += 8) {                     // eight workers' loads are issued before the first is consumed
        uint32_t c[8], sb[8];
#pragma unroll
        for (int j = 0; j < 8; j++) { c[j] = codes_of(w + j); sb[j] = signs_of(w + j); }
#pragma unroll
        for (int j = 0; j < 8; j++) add(c[j], sb[j]);
    }
    if (w + 4 <= K) {
        uint32_t c[4], sb[4];
#pragma unroll
        for (int j = 0; j < 4; j++) { c[j] = codes_of(w + j); sb[j] = signs_of(w + j); }
#pragma unroll
        for (int j = 0; j < 4; j++) add(c[j], sb[j]);
        w += 4;
    }
    if (w + 2 <= K) {
        const uint32_t c0 = codes_of(w), c1 = codes_of(w + 1), b0 = signs_of(w), b1 = signs_of(w + 1);
        add(c0, b0); add(c1, b1);
        w += 2;
    }
    if (w < K) add(codes_of(w), signs_of(w));
    if constexpr (!TABLE && SCHEME == 0) {
        s0 = even & 0x00FF00FFu; s2 = (even >> 8) & 0x00FF00FFu;
        s1 = odd & 0x00FF00FFu; s3 = (odd >> 8) & 0x00FF00FFu;
    }
    const int off = K * kBias;
    int a[8];
    if constexpr (TABLE) {
        a[0] = (int)(s0 & 0xFFFFu) - off; a[1] = (int)(s0 >> 16) - off; a[2] = (int)(s1 & 0xFFFFu) - off; a[3] = (int)(s1 >> 16) - off;
        a[4] = (int)(s2 & 0xFFFFu) - off; a[5] = (int)(s2 >> 16) - off; a[6] = (int)(s3 & 0xFFFFu) - off; a[7] = (int)(s3 >> 16) - off;
    } else {
        a[0] = (int)(s0 & 0xFFFFu) - off; a[4] = (int)(s0 >> 16) - off; a[1] = (int)(s1 & 0xFFFFu) - off; a[5] = (int)(s1 >> 16) - off;
        a[2] = (int)(s2 & 0xFFFFu) - off; a[6] = (int)(s2 >> 16) - off; a[3] = (int)(s3 & 0xFFFFu) - off; a[7] = (int)(s3 >> 16) - off;
    }
    if (agg_fmt == GQ_AGG_I16) {
        const u32x4 o = {((uint32_t)a[0] & 0xFFFFu) | ((uint32_t)a[1] << 16), ((uint32_t)a[2] & 0xFFFFu) | ((uint32_t)a[3] << 16),
                         ((uint32_t)a[4] & 0xFFFFu) | ((uint32_t)a[5] << 16), ((uint32_t)a[6] & 0xFFFFu) | ((uint32_t)a[7] << 16)};
        __builtin_nontemporal_store(o, reinterpret_cast<u32x4 *>(agg_out) + u);
    } else {
        const int t = (int)threadIdx.x;
        *reinterpret_cast<i32x4 *>(&stage[8 * t]) = i32x4{a[0], a[1], a[2], a[3]};
        *reinterpret_cast<i32x4 *>(&stage[8 * t + 4]) = i32x4{a[4], a[5], a[6], a[7]};
        __syncthreads();
        i32x4 *out = reinterpret_cast<i32x4 *>(agg_out) + (int64_t)blockIdx.x * (kNibBlock * kNibCoords / 4);
        __builtin_nontemporal_store(*reinterpret_cast<const i32x4 *>(&stage[4 * t]), out + t);
        __builtin_nontemporal_store(*reinterpret_cast<const i32x4 *>(&stage[4 * (kNibBlock + t)]), out + kNibBlock + t);
    }
}

// =============================================================================================
// Eq. (1): out = norm * A / (n * unit).
// =============================================================================================
template <typename T>
__global__ void __launch_bounds__(kBlock)
dequantize_kernel(const T *__restrict__ agg, int64_t d, const float *__restrict__ norm, float deq_div,
                  float *__restrict__ out)
{
    typedef T tx4 __attribute__((ext_vector_type(4)));
    const int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t nfull = d >> 2;
    const int nvalid = v < nfull ? 4 : (v == nfull ? (int)(d & 3) : 0);
    if (nvalid == 0) return;
    const float nrm = *norm;
    const float c = (nrm > 0.0f && nrm <= 3.402823466e+38f) ? nrm / deq_div : 0.0f;
    if (nvalid == 4) {
        const tx4 a = __builtin_nontemporal_load(reinterpret_cast<const tx4 *>(agg) + v);
        const f32x4 o = {(float)a.x * c, (float)a.y * c, (float)a.z * c, (float)a.w * c};
        __builtin_nontemporal_store(o, reinterpret_cast<f32x4 *>(out) + v);
    } else {
        for (int i = 0; i < nvalid; i++) out[(v << 2) + i] = (float)agg[(v << 2) + i] * c;
    }
}

}  // namespace gq

using namespace gq;

extern "C" {

gq_status gq_int_aggregate(const void *const *levels, const uint32_t *const *signplanes, int K, int64_t d,
                           const gq_params *p, void *agg_out, void *hip_stream)
{
    gq_status st = check_params(p, true, true);
    if (st != GQ_OK) return st;
    if (!levels || K < 1 || K > GQ_MAX_WORKERS || d < 0) return GQ_ERR_INVALID_ARG;
    st = gq_check_width(p, K);
    if (st != GQ_OK) return st;
    const bool plane = p->pack >= GQ_PACK_U8_SIGNPLANE;
    if (plane && !signplanes) return GQ_ERR_INVALID_ARG;
    LevelCPtrs L;
    for (int i = 0; i < K; i++) {
        if (d > 0 && !aligned(levels[i], 16)) return GQ_ERR_INVALID_ARG;
        L.lv[i] = levels[i];
        L.sp[i] = nullptr;
        if (plane) {
            if (d > 0 && !aligned(signplanes[i], 4)) return GQ_ERR_INVALID_ARG;
            L.sp[i] = signplanes[i];
        }
    }
    if (d > 0 && !aligned(agg_out, 16)) return GQ_ERR_INVALID_ARG;
    if (d == 0) return GQ_OK;
    hipStream_t s = (hipStream_t)hip_stream;
    const int64_t nvec = (d + 3) / 4;
    // packed 4-bit codes: the workgroups that lie wholly inside the buffer take the eight-coordinates-per-lane
    // kernel, the ragged rest (fewer than 1024 coordinates) the general one
    int64_t v_begin = 0;
    const bool nibble_sum = p->pack == GQ_PACK_I4 || (p->pack == GQ_PACK_U4_SIGNPLANE && p->scheme == GQ_LINEAR);
    if (nibble_sum) {
        const int64_t wide_blocks = d / (kNibBlock * kNibCoords);
        if (!grid_fits(wide_blocks, kNibBlock)) return GQ_ERR_INVALID_ARG;
        if (wide_blocks > 0) {
            const dim3 wgrid((unsigned)wide_blocks), wblock(kNibBlock);
            const int per_cu = nibble_workgroups(p, K, d);
#define GQ_NIB(SC, PLANE, TABLE) hipLaunchKernelGGL((int_aggregate_nibble_kernel<SC, PLANE, TABLE>), wgrid, wblock, \
                                                    lds_for_workgroups(per_cu, nibble_lds(PLANE, TABLE)), s, \
                                                    codes_of_format<PLANE ? GQ_PACK_U4_SIGNPLANE : GQ_PACK_I4>(L), K, agg_out, p->agg)
            const bool table = K >= kNibTableFrom;
            if (p->pack == GQ_PACK_U4_SIGNPLANE) GQ_NIB(0, true, true);
            else if (p->scheme == GQ_LINEAR) { if (table) GQ_NIB(0, false, true); else GQ_NIB(0, false, false); }
            else { if (table) GQ_NIB(1, false, true); else GQ_NIB(1, false, false); }
#undef GQ_NIB
            if (launched() != GQ_OK) return GQ_ERR_DEVICE;
            v_begin = wide_blocks * (kNibBlock * kNibCoords / 4);
            if (v_begin >= nvec) return GQ_OK;
        }
    }
    const int64_t blocks = (nvec - v_begin + kAggBlock - 1) / kAggBlock;
    if (!grid_fits(blocks, kAggBlock)) return GQ_ERR_INVALID_ARG;
    const dim3 grid((unsigned)blocks), block(kAggBlock);
#define GQ_AGG(SC, PK) hipLaunchKernelGGL((int_aggregate_kernel<SC, PK>), grid, block, 0, s, codes_of_format<PK>(L), K, d, v_begin, agg_out, p->agg)
    if (p->scheme == GQ_LINEAR) {
        switch (p->pack) {
        case GQ_PACK_I8: GQ_AGG(0, GQ_PACK_I8); break;
        case GQ_PACK_I4: GQ_AGG(0, GQ_PACK_I4); break;
        case GQ_PACK_U8_SIGNPLANE: GQ_AGG(0, GQ_PACK_U8_SIGNPLANE); break;
        default: GQ_AGG(0, GQ_PACK_U4_SIGNPLANE); break;
        }
    } else {
        switch (p->pack) {
        case GQ_PACK_I8: GQ_AGG(1, GQ_PACK_I8); break;
        case GQ_PACK_I4: GQ_AGG(1, GQ_PACK_I4); break;
        case GQ_PACK_U8_SIGNPLANE: GQ_AGG(1, GQ_PACK_U8_SIGNPLANE); break;
        default: GQ_AGG(1, GQ_PACK_U4_SIGNPLANE); break;
        }
    }
#undef GQ_AGG
    return launched();
}

gq_status gq_dequantize(const void *agg, int64_t d, const float *norm, const gq_params *p, int K, float *out,
                        void *hip_stream)
{
    const gq_status st = check_params(p, false, true);
    if (st != GQ_OK) return st;
    if (K < 1 || K > GQ_MAX_WORKERS || d < 0 || !aligned(norm, 4)) return GQ_ERR_INVALID_ARG;
    if (d > 0 && (!aligned(agg, 16) || !aligned(out, 16))) return GQ_ERR_INVALID_ARG;
    if (d == 0) return GQ_OK;
    const int64_t nvec = (d + 3) / 4;
    const int64_t blocks = (nvec + kBlock - 1) / kBlock;
    if (!grid_fits(blocks, kBlock)) return GQ_ERR_INVALID_ARG;
    const dim3 grid((unsigned)blocks), block(kBlock);
    const float div = dequant_divisor(p, K);
    hipStream_t s = (hipStream_t)hip_stream;
    if (p->agg == GQ_AGG_I32)
        hipLaunchKernelGGL(dequantize_kernel<int>, grid, block, 0, s, (const int *)agg, d, norm, div, out);
    else
        hipLaunchKernelGGL(dequantize_kernel<short>, grid, block, 0, s, (const short *)agg, d, norm, div, out);
    return launched();
}

}  // extern "C"
