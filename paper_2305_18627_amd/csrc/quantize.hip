// Algorithm 1's quantisation loop (with its aggregation step fused in) on MI355X (gfx950): stochastic rounding of the gradients
// to integer codes, for one worker with the codes stored, or for all K workers with the integer sum
// formed in registers.  The contract of the entry points is stated in include/gqsgd.h.
//
// Data layout.  Every buffer is a flat array in HBM.  A lane owns vectors of four consecutive
// coordinates of a gradient (one 128-bit load per worker and vector), so that a wave reads 1 KiB of
// contiguous gradient per load.  With full draws (32 random bits per coordinate) a lane owns one
// vector, whose coordinates take the four words of one Philox call; with short draws (16 bits) it owns
// two vectors 64 apart and shares the words of its call with its neighbour lane.  All traffic is
// streaming with no reuse: nothing is staged through LDS.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include "gqsgd.h"
#include "gq_device.hpp"
#include "gq_host.hpp"

namespace gq {

// =============================================================================================
// Algorithm 1's quantisation loop and aggregation step fused: quantize the K workers' coordinates in registers, add the
// integer values, write the sum (and/or its dequantised mean, Eq. (1), and/or the packed codes).
//   SCHEME      0 linear, 1 exponential
//   KT          compile-time worker count (fully unrolled, K loads in flight), 0 = run-time K
//   LEVELS      also store every worker's packed codes
//   UNIFORM_HI  the high word of the Philox call index is the same for the whole launch
//   WINDOWS     keep few loads in flight per lane and store the sum only inside chip-wide time
//               windows (see below)
//   HALF        short draws: 16 random bits per coordinate, one Philox call per eight coordinates
// =============================================================================================
// OR over the 8 lanes that share one 32-bit sign word.  Every lane of the wave must be active.
__device__ __forceinline__ uint32_t or_over_8_lanes(uint32_t v)
{
    v |= dpp32<kDppQuadXor1>(v);
    v |= dpp32<kDppQuadXor2>(v);
    v |= dpp32<kDppHalfMirror>(v);
    return v;
}

// Store the codes of vector v (nvalid of its coordinates exist; the codes of the others are 0).  The lanes of a wave must
// hold consecutive vectors, lane 0 a multiple of 8, and all be active (the sign words are assembled across lanes).
template <int SCHEME>
__device__ __forceinline__ void store_codes(void *lv, uint32_t *sp, int pack, int64_t v, int nvalid, int64_t d, const Quad4<SCHEME> &q)
{
    if (pack >= 2) {
        const uint32_t word = or_over_8_lanes(q.sign_nibble() << (4 * (threadIdx.x & 7)));
        if ((threadIdx.x & 7) == 0 && ((v & ~(int64_t)7) << 2) < d) sp[v >> 3] = word;
    }
    if (nvalid == 0) return;
    if (pack == GQ_PACK_I8 || pack == GQ_PACK_U8_SIGNPLANE) {
        const uint32_t w = pack == GQ_PACK_I8 ? q.signed_bytes() : q.magnitude_bytes();
        if (nvalid == 4) {
            __builtin_nontemporal_store(w, reinterpret_cast<uint32_t *>(lv) + v);
        } else {
            uint8_t *b = reinterpret_cast<uint8_t *>(lv) + (v << 2);
            for (int i = 0; i < nvalid; i++) b[i] = (uint8_t)(w >> (8 * i));
        }
    } else {
        const uint32_t w = pack == GQ_PACK_I4 ? q.signed_nibbles() : q.magnitude_nibbles();
        if (nvalid == 4) {
            __builtin_nontemporal_store((uint16_t)w, reinterpret_cast<uint16_t *>(lv) + v);
        } else {
            uint8_t *b = reinterpret_cast<uint8_t *>(lv) + (v << 1);
            b[0] = (uint8_t)w;
            if (nvalid == 3) b[1] = (uint8_t)(w >> 8);
        }
    }
}

// Threads per workgroup of the fused kernel.  Small groups retire and refill wave slots at a finer
// grain, which measurably helps the HBM read/write mix of this kernel (128 and 64 alike, 256 slower on MI355X).
constexpr int kFusedBlock = 128;

// The integer sum of one lane's four coordinates: as floats, converted once, where the sum stays within 2^24 and is
// exact (every linear sum; exponential ones if the host says so), else as ints (exponential values reach 2^30).  A
// conversion less per worker and coordinate, and the cheaper rounding, take K = 32 at 50e6 coordinates (s = 7) from 1.08
// to 1.03 ms; with the codes stored, 25.6e6 x 8 (s = 16) goes from 0.212 to 0.190 ms.
template <bool FLOAT> struct Acc;
template <> struct Acc<true> {
    float a0 = 0.0f, a1 = 0.0f, a2 = 0.0f, a3 = 0.0f;
    __device__ __forceinline__ void add(float f0, float f1, float f2, float f3) { a0 += f0; a1 += f1; a2 += f2; a3 += f3; }
    __device__ __forceinline__ i32x4 get() const { return i32x4{(int)a0, (int)a1, (int)a2, (int)a3}; }
    __device__ __forceinline__ void pin() { asm volatile("" : "+v"(a0), "+v"(a1), "+v"(a2), "+v"(a3) : : "memory"); }
};
template <> struct Acc<false> {
    int a0 = 0, a1 = 0, a2 = 0, a3 = 0;
    __device__ __forceinline__ void add(float f0, float f1, float f2, float f3) { a0 += (int)f0; a1 += (int)f1; a2 += (int)f2; a3 += (int)f3; }
    __device__ __forceinline__ i32x4 get() const { return i32x4{a0, a1, a2, a3}; }
    __device__ __forceinline__ void pin() { asm volatile("" : "+v"(a0), "+v"(a1), "+v"(a2), "+v"(a3) : : "memory"); }
};

// Workgroups per compute unit (of 16) where the worker count is known at compile time, the draws are long and no windows
// separate reads and writes.  us without a limit / with it, in turn in one process: K = 4 linear, 41e6 coordinates 133.6 / 126, 110e6
// 361 / 339, exponential with 16-bit sum and mean 142 / 137, 393 / 372, with the sum alone 117.2 / 118.5, 314.1 / 314.6; K = 8 with the
// mean 281 / 267, 750 / 727, exponential with a 16-bit sum 260 / 250, 711 / 688.  K = 8 without the mean is equal, shorter
// launches lose (K = 4: 25.6e6 83 / 77 to 90, 6.5e6 21.7 / 23.1), so does K = 16 with its windows (110e6: 1168 / 1394), and
// short draws are equal.  Other worker counts run with the loop of run-time length and were not measured with a limit.
constexpr int64_t kFusedLimitFrom = 40000000;
template <int SCHEME, int KT, bool LEVELS, bool WINDOWS, bool HALF> static inline int fused_workgroups(int64_t coords, bool mean)
{
    if (LEVELS || WINDOWS || HALF || coords < kFusedLimitFrom) return 0;
    return KT == 4 ? (SCHEME == 0 ? 8 : 10) : (KT == 8 && mean ? 8 : 0);
}

// Launches whose time is latency rather than memory or issue.  At 6.5e6 coordinates the kernels of this file for short launches
// win and lose by 2 to 4 % (K = 1 9.5 / 9.1 us, K = 4 20.9 / 21.2, K = 32 148 / 153), with the codes stored they lose from 8e6 loads on
// (K = 8 at 1048576 coordinates 9.3 / 9.3, K = 16 17.6 / 18.4), at 41e6 they lose 4 to 13 %.
static inline bool short_launch(int K, int64_t d, bool levels) { return d <= 4194304 && (!levels || K * d <= 8388608); }

// Write windows.  The kernel reads 4K bytes and writes 4 bytes per coordinate.  With every wave storing
// whenever it happens to finish, HBM sees writes sprinkled evenly into the read stream and pays a bus
// turnaround for each; measured on MI355X this mix runs at 5.8-6.1 TB/s while the same reads alone
// reach 7 TB/s.  With WINDOWS a wave that has finished its sum waits (sleeping) until the constant
// 100 MHz counter, which all compute units share, enters the first tenth of a period of
// kWindowTicksPerWorker * K ticks, and stores then: the chip alternates between a long stretch of pure
// reads and a short burst of writes (6.3-6.5 TB/s for K >= 12).  The period is the time one
// generation of resident waves needs for its K loads, so a wave waits for about one window, not more.
// The wait is bounded (at most kWindowMaxPolls polls, a few periods even at K = 64) and touches no memory, so it
// changes timing only: if the counter did not advance, a wave would lose about 0.25 ms and go on.  For this
// to work the loads of a lane must really stay few in flight: the accumulators are pinned after each
// batch of four workers, which stops the compiler from hoisting all K loads to the top (it would
// otherwise, and with every load issued up front the windows were measured to gain nothing).
constexpr uint32_t kWindowTicksPerWorker = 62;    // ticks of the 100 MHz counter per worker and period
// The fewest workers for which the windows win, by the bytes written per coordinate: the more is written, the longer a burst
// and the more reads it takes to pay for the wait.  Windows on against off, 48e6 coordinates: 2 bytes K = 8 +1.1 %, 9 +2.4 %;
// 4 bytes K = 8 -0.8 % (110e6: +1.0), 9 +0.4, 10 +2.0; 6 bytes K = 9 -0.2, 10 +1.5, 12 +5.1; 8 bytes (32-bit sum and mean)
// K = 8 -2.6, 9 -3.2, 10 -2.8, 12 +2.3, 16 +3.7.  K = 8 with the mean in buckets of 67e6: 458 with, 438 us without where the
// gradients are rows of one allocation, 440 either way where each has its own; 22.4 such buckets with their norms 17.26 -> 16.95 ms.
constexpr int window_min_workers(int bytes) { return bytes <= 4 ? 8 : bytes <= 6 ? 10 : 12; }
constexpr double kWindowMinLoads = 2.5e8;         // K * d from which the windows win (measured)
constexpr int kWindowMaxPolls = 1024;             // polls of about 0.2 us each: the longest period (K = 64, short draws) is 79 us

// The sums and means of one vector of which nv > 0 coordinates exist; c = norm / (n * unit), Eq. (1).
__device__ __forceinline__ void store_sums(i32x4 a, int64_t v, int nv, float c, void *agg_out, int agg_fmt, float *deq_out)
{
    if (agg_out) {
        if (agg_fmt == GQ_AGG_I32) {
            if (nv == 4) {
                __builtin_nontemporal_store(a, reinterpret_cast<i32x4 *>(agg_out) + v);
            } else {
                int *o = reinterpret_cast<int *>(agg_out) + (v << 2);
                o[0] = a.x;
                if (nv > 1) o[1] = a.y;
                if (nv > 2) o[2] = a.z;
            }
        } else {
            if (nv == 4) {
                const i16x4 o = {(short)a.x, (short)a.y, (short)a.z, (short)a.w};
                __builtin_nontemporal_store(o, reinterpret_cast<i16x4 *>(agg_out) + v);
            } else {
                short *o = reinterpret_cast<short *>(agg_out) + (v << 2);
                o[0] = (short)a.x;
                if (nv > 1) o[1] = (short)a.y;
                if (nv > 2) o[2] = (short)a.z;
            }
        }
    }
    if (deq_out) {
        if (nv == 4) {
            const f32x4 o = {(float)a.x * c, (float)a.y * c, (float)a.z * c, (float)a.w * c};
            __builtin_nontemporal_store(o, reinterpret_cast<f32x4 *>(deq_out) + v);
        } else {
            float *o = deq_out + (v << 2);
            o[0] = (float)a.x * c;
            if (nv > 1) o[1] = (float)a.y * c;
            if (nv > 2) o[2] = (float)a.z * c;
        }
    }
}

// The launch covers the vectors v0 <= v < vend of the buffers (HALF: v0 = 0).  With UNIFORM_HI the host
// guarantees that the Philox call index does not cross a multiple of 2^32 inside the launch, so the high
// counter word is a scalar: the first round and half of the second are then shared by all lanes or all
// workers and leave the vector ALU.
template <int SCHEME, int KT, bool LEVELS, bool UNIFORM_HI, bool WINDOWS, bool HALF>
__global__ void __launch_bounds__(kFusedBlock)
quantize_aggregate_kernel(GradPtrsFor<KT> P, typename std::conditional<LEVELS, LevelPtrs, NoPtrs>::type L, int K, int64_t d, int64_t v0, int64_t vend, const float *__restrict__ norm, int s,
                          uint64_t seed, uint32_t worker0, uint64_t call_base, int pack,
                          void *__restrict__ agg_out, int agg_fmt, float *__restrict__ deq_out, float deq_div,
                          uint32_t win_period, uint32_t win_open)
{
    constexpr int NV = HALF ? 2 : 1;             // vectors per lane
    const int64_t nfull = d >> 2;
    const int lane = (int)(threadIdx.x & 63u);
    // the workgroup's first vector (scalar) and this lane's vectors relative to it: kept apart, so that an address is a
    // scalar base and a 32-bit lane offset and costs no vector instruction per worker
    const int64_t vb = v0 + (int64_t)blockIdx.x * (kFusedBlock * NV);
    uint32_t li[NV];
    uint64_t local_call;                         // call index of this lane relative to the launch's first
    if (HALF) {
        const uint64_t chunk = (uint64_t)blockIdx.x * (kFusedBlock / 64) + (threadIdx.x >> 6);   // 128 vectors per wave
        li[0] = (threadIdx.x >> 6) * 128u + (uint32_t)lane;
        li[NV - 1] = li[0] + 64u;
        local_call = chunk * 64u + (uint64_t)(lane >> 1) + (uint64_t)(lane & 1) * 32u;
    } else {
        li[0] = threadIdx.x;
        local_call = (uint64_t)blockIdx.x * kFusedBlock + threadIdx.x;
    }
    int64_t v[NV];
#pragma unroll
    for (int t = 0; t < NV; t++) v[t] = vb + li[t];
    int nvalid[NV];
#pragma unroll
    for (int t = 0; t < NV; t++) nvalid[t] = v[t] >= vend ? 0 : (v[t] < nfull ? 4 : (v[t] == nfull ? (int)(d & 3) : 0));
    // whole waves are needed by the sign-plane exchange (LEVELS) and by the exchange of short draws
    if (!LEVELS && !HALF && nvalid[0] == 0) return;

    const float nrm = *norm;
    const Scale sc = make_scale<SCHEME>(nrm, s);
    const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    const uint64_t first = call_base + (uint64_t)(HALF ? (v0 >> 1) : v0);      // scalar
    uint32_t c_lo, c_hi;
    if (UNIFORM_HI) {
        c_hi = (uint32_t)(first >> 32);
        c_lo = (uint32_t)first + (uint32_t)local_call;                            // fits and no carry (host)
    } else {
        const uint64_t call = first + local_call;
        c_lo = (uint32_t)call;
        c_hi = (uint32_t)(call >> 32);
    }
    const int Kc = KT > 0 ? KT : K;
    // every coordinate of the workgroup exists (uniform)
    const bool whole = vb + kFusedBlock * NV <= (vend < nfull ? vend : nfull);

    struct Unit { f32x4 g[NV]; };
    auto fetch = [&](int w) {
        Unit x;
#pragma unroll
        for (int t = 0; t < NV; t++) x.g[t] = load_coords(P.x[w], v[t], nvalid[t]);
        return x;
    };
    auto fetch_whole = [&](int w) {
        Unit x;
#pragma unroll
        for (int t = 0; t < NV; t++) x.g[t] = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(P.x[w]) + vb + li[t]);
        return x;
    };
    Acc<SCHEME == 0 || (KT > 0)> acc[NV];           // exponential with a compile-time K: the host checked the range
    auto one_worker = [&](int w, const Unit &x) {
        const Words4 r = philox4x32_10(c_lo, c_hi, worker0 + (uint32_t)w, 0u, k0, k1);
        uint32_t draw[NV][4];
        if (HALF) {
            const ShortDraws sd = share_short_draws(r, (lane & 1) != 0);
#pragma unroll
            for (int j = 0; j < 4; j++) { draw[0][j] = short_draw(sd.a, j); draw[NV - 1][j] = short_draw(sd.b, j); }
        } else {
#pragma unroll
            for (int j = 0; j < 4; j++) draw[0][j] = r.w[j];
        }
#pragma unroll
        for (int t = 0; t < NV; t++) {
            const Quad4<SCHEME> q(x.g[t], sc, draw[t]);
            acc[t].add(q.v[0], q.v[1], q.v[2], q.v[3]);
            if constexpr (LEVELS) store_codes<SCHEME>(L.lv[w], L.sp[w], pack, v[t], nvalid[t], d, q);
        }
    };
    if (KT > 0) {
        // workers whose loads are issued before the first is consumed: few with WINDOWS, else up to 16
        // vectors; the bound is enforced (accumulators pinned) where the hoisted loads would not fit
        constexpr int kMost = WINDOWS ? 4 : 16 / NV;
        constexpr bool kPin = WINDOWS || HALF;
        constexpr int kInFlight = KT > kMost ? kMost : (KT > 0 ? KT : 1);
#pragma unroll
        for (int w0 = 0; w0 < KT; w0 += kInFlight) {
            Unit x[kInFlight];
            if (whole) {                             // one branch per batch, not per worker
#pragma unroll
                for (int j = 0; j < kInFlight; j++) x[j] = fetch_whole(w0 + j);
            } else {
#pragma unroll
                for (int j = 0; j < kInFlight; j++) x[j] = fetch(w0 + j);
            }
#pragma unroll
            for (int j = 0; j < kInFlight; j++) one_worker(w0 + j, x[j]);
            if (kPin) {
#pragma unroll
                for (int t = 0; t < NV; t++) acc[t].pin();
            }
        }
    } else {
        int w = 0;
        for (; w + 4 <= Kc; w += 4) {
            Unit x0, x1, x2, x3;
            if (whole) { x0 = fetch_whole(w); x1 = fetch_whole(w + 1); x2 = fetch_whole(w + 2); x3 = fetch_whole(w + 3); }
            else { x0 = fetch(w); x1 = fetch(w + 1); x2 = fetch(w + 2); x3 = fetch(w + 3); }
            one_worker(w, x0); one_worker(w + 1, x1); one_worker(w + 2, x2); one_worker(w + 3, x3);
        }
        for (; w < Kc; w++) one_worker(w, fetch(w));
    }
    if (nvalid[0] == 0) return;

    if (WINDOWS) {
        for (int it = 0; it < kWindowMaxPolls; it++) {
            const uint32_t t = (uint32_t)__builtin_amdgcn_s_memrealtime();
            if ((t % win_period) < win_open) break;
            __builtin_amdgcn_s_sleep(8);
        }
    }
    const float c = sc.scale != 0.0f ? nrm / deq_div : 0.0f;
#pragma unroll
    for (int t = 0; t < NV; t++) {
        if (nvalid[t] == 0) break;
        store_sums(acc[t].get(), v[t], nvalid[t], c, agg_out, agg_fmt, deq_out);
    }
}

// Short launches.  Their time is latency: a workgroup has code of its own at the ragged end, so that neither the first worker's
// arithmetic waits for the loads of all workers nor the guarded loads wait for each other, as they do in the kernel above (two
// sets of loads beside a branch: one wait for all behind it, and one between any two guarded ones).  us a call, above / here:
//   100003 coordinates   linear K = 4 3.0 / 2.4, 8 4.45 / 3.25, 16 7.3 / 4.9, 32 11.0 / 8.2;  exponential 3.1 / 2.5, 4.7 / 3.4, 7.6 / 5.1, 12.3 / 8.6;
//                        short draws, linear 3.8 / 3.1, 5.7 / 4.35, 9.9 / 7.1, 18.3 / 12.7;  int8 codes stored 4.4 / 3.7, 7.1 / 5.6 (K = 4, 8)
//   1048576 coordinates  linear 4.55 / 4.35, 7.55 / 6.8, 14.8 / 13.3, 29.9 / 26.7;  short draws 4.85 / 4.5, 8.2 / 6.95, 13.5 / 11.5, 25.1 / 23.75
// WHOLE: every vector of the workgroup exists and nothing is guarded; else the loads are clamped.  The early return and the
// __restrict__ are needed: without either the scheduler draws the random words of all workers first, in up to 290 registers.
template <int SCHEME, int KT, bool LEVELS, bool HALF, bool WHOLE>
__device__ __forceinline__ void
quantize_aggregate_short_block(const GradPtrsFor<KT> &P, const typename std::conditional<LEVELS, LevelPtrs, NoPtrs>::type &L, int K, int64_t d, int64_t vb,
                               const float *__restrict__ norm, int s, uint64_t seed, uint32_t worker0, uint64_t call_base, int pack, void *__restrict__ agg_out, int agg_fmt, float *__restrict__ deq_out,
                               float deq_div)
{
    constexpr int NV = HALF ? 2 : 1;             // vectors per lane
    const int64_t nfull = d >> 2;
    const int lane = (int)(threadIdx.x & 63u);
    uint32_t li[NV], local_call;                 // this lane's vectors and its call index relative to the workgroup's first
    if (HALF) {
        li[0] = (threadIdx.x >> 6) * 128u + (uint32_t)lane;
        li[NV - 1] = li[0] + 64u;
        local_call = (threadIdx.x >> 6) * 64u + (uint32_t)(lane >> 1) + (uint32_t)(lane & 1) * 32u;
    } else {
        local_call = li[0] = threadIdx.x;
    }
    int64_t v[NV];
    int nvalid[NV];
#pragma unroll
    for (int t = 0; t < NV; t++) {
        v[t] = vb + li[t];
        nvalid[t] = WHOLE || v[t] < nfull ? 4 : (v[t] == nfull ? (int)(d & 3) : 0);
    }
    if (!LEVELS && !HALF && nvalid[0] == 0) return;
    const uint32_t last = WHOLE ? 0u : last_coord(vb, d);
    const float nrm = *norm;
    const Scale sc = make_scale<SCHEME>(nrm, s);
    const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    const uint64_t first = call_base + (uint64_t)(HALF ? vb >> 1 : vb);           // scalar
    const uint32_t c_hi = (uint32_t)(first >> 32), c_lo = (uint32_t)first + local_call;     // no carry (host)
    const int Kc = KT > 0 ? KT : K;

    struct Unit { f32x4 g[NV]; };
    auto fetch = [&](int w) {
        Unit x;
#pragma unroll
        for (int t = 0; t < NV; t++) {
            if (WHOLE) x.g[t] = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(P.x[w]) + vb + li[t]);
            else x.g[t] = load_clamped(P.x[w] + (vb << 2), li[t], last);
        }
        return x;
    };
    Acc<SCHEME == 0 || (KT > 0)> acc[NV];           // exponential with a compile-time K: the host checked the range
    auto one_worker = [&](int w, const Unit &x) {
        // the scalar products of the first rounds take longer than the vector unit's where few waves hide them
        const Words4 r = philox4x32_10<false>(c_lo, c_hi, worker0 + (uint32_t)w, 0u, k0, k1);
        uint32_t draw[NV][4];
        if (HALF) {
            const ShortDraws sd = share_short_draws(r, (lane & 1) != 0);
#pragma unroll
            for (int j = 0; j < 4; j++) { draw[0][j] = short_draw(sd.a, j); draw[NV - 1][j] = short_draw(sd.b, j); }
        } else {
#pragma unroll
            for (int j = 0; j < 4; j++) draw[0][j] = r.w[j];
        }
#pragma unroll
        for (int t = 0; t < NV; t++) {
            const Quad4<SCHEME> q(LEVELS && !WHOLE ? existing(x.g[t], li[t], last) : x.g[t], sc, draw[t]);
            acc[t].add(q.v[0], q.v[1], q.v[2], q.v[3]);
            if constexpr (LEVELS) store_codes<SCHEME>(L.lv[w], L.sp[w], pack, v[t], nvalid[t], d, q);
        }
    };
    // batches whose loads are all issued before the first is consumed
    constexpr int kBatch = KT == 0 ? (HALF && !WHOLE ? 2 : 4) : (KT < 16 / NV ? KT : 16 / NV);
    if (KT > 0) {
#pragma unroll
        for (int w0 = 0; w0 < KT; w0 += kBatch) {
            Unit x[kBatch];
#pragma unroll
            for (int j = 0; j < kBatch; j++) x[j] = fetch(w0 + j);
            if (!WHOLE) all_asked_for();
#pragma unroll
            for (int j = 0; j < kBatch; j++) one_worker(w0 + j, x[j]);
            if (HALF) {                              // bounds the loads in flight to one batch
#pragma unroll
                for (int t = 0; t < NV; t++) acc[t].pin();
            }
        }
    } else {
        int w = 0;
        for (; w + kBatch <= Kc; w += kBatch) {
            Unit x[kBatch];
#pragma unroll
            for (int j = 0; j < kBatch; j++) x[j] = fetch(w + j);
            if (!WHOLE) all_asked_for();
#pragma unroll
            for (int j = 0; j < kBatch; j++) one_worker(w + j, x[j]);
        }
        for (; w < Kc; w++) one_worker(w, fetch(w));
    }
    if (nvalid[0] == 0) return;
    const float c = sc.scale != 0.0f ? nrm / deq_div : 0.0f;
#pragma unroll
    for (int t = 0; t < NV; t++) {
        if (nvalid[t] == 0) break;
        store_sums(acc[t].get(), v[t], nvalid[t], c, agg_out, agg_fmt, deq_out);
    }
}

template <int SCHEME, int KT, bool LEVELS, bool HALF>
__global__ void __launch_bounds__(kFusedBlock)
quantize_aggregate_short_kernel(GradPtrsFor<KT> P, typename std::conditional<LEVELS, LevelPtrs, NoPtrs>::type L, int K, int64_t d, const float *__restrict__ norm, int s,
                                uint64_t seed, uint32_t worker0, uint64_t call_base, int pack, void *__restrict__ agg_out, int agg_fmt, float *__restrict__ deq_out, float deq_div)
{
    constexpr int kBlockVecs = kFusedBlock * (HALF ? 2 : 1);
    const int64_t vb = (int64_t)blockIdx.x * kBlockVecs;                     // scalar
    if (vb + kBlockVecs <= (d >> 2))                                        // uniform over the workgroup
        quantize_aggregate_short_block<SCHEME, KT, LEVELS, HALF, true>(P, L, K, d, vb, norm, s, seed, worker0, call_base, pack, agg_out, agg_fmt, deq_out, deq_div);
    else
        quantize_aggregate_short_block<SCHEME, KT, LEVELS, HALF, false>(P, L, K, d, vb, norm, s, seed, worker0, call_base, pack, agg_out, agg_fmt, deq_out, deq_div);
}

// =============================================================================================
// Algorithm 1's quantisation loop for one worker with the codes stored: a lane owns kQuantVec vectors of four
// coordinates, kQuantBlock vectors apart (short draws: two pairs 64 apart, see share_short_draws), and
// issues all its loads before the first Philox call.
// =============================================================================================
constexpr int kQuantBlock = 128;
constexpr int kQuantVec = 4;

// The work of one workgroup.  WHOLE: its kQuantBlock * kQuantVec vectors all lie inside the buffer; the loads
// need no guards and the code words are staged in LDS and written out as one run, 16 (bytes) or 8 (nibbles)
// bytes per thread, instead of four narrow stores per thread.  Otherwise (the ragged last workgroup) every
// vector is guarded and stored on its own.
// PACK: the format, or kRunTimePack.  Short launches, whose time is latency, know it at compile time and clamp the loads of the
// ragged workgroup instead of guarding them: four calls of 100003 coordinates, 4 bits + planes 13.3 -> 11.7 us, exponential int4
// 12.9 -> 11.5, short draws 11.5 -> 10.2.  Long ones pick it as they run: that is equal, or up to 4 % faster (linear 8 bits +
// planes, 4 x 67e6: 227 us, 236 with the format known).
constexpr int kRunTimePack = -1;
template <int SCHEME, int PACK, bool UNIFORM_HI, bool HALF, bool WHOLE>
__device__ __forceinline__ void quantize_block(const float *__restrict__ x, void *__restrict__ lv, uint32_t *__restrict__ sp,
                                               int64_t d, const Scale &sc, uint64_t seed, uint32_t worker,
                                               uint64_t call_base, int run_time_pack, uint32_t *stage, uint32_t *stage_signs)
{
    constexpr int kBlockVecs = kQuantBlock * kQuantVec;
    const int pack = PACK == kRunTimePack ? run_time_pack : PACK;
    const int64_t nfull = d >> 2;
    const int lane = (int)(threadIdx.x & 63u);
    const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    const int64_t vblock = (int64_t)blockIdx.x * kBlockVecs;          // scalar
    // vector j of this lane within the workgroup, and the Philox call (relative to the workgroup's first) that
    // it runs for vectors j, j+1 (short draws) or j (full draws)
    uint32_t li[kQuantVec];
    uint32_t lcall[kQuantVec];
#pragma unroll
    for (int j = 0; j < kQuantVec; j++) {
        if (HALF) {
            // the workgroup's 512 vectors are four chunks of 128; wave w takes chunks w and w + 2
            const uint32_t chunk = (threadIdx.x >> 6) + 2 * (j >> 1);
            li[j] = chunk * 128 + 64 * (j & 1) + (uint32_t)lane;
            lcall[j] = chunk * 64 + (uint32_t)(lane >> 1) + (uint32_t)(lane & 1) * 32;
        } else {
            li[j] = j * kQuantBlock + threadIdx.x;
            lcall[j] = li[j];
        }
    }
    const float *xb = x + (vblock << 2);
    f32x4 g[kQuantVec];
    int nvalid[kQuantVec];
#pragma unroll
    for (int j = 0; j < kQuantVec; j++) {
        if (WHOLE) {
            nvalid[j] = 4;
            g[j] = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(xb) + li[j]);
        } else {
            const int64_t v = vblock + li[j];
            nvalid[j] = v < nfull ? 4 : (v == nfull ? (int)(d & 3) : 0);
            g[j] = PACK == kRunTimePack ? load_coords(x, v, nvalid[j]) : load_clamped(xb, li[j], last_coord(vblock, d));
        }
    }
    if (!WHOLE && PACK != kRunTimePack) {
        all_asked_for();
#pragma unroll
        for (int j = 0; j < kQuantVec; j++) g[j] = existing(g[j], li[j], last_coord(vblock, d));
    }
    const uint64_t first = call_base + (uint64_t)(HALF ? (vblock >> 1) : vblock);    // scalar
    auto counter = [&](uint32_t c, uint32_t &c_lo, uint32_t &c_hi) {
        if (UNIFORM_HI) {                             // host: the launch stays below the next multiple of 2^32 calls
            c_hi = (uint32_t)(first >> 32);
            c_lo = (uint32_t)first + c;
        } else {
            const uint64_t cc = first + (uint64_t)c;
            c_lo = (uint32_t)cc;
            c_hi = (uint32_t)(cc >> 32);
        }
    };
    const bool bytes = pack == GQ_PACK_I8 || pack == GQ_PACK_U8_SIGNPLANE;
    auto emit = [&](int j, const uint32_t *draw) {
        const Quad4<SCHEME> q(g[j], sc, draw);
        if (!WHOLE) {
            store_codes<SCHEME>(lv, sp, pack, vblock + li[j], nvalid[j], d, q);
            return;
        }
        if (pack >= 2) {
            const uint32_t word = or_over_8_lanes(q.sign_nibble() << (4 * (threadIdx.x & 7)));
            if ((threadIdx.x & 7) == 0) stage_signs[li[j] >> 3] = word;
        }
        if (pack == GQ_PACK_I8) stage[li[j]] = q.signed_bytes();
        else if (pack == GQ_PACK_U8_SIGNPLANE) stage[li[j]] = q.magnitude_bytes();
        else reinterpret_cast<uint16_t *>(stage)[li[j]] = (uint16_t)(pack == GQ_PACK_I4 ? q.signed_nibbles() : q.magnitude_nibbles());
    };
    // no lane leaves early: the sign-plane exchange and the exchange of short draws need whole waves
    if (HALF) {
#pragma unroll
        for (int j = 0; j < kQuantVec; j += 2) {
            uint32_t c_lo, c_hi;
            counter(lcall[j], c_lo, c_hi);
            const ShortDraws sd = share_short_draws(philox4x32_10(c_lo, c_hi, worker, 0u, k0, k1), (lane & 1) != 0);
            uint32_t da[4], db[4];
#pragma unroll
            for (int i = 0; i < 4; i++) { da[i] = short_draw(sd.a, i); db[i] = short_draw(sd.b, i); }
            emit(j, da);
            emit(j + 1, db);
        }
    } else {
#pragma unroll
        for (int j = 0; j < kQuantVec; j++) {
            uint32_t c_lo, c_hi;
            counter(lcall[j], c_lo, c_hi);
            const Words4 r = philox4x32_10(c_lo, c_hi, worker, 0u, k0, k1);
            emit(j, r.w);
        }
    }
    if (WHOLE) {
        __syncthreads();
        const int t = (int)threadIdx.x;
        if (bytes) {
            const u32x4 w = *reinterpret_cast<const u32x4 *>(&stage[4 * t]);
            __builtin_nontemporal_store(w, reinterpret_cast<u32x4 *>(lv) + (vblock / 4 + t));
        } else {
            const uint64_t w = *reinterpret_cast<const uint64_t *>(reinterpret_cast<const uint16_t *>(stage) + 4 * t);
            __builtin_nontemporal_store(w, reinterpret_cast<uint64_t *>(lv) + (vblock / 4 + t));
        }
        if (pack >= 2 && t < kBlockVecs / 8) sp[vblock / 8 + t] = stage_signs[t];
    }
}

template <int SCHEME, int PACK, bool UNIFORM_HI, bool HALF>
__global__ void __launch_bounds__(kQuantBlock)
quantize_kernel(const float *__restrict__ x, void *__restrict__ lv, uint32_t *__restrict__ sp, int64_t d,
                const float *__restrict__ norm, int s, uint64_t seed, uint32_t worker, uint64_t call_base, int pack)
{
    __shared__ uint32_t stage[kQuantBlock * kQuantVec];              // one code word per vector
    __shared__ uint32_t stage_signs[kQuantBlock * kQuantVec / 8];    // one sign word per 8 vectors
    const Scale sc = make_scale<SCHEME>(*norm, s);
    const bool whole = ((int64_t)blockIdx.x + 1) * (kQuantBlock * kQuantVec) <= (d >> 2);   // uniform over the workgroup
    if (whole) quantize_block<SCHEME, PACK, UNIFORM_HI, HALF, true>(x, lv, sp, d, sc, seed, worker, call_base, pack, stage, stage_signs);
    else quantize_block<SCHEME, PACK, UNIFORM_HI, HALF, false>(x, lv, sp, d, sc, seed, worker, call_base, pack, stage, stage_signs);
}

// Workgroups per compute unit (of 16) in launches of at least kQuantLimitFrom coordinates: fewer where memory and not
// arithmetic is the bound, which in the middle of other calls, with the chip's clock up, is the whole linear grid.  Shorter
// launches lose by their last wave of workgroups (6.5e6: 5 %).  Four calls of 110e6 coordinates between a norm pass and an integer
// sum, us without a limit / with 12; the four calls in a loop of their own:
//   linear  int8 757 / 754.5, 351 / 346;  int4 693 / 681, 316 / 310;  8 bits + planes 819 / 814, 356 / 346;  4 bits + planes 706 / 689, 316 / 333
//   exponential, 8 bits + planes  844 / 825, 358 / 381;  its other formats only lose (with 14: int4 684 / 676, 334 / 346;  4 bits + planes 794 / 790,
//   347 / 358;  int8 equal, 349 / 359)
// Again, in turn in one process: four calls of 110e6 between norm and sum, eight of 67e6, four of 110e6 in a loop: 4 bits + planes
// 729 / 705, 838 / 818, 326 / 342;  exponential, 8 bits + planes 855 / 840, 949 / 932, 361 / 383.  These two formats pay 5 to 6 % where
// a caller only encodes and gain 2 to 3 % where it takes the norm and the sum as well, which is what the codes are for.
constexpr int64_t kQuantLimitFrom = 50000000;
static inline int quantize_workgroups(const gq_params *p, int64_t d)
{
    return d >= kQuantLimitFrom && (p->scheme == GQ_LINEAR || p->pack == GQ_PACK_U8_SIGNPLANE) ? 12 : 0;
}

template <bool LEVELS> static inline typename std::conditional<LEVELS, const LevelPtrs &, NoPtrs>::type level_ptrs(const LevelPtrs &L)
{
    if constexpr (LEVELS) return L;
    else return NoPtrs{};
}

template <int SCHEME, bool HALF>
static gq_status launch_quantize_aggregate(const GradPtrs &P, const LevelPtrs &L, bool levels, int K, int64_t d,
                                           const float *norm, const gq_params *p, uint32_t worker0,
                                           int64_t index_base, void *agg_out, float *deq_out, hipStream_t st)
{
    constexpr int kLaneVecs = HALF ? 2 : 1;              // vectors per lane = vectors per Philox call
    const int64_t nvec = (d + 3) / 4;
    const uint64_t call_base = (uint64_t)index_base / (uint64_t)(4 * kLaneVecs);
    const float div = dequant_divisor(p, K);
    const dim3 block(kFusedBlock);
    // Write windows pay once a launch lasts many periods and a wave's K loads span about one period;
    // below these sizes the wait for the next window costs more than the cleaner read/write mix gains.
    // The caller may override the policy either way (gq_params.flags).
    const int out_bytes = (agg_out ? (p->agg == GQ_AGG_I16 ? 2 : 4) : 0) + (deq_out ? 4 : 0);
    const bool by_policy = K >= window_min_workers(out_bytes) && (double)K * (double)d >= kWindowMinLoads;
    const bool win = !levels && !(p->flags & GQ_FLAG_WRITE_WINDOWS_OFF) && (by_policy || (p->flags & GQ_FLAG_WRITE_WINDOWS_ON));
    const uint32_t win_period = kWindowTicksPerWorker * (uint32_t)K * (uint32_t)kLaneVecs;   // a wave loads kLaneVecs KiB per worker
    const uint32_t win_open = win_period / 10u;
#define GQ_LAUNCH(KT, LV, UH, WIN, V0, COUNT)                                                                  \
    do {                                                                                                      \
        const int64_t blocks_ = ((COUNT) + kFusedBlock * kLaneVecs - 1) / (kFusedBlock * kLaneVecs);          \
        if (!grid_fits(blocks_, kFusedBlock)) return GQ_ERR_INVALID_ARG;                                                   \
        hipLaunchKernelGGL((quantize_aggregate_kernel<SCHEME, KT, LV, UH, WIN, HALF>), dim3((unsigned)blocks_), block, lds_for_workgroups(fused_workgroups<SCHEME, KT, LV, WIN, HALF>((COUNT) * 4, deq_out != nullptr), 0), st, \
                           pointers_for<KT>(P), level_ptrs<LV>(L), K, d, (int64_t)(V0), (int64_t)(V0) + (int64_t)(COUNT), norm, p->s, p->seed, worker0,  \
                           call_base, p->pack, agg_out, p->agg, deq_out, div, win_period, win_open);          \
    } while (0)
    // the kernels with a compile-time worker count sum as floats: exponential sums beyond 2^24 take the general one
    const bool float_sum = max_aggregate(p, K) <= ((int64_t)1 << 24);
#define GQ_LAUNCH_K(UH, WIN, V0, COUNT)                                                                        \
    do {                                                                                                      \
        if (!float_sum) GQ_LAUNCH(0, false, UH, WIN, V0, COUNT);                                              \
        else if (K == 4) GQ_LAUNCH(4, false, UH, WIN, V0, COUNT);                                                  \
        else if (K == 8) GQ_LAUNCH(8, false, UH, WIN, V0, COUNT);                                             \
        else if (K == 16) GQ_LAUNCH(16, false, UH, WIN, V0, COUNT);                                           \
        else if (K == 32) GQ_LAUNCH(32, false, UH, WIN, V0, COUNT);                                           \
        else GQ_LAUNCH(0, false, UH, WIN, V0, COUNT);                                                         \
    } while (0)
    // calls of the launch, counting the lanes past the end of whole workgroups
    const uint64_t calls_padded = (uint64_t)((nvec + kFusedBlock * kLaneVecs - 1) / (kFusedBlock * kLaneVecs)) * kFusedBlock;
    const bool one_stretch = ((call_base & 0xFFFFFFFFull) + calls_padded) <= ((uint64_t)1 << 32);
    if (one_stretch && !win && short_launch(K, d, levels) && !(HALF && levels)) {
        const int64_t blocks = (nvec + kFusedBlock * kLaneVecs - 1) / (kFusedBlock * kLaneVecs);
#define GQ_SHORT(KT, LV) hipLaunchKernelGGL((quantize_aggregate_short_kernel<SCHEME, KT, LV, HALF>), dim3((unsigned)blocks), block, 0, st, pointers_for<KT>(P), \
                                            level_ptrs<LV>(L), K, d, norm, p->s, p->seed, worker0, call_base, p->pack, agg_out, p->agg, deq_out, div)
        if constexpr (!HALF) {
            if (levels) { GQ_SHORT(0, true); return launched(); }
        }
        if (!float_sum) GQ_SHORT(0, false);
        else if (K == 4) GQ_SHORT(4, false);
        else if (K == 8) GQ_SHORT(8, false);
        else if (K == 16) GQ_SHORT(16, false);
        else if (K == 32) GQ_SHORT(32, false);
        else GQ_SHORT(0, false);
#undef GQ_SHORT
        return launched();
    }
    if (levels) {
        // storing codes: one launch; the scalar high word is used when the bucket does not cross 2^32 calls
        if (one_stretch) GQ_LAUNCH(0, true, true, false, 0, nvec);
        else GQ_LAUNCH(0, true, false, false, 0, nvec);
        return launched();
    }
    if (HALF) {
        // short draws pair the lanes of a wave, so the launch is not cut: a bucket that crosses a multiple
        // of 2^32 calls (2^35 coordinates) runs with the high counter word per lane
        if (one_stretch) { if (win) GQ_LAUNCH_K(true, true, 0, nvec); else GQ_LAUNCH_K(true, false, 0, nvec); }
        else             { if (win) GQ_LAUNCH_K(false, true, 0, nvec); else GQ_LAUNCH_K(false, false, 0, nvec); }
        return launched();
    }
    constexpr int64_t kMaxLaunchVecs = (int64_t)1 << 31;
    // One launch per stretch of vectors whose Philox call index shares its high 32 bits (a second
    // stretch exists only if the bucket crosses a multiple of 2^34 coordinates).
    int64_t v0 = 0;
    while (v0 < nvec) {
        const uint64_t first = call_base + (uint64_t)v0;
        const uint64_t room = ((uint64_t)1 << 32) - (first & 0xFFFFFFFFull);
        int64_t count = (uint64_t)(nvec - v0) < room ? (nvec - v0) : (int64_t)room;
        if (count > kMaxLaunchVecs) count = kMaxLaunchVecs;       // and no launch beyond HIP's limit of 2^32 - 1 threads
        if (win) GQ_LAUNCH_K(true, true, v0, count);
        else GQ_LAUNCH_K(true, false, v0, count);
        if (launched() != GQ_OK) return GQ_ERR_DEVICE;
        v0 += count;
    }
#undef GQ_LAUNCH_K
#undef GQ_LAUNCH
    return GQ_OK;
}

}  // namespace gq

using namespace gq;

extern "C" {

gq_status gq_quantize(const float *x, int64_t d, const float *norm, const gq_params *p, uint32_t worker,
                      int64_t index_base, void *levels_out, uint32_t *signplane_out, void *hip_stream)
{
    const gq_status st = check_params(p, true, false);
    if (st != GQ_OK) return st;
    const bool half = short_draws(p);
    if (d < 0 || index_base < 0 || (index_base & (half ? 7 : 3)) != 0) return GQ_ERR_INVALID_ARG;
    if (!aligned(norm, 4)) return GQ_ERR_INVALID_ARG;
    const bool plane = p->pack >= GQ_PACK_U8_SIGNPLANE;
    if (d > 0 && (!aligned(x, 16) || !aligned(levels_out, 16))) return GQ_ERR_INVALID_ARG;
    if (d > 0 && plane && !aligned(signplane_out, 4)) return GQ_ERR_INVALID_ARG;
    if (d == 0) return GQ_OK;
    const int64_t nvec = (d + 3) / 4;
    const int64_t per_block = (int64_t)kQuantBlock * kQuantVec;          // vectors per workgroup, either mode
    const int64_t blocks = (nvec + per_block - 1) / per_block;
    if (!grid_fits(blocks, kQuantBlock)) return GQ_ERR_INVALID_ARG;
    const dim3 grid((unsigned)blocks), block(kQuantBlock);
    const int lane_vecs = half ? 2 : 1;                                  // vectors per Philox call
    const uint64_t call_base = (uint64_t)index_base / (uint64_t)(4 * lane_vecs);
    // the high counter word is a scalar unless the bucket (rounded up to whole blocks) crosses 2^32 calls
    const bool one_stretch = ((call_base & 0xFFFFFFFFull) + (uint64_t)(blocks * per_block / lane_vecs)) <= ((uint64_t)1 << 32);
    uint32_t *sp = plane ? signplane_out : nullptr;
    hipStream_t st2 = (hipStream_t)hip_stream;
    const unsigned lds = lds_for_workgroups(quantize_workgroups(p, d), kQuantBlock * kQuantVec * 4 + kQuantBlock * kQuantVec / 2);
#define GQ_QUANT(SC, PK, UH, HF) hipLaunchKernelGGL((quantize_kernel<SC, PK, UH, HF>), grid, block, lds, st2, x, levels_out, sp, d, norm, \
                                                    p->s, p->seed, worker, call_base, p->pack)
#define GQ_QUANT2(SC, PK, UH) do { if (half) GQ_QUANT(SC, PK, UH, true); else GQ_QUANT(SC, PK, UH, false); } while (0)
#define GQ_QUANT3(PK, UH) do { if (p->scheme == GQ_LINEAR) GQ_QUANT2(0, PK, UH); else GQ_QUANT2(1, PK, UH); } while (0)
    if (one_stretch && short_launch(1, d, false)) {
        switch (p->pack) {
        case GQ_PACK_I8: GQ_QUANT3(GQ_PACK_I8, true); break;
        case GQ_PACK_I4: GQ_QUANT3(GQ_PACK_I4, true); break;
        case GQ_PACK_U8_SIGNPLANE: GQ_QUANT3(GQ_PACK_U8_SIGNPLANE, true); break;
        default: GQ_QUANT3(GQ_PACK_U4_SIGNPLANE, true); break;
        }
    } else if (one_stretch) {
        GQ_QUANT3(kRunTimePack, true);
    } else {
        GQ_QUANT3(kRunTimePack, false);
    }
#undef GQ_QUANT3
#undef GQ_QUANT2
#undef GQ_QUANT
    return launched();
}

gq_status gq_fused_quantize_aggregate(const float *const *x, int K, int64_t d, const float *norm, const gq_params *p,
                                      int64_t index_base, void *agg_out, float *dequant_out,
                                      void *const *levels_out, uint32_t *const *signplanes_out, void *hip_stream)
{
    const bool levels = levels_out != nullptr;
    gq_status st = check_params(p, levels, agg_out != nullptr);
    if (st != GQ_OK) return st;
    const bool half = short_draws(p);
    if (!x || K < 1 || K > GQ_MAX_WORKERS || d < 0 || index_base < 0 || (index_base & (half ? 7 : 3)) != 0) return GQ_ERR_INVALID_ARG;
    if (!agg_out && !dequant_out) return GQ_ERR_INVALID_ARG;
    if (!aligned(norm, 4)) return GQ_ERR_INVALID_ARG;
    // the sum is formed in 32-bit registers whatever is stored; a 16-bit store must also hold it
    const int64_t lim = (agg_out && p->agg == GQ_AGG_I16) ? 32767LL : 2147483647LL;
    if (max_aggregate(p, K) > lim) return GQ_ERR_OVERFLOW;
    const bool plane = levels && p->pack >= GQ_PACK_U8_SIGNPLANE;
    if (plane && !signplanes_out) return GQ_ERR_INVALID_ARG;
    GradPtrs P;
    LevelPtrs L;
    for (int i = 0; i < K; i++) {
        if (d > 0 && !aligned(x[i], 16)) return GQ_ERR_INVALID_ARG;
        P.x[i] = x[i];
        if (levels) {
            L.sp[i] = nullptr;
            if (d > 0 && !aligned(levels_out[i], 16)) return GQ_ERR_INVALID_ARG;
            L.lv[i] = levels_out[i];
            if (plane) {
                if (d > 0 && !aligned(signplanes_out[i], 4)) return GQ_ERR_INVALID_ARG;
                L.sp[i] = signplanes_out[i];
            }
        }
    }
    if (d > 0 && ((agg_out && !aligned(agg_out, 16)) || (dequant_out && !aligned(dequant_out, 16)))) return GQ_ERR_INVALID_ARG;
    if (d == 0) return GQ_OK;
    hipStream_t hs = (hipStream_t)hip_stream;
    if (p->scheme == GQ_LINEAR) {
        if (half) return launch_quantize_aggregate<0, true>(P, L, levels, K, d, norm, p, 0u, index_base, agg_out, dequant_out, hs);
        return launch_quantize_aggregate<0, false>(P, L, levels, K, d, norm, p, 0u, index_base, agg_out, dequant_out, hs);
    }
    if (half) return launch_quantize_aggregate<1, true>(P, L, levels, K, d, norm, p, 0u, index_base, agg_out, dequant_out, hs);
    return launch_quantize_aggregate<1, false>(P, L, levels, K, d, norm, p, 0u, index_base, agg_out, dequant_out, hs);
}

}  // extern "C"
