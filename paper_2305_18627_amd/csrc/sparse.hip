// Algorithm 1's sparse branch on MI355X (gfx950): compaction of non-zero codes and the sum of the K lists.
// Contracts: include/gqsgd.h.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include "gqsgd.h"
#include "gq_device.hpp"
#include "gq_host.hpp"

namespace gq {

// =============================================================================================
// Algorithm 1's sparse branch.  Sender side: the (index, code) pairs of a worker's non-zero int8 codes in
// increasing index order, in one pass over the codes (every workgroup learns its place in the list from the
// counts the workgroups before it publish; the non-zeros inside a workgroup's span are ranked with wave scans).
// Receiver side: the K sorted lists are added span by span into the dense int32 sum.
// =============================================================================================
constexpr int kCompactTile = 4096;                      // codes per entry of the table of tile starts
constexpr int kWordSpan = 32768;                        // codes per 64-bit word of the scan
constexpr int kCell = 1024;                             // codes in a row that one wave owns; the granularity of the counts inside a span
constexpr int kRow = 512;                               // codes whose entries a wave ranks and copies out at a time
constexpr int kCompactWaves = 8;                        // waves per workgroup
constexpr int kStage = kCompactWaves * kRow;            // entries that a workgroup can stage
constexpr int kMaxSpan = kWordSpan;
// Scalar registers of gq_compact's kernel, so that eight waves fit on a SIMD (800 for all, handed out in steps of 16, and 16 more to
// each wave for the trap handler).  With the 87 that help would take, every call is 5 to 12 % slower.  Against no help at all
// it is equal, but for the longest gradients (300e6: 0.2 % non-zeros 82.9 / 84.8 us, 3 % 89.5 / 94.7).
constexpr int kCompactScalars = 82;

// A workgroup's span of SPAN codes: cell k of it belongs to wave k mod kCompactWaves.
template <int SPAN> struct Geometry {
    static constexpr int kSpanCells = SPAN / kCell;
    static constexpr int kWaveCells = kSpanCells / kCompactWaves;
    static constexpr int kPerWord = kWordSpan / SPAN;               // spans that share a 64-bit word of the scan
    static constexpr int kFieldBits = 64 / kPerWord;
    typedef typename std::conditional<kPerWord == 1, uint64_t, uint32_t>::type Field;
    static constexpr Field kPublished = (Field)1 << (kFieldBits - 1);
    static_assert(kPerWord <= 2 && kWaveCells >= 1, "fields of 32 or 64 bits, at least one cell per wave");
};

__device__ __forceinline__ uint32_t nonzero_bytes(uint32_t x)    // 0x80 in every byte of x that is not zero
{
    return (x | ((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu)) & 0x80808080u;
}

// the 8 codes of unit t (bytes 8t .. 8t+7), zeros past the end of the buffer
__device__ __forceinline__ u32x2 load_code_unit(const uint8_t *lv, int64_t t, int64_t d)
{
    const int64_t first = t << 3;
    if (first + 8 <= d) return __builtin_nontemporal_load(reinterpret_cast<const u32x2 *>(lv) + t);
    uint32_t q[2] = {0u, 0u};
    for (int i = 0; i < 8 && first + i < d; i++) q[i >> 2] |= (uint32_t)lv[first + i] << (8 * (i & 3));
    return u32x2{q[0], q[1]};
}

// ---------------------------------------------------------------------------------------------------------
// Sender side in ONE pass over the codes: a block counts the non-zeros of its span, learns how many lie before
// the span from the counts the blocks before it have published, and writes its pairs.  The codes are read once
// and nothing but the list is written: d + 5 * nnz bytes, the method's own traffic.
//
// A 64-bit word belongs to every kWordSpan codes; a workgroup's span is all of that or half (span_size), and then
// two spans share the word, a 32-bit field each.  64 words make a group, which has a word of its own.  Plain stores and
// loads throughout: read-modify-write atomics on one address serialise chip-wide at about 20 ns each (adding the
// counts of a group into its word with them makes a call two to five times slower).
//   span field   the count of the span, top bit set once it is published
//   group word   bits 39..0 the sum of the counts of the group's spans, bit 40 set once it is published
// A block publishes its count as soon as it has counted, before it waits for anybody.  What lies before block b is the
// counts of the earlier blocks of its own group and of up to kWindow groups before it, plus the sums of all groups before
// those; the last block of a group, which has just added up its predecessors for itself, publishes the group's word.
// No block waits for another block's prefix, so the waits do not chain: a few hundred words are read once or twice per
// block.
//
// Why every wait ends.  Workgroups of a one-dimensional grid are handed to the eight XCDs in turn and each XCD starts its
// share in increasing order.  While a grid has the chip to itself, the smallest span not yet finished has therefore a free
// slot and has started, it publishes its count after a bounded amount of work of its own, and everything that it waits for
// is there.  Beside other grids that need not hold: two senders on two streams can each fill the slots that the other's
// oldest span needs.  So a wave of gq_compact that has polled kHelpAfterPolls times, far longer than any wait of a lone grid,
// counts a missing span itself and publishes the count (help); the span's own workgroup will store the same value.  Each
// such step puts in one of finitely many words, so every wait ends whatever the order in which workgroups start.
// gq_quantize_compact has no help: a wave would have to quantise the span, and its registers alone made every call 3 to 15 %
// slower.  Beside gq_compact and every other kernel it still gets its slots in the end; two of it that share the GPU may
// wait for each other.  All waits are bounded (kPrefixMaxPolls polls of about a microsecond): a workgroup that gives up
// writes nothing and raises count_out to 2^64 - 1, which no real count reaches.
//
// GQ_MUTE_SPANS = n (a test's build, 0 in the library): spans and groups whose number leaves 1 when divided by n publish
// nothing, as if they had not started, so that their words come from help alone.
// ---------------------------------------------------------------------------------------------------------
constexpr int kGroupWords = 64;
constexpr uint64_t kGroupPublished = 1ull << 40;
// Groups before the own one whose counts are read span by span, in grids of at least kWindowMinGroups groups (us a call on
// MI355X with 0 / 1 / 4 / 8 / 13 of them; 0 reads group sums only).  The more workgroups lie between a span and the oldest one
// still running, the more it gains; a short grid only pays for the extra words (12 groups below at 25.6e6, 24 at 50e6 and more).
//   gq_quantize_compact   110e6: 0.1 % non-zeros 86.3 / 86.9 / 79.7 / 78.7 / 89.8, 21 % 109.9 / 110.0 / 108.4 / 107.0 / 124.5;
//                         50e6: 42.2 / 42.5 / 40.0 / 40.1 / 47.5, 55.7 / 55.2 / 55.1 / 56.5 / 66.1;
//                         25.6e6: 25.4 / 25.9 / 25.9 / 26.0 / 27.8, 35.4 / 35.7 / 35.9 / 36.7 / 40.5
//   gq_compact            110e6: 32.0 / 31.7 / 30.5 / 29.2 / 42.7, 59.8 / 60.5 / 58.8 / 58.0 / 73.9;
//                         25.6e6: 12.6 / 12.5 / 12.4 / 12.9 / 14.8, 19.6 / 19.6 / 19.9 / 20.7 / 22.5
constexpr int kWindow = 4;
constexpr int kWindowMinGroups = 20;
#ifndef GQ_MUTE_SPANS
#define GQ_MUTE_SPANS 0
#endif
constexpr int kMuteSpans = GQ_MUTE_SPANS;
constexpr int kHelpAfterPolls = kMuteSpans > 0 ? 8 : 4096;                  // a poll takes about a microsecond
constexpr int kPrefixMaxPolls = kMuteSpans > 0 ? 1 << 13 : 1 << 21;
__device__ __forceinline__ bool mute(int64_t i) { return kMuteSpans > 0 && i % (kMuteSpans > 0 ? kMuteSpans : 1) == 1; }

// `empty_starts`: the one entry of the table of tile starts of an empty gradient, or nullptr
__global__ void __launch_bounds__(kBlock) compact_clear_kernel(uint64_t *__restrict__ state, int64_t words, uint64_t *__restrict__ count_out,
                                                               uint32_t *__restrict__ empty_starts)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < words) state[i] = 0;
    if (i == 0) *count_out = 0;
    if (i == 0 && empty_starts) empty_starts[0] = 0;
}

__device__ __forceinline__ uint64_t state_load(const uint64_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Inclusive prefix sum over the lanes of a wave: shifts inside the rows of 16, then the last lane of row 0 (2) is added to
// row 1 (3) and the last lane of row 1 to rows 2 and 3.  Every lane must be active.
__device__ __forceinline__ uint32_t wave_scan(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, true);     // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, true);     // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, true);     // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, true);     // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);    // row_bcast:15 into rows 1 and 3
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);    // row_bcast:31 into rows 2 and 3
    return v;
}
// the lanes for which c holds (the condition goes straight into a scalar mask)
__device__ __forceinline__ uint64_t ballot(bool c) { return __builtin_amdgcn_ballot_w64(c); }

__device__ __forceinline__ uint32_t last_lane(uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)v, 63); }

// Number of non-zero codes before span `span`: the counts of the earlier spans of its own group and of the kWindow groups
// before it, plus the sums of the groups before those.  Run by one whole wave; the result is uniform.  The counts of
// the workgroups that run at the same time are so read directly, one trip to memory after they were published; a group's
// sum, published by its last span a trip later, is only asked for when it is long there.  All words are asked for in the
// same round trip (a poll queues behind the bulk reads of the whole chip, so trips are what costs), and a group whose
// counts are complete is not asked for again.
struct Before {
    uint64_t total;              // what is known so far
    uint32_t in_group;           // the own group's part, once bit kWindow of `open` is clear
    uint32_t open;               // bit j: the counts of group (own - kWindow + j) are still missing
    int64_t next_group, groups;  // sums of the groups next_group .. groups - 1 are still missing
};

template <int SPAN> __device__ __forceinline__ Before nothing_known(int64_t span)
{
    constexpr int kGroupSpans = kGroupWords * Geometry<SPAN>::kPerWord;
    const int64_t group = span / kGroupSpans;
    if (gridDim.x < (unsigned)(kWindowMinGroups * kGroupSpans)) return {0, 0, 1u << kWindow, 0, group};
    const int first = group < kWindow ? kWindow - (int)group : 0;            // groups of the window that exist: first .. kWindow
    return {0, 0, ((2u << kWindow) - 1u) & ~((1u << first) - 1u), 0, group < kWindow ? 0 : group - kWindow};
}

template <int SPAN>
__device__ __forceinline__ void poll_before(const uint64_t *span_words, const uint64_t *group_words, int64_t span, Before *st)
{
    constexpr int kPerWord = Geometry<SPAN>::kPerWord;
    const int lane = (int)(threadIdx.x & 63u);
    const int64_t group = span / (kGroupWords * kPerWord);
    const int member = (int)(span - group * (kGroupWords * kPerWord));
    uint64_t w[kWindow + 1], w_gr = kGroupPublished;
    static_for<0, kWindow + 1>([&](auto jj) {
        constexpr int j = decltype(jj)::value;
        const int mine = j < kWindow ? kPerWord : member - lane * kPerWord;  // spans in this lane's word that lie before `span`
        w[j] = 0;
        if ((st->open >> j & 1u) != 0u && mine > 0) w[j] = state_load(span_words + (group - kWindow + j) * kGroupWords + lane);
    });
    if (st->next_group + lane < st->groups) w_gr = state_load(group_words + st->next_group + lane);
    static_for<0, kWindow + 1>([&](auto jj) {
        constexpr int j = decltype(jj)::value;
        if ((st->open >> j & 1u) == 0u) return;
        const int mine = j < kWindow ? kPerWord : member - lane * kPerWord;
        // one field: the flag is the top bit of the upper half, the count the lower half; two: each half has both
        const uint32_t lo = (uint32_t)w[j], hi = (uint32_t)(w[j] >> 32);
        const bool missing = kPerWord == 1 ? mine > 0 && (hi >> 31) == 0u : (mine > 0 && (lo >> 31) == 0u) || (mine > 1 && (hi >> 31) == 0u);
        if (ballot(missing) != 0) return;
        const uint32_t sum = kPerWord == 1 ? (mine > 0 ? lo : 0u)
                                           : (mine > 0 ? lo & 0x7FFFFFFFu : 0u) + (mine > 1 ? hi & 0x7FFFFFFFu : 0u);
        const uint32_t all = last_lane(wave_scan(sum));                      // at most 2^21
        if (j == kWindow) st->in_group = all;
        st->total += all;
        st->open &= ~(1u << j);
    });
    if (st->next_group < st->groups && ballot(((uint32_t)(w_gr >> 40) & 1u) == 0u) == 0) {
        st->total += last_lane(wave_scan((uint32_t)w_gr));                   // at most 64 * 2^21
        st->next_group += 64;
    }
}

struct NoHelp {};

// One missing word of those that `span` waits for, put in by the wave that waits: the count of a span, which `count_of` finds
// (run by the whole wave, the result is uniform), or, where all counts of a group are there, its sum.  Which missing span is
// counted depends on the one that waits, so that many waves count different ones.
template <int SPAN, typename F>
__device__ __forceinline__ void help(uint64_t *span_words, uint64_t *group_words, int64_t span, const Before &st, F &&count_of)
{
    typedef Geometry<SPAN> G;
    constexpr int kPerWord = G::kPerWord, kGroupSpans = kGroupWords * kPerWord;
    const int lane = (int)(threadIdx.x & 63u);
    int64_t group = span / kGroupSpans;
    if (st.open != 0u) {
        group += __builtin_ctz(st.open) - kWindow;
    } else {
        const bool wanted = st.next_group + lane < st.groups;
        const uint64_t w = wanted ? state_load(group_words + st.next_group + lane) : kGroupPublished;
        const uint64_t missing = ballot((w & kGroupPublished) == 0);
        if (missing == 0) return;
        group = st.next_group + __builtin_ctzll(missing);
    }
    const int64_t first = group * kGroupSpans;
    const int before = span - first < kGroupSpans ? (int)(span - first) : kGroupSpans;       // spans of the group that count
    const int mine = before - lane * kPerWord;
    const uint64_t w = mine > 0 ? state_load(span_words + group * kGroupWords + lane) : 0;
    const uint32_t lo = (uint32_t)w, hi = (uint32_t)(w >> 32);
    const uint64_t low = ballot(mine > 0 && ((kPerWord == 1 ? hi : lo) >> 31) == 0u), high = ballot(kPerWord == 2 && mine > 1 && (hi >> 31) == 0u);
    if ((low | high) != 0) {
        const uint64_t any = low | high, later = any >> (span & 63) << (span & 63);
        const int at = __builtin_ctzll(later != 0 ? later : any);
        const int64_t other = first + at * kPerWord + ((low >> at & 1) == 0 ? 1 : 0);
        const uint32_t count = count_of(other);
        if (lane == 0)
            __hip_atomic_store(reinterpret_cast<typename G::Field *>(span_words) + other, (typename G::Field)(G::kPublished | count), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    } else if (st.open == 0u) {
        const uint32_t sum = last_lane(wave_scan(kPerWord == 1 ? lo : (lo & 0x7FFFFFFFu) + (hi & 0x7FFFFFFFu)));
        if (lane == 0) __hip_atomic_store(group_words + group, kGroupPublished | (uint64_t)sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// What the waves of a workgroup share while they turn a span into list entries.
template <int STAGE> struct SpanShared {
    uint32_t cells[kMaxSpan / kCell];        // non-zeros in every cell of the span
    int64_t base;                            // entries before the span
    uint32_t stage[STAGE];                   // entries: offset in the span << 8 | code
};

// The list entries of one span.  Wave w holds the codes of cells w, w + kCompactWaves .. of the span, four words per
// lane and cell: word 4 b + i of lane l holds
//   W = 2 words in a row per lane   codes 512 (i / 2) + 8 l + 4 (i % 2) .. + 3 of the wave's cell b
//   W = 1                           codes 256 i + 4 l .. + 3
// and S.cells holds the counts of the whole span (the caller's barrier has passed).  Every thread must call it.
//
// The span's count is published before anything else: it is what the other workgroups wait for.  Finding out what lies
// before the span takes several round trips to memory (a poll queues behind the bulk reads of the chip), in which
// the workgroup's slots do nothing (with the wait taken out, 110e6 codes took 23 instead of 37 us).  A span whose entries
// fit the staging area (one code in four of a short span) is therefore ranked into it before the wait, and every wave but
// the first ends: the slots go to the next workgroups' reads, and the one wave left copies the entries out.  Denser
// spans wait with all waves, which then rank and copy out 512 codes at a time, each wave in its own part of the
// staging area and without a barrier.
// `count_of` is help's, or NoHelp.
template <int SPAN, int W, int STAGE, typename F>
__device__ __forceinline__ void emit_span(const uint32_t (&c)[4 * Geometry<SPAN>::kWaveCells], SpanShared<STAGE> &S, int64_t d,
                                          uint64_t *__restrict__ state, int64_t nwords, uint32_t *__restrict__ indices_out,
                                          int8_t *__restrict__ values_out, int64_t capacity, uint64_t *__restrict__ count_out,
                                          uint32_t *__restrict__ tile_starts_out, F count_of)
{
    typedef Geometry<SPAN> G;
    constexpr int kSpanCells = G::kSpanCells, kWaveCells = G::kWaveCells, kGroupSpans = kGroupWords * G::kPerWord;
    constexpr int kSteps = 2 / W;                            // steps per row of 512 codes
    const int lane = (int)(threadIdx.x & 63u), wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    uint64_t *span_words = state + 2;
    uint64_t *group_words = span_words + nwords;
    const int64_t span = blockIdx.x, last_span = (int64_t)gridDim.x - 1;
    const uint32_t cell_count = lane < kSpanCells ? S.cells[lane] : 0u;
    const uint32_t cell_start = wave_scan(cell_count) - cell_count;      // entries of the span before cell `lane`
    const uint32_t span_total = (uint32_t)__builtin_amdgcn_readlane((int)cell_start, kSpanCells);
    const uint32_t first_index = (uint32_t)(span * SPAN);
    constexpr bool kHelps = !std::is_same<F, NoHelp>::value;
    if (threadIdx.x == 0 && !(kHelps && mute(span)))
        __hip_atomic_store(reinterpret_cast<typename G::Field *>(span_words) + span, (typename G::Field)(G::kPublished | span_total), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);

    // The entries of row h of the wave's cell b go to stage[r ..]; returns how many there are.
    auto rank_row = [&](auto bb, auto hh, uint32_t *stage) -> uint32_t {
        constexpr int b = decltype(bb)::value, h = decltype(hh)::value;
        uint32_t n = 0;
        static_for<0, kSteps>([&](auto ss) {
            constexpr int step = decltype(ss)::value;
            uint32_t w[W], any = 0, cnt = 0;
#pragma unroll
            for (int i = 0; i < W; i++) {
                w[i] = c[4 * b + 2 * h + (W == 2 ? i : step)];
                any |= w[i];
            }
            if (ballot(any != 0) == 0) return;          // nothing in the whole wave
#pragma unroll
            for (int i = 0; i < W; i++) cnt += (uint32_t)__builtin_popcount(nonzero_bytes(w[i]));
            const uint32_t incl = wave_scan(cnt);
            uint32_t r = n + incl - cnt;
            n += last_lane(incl);
            // offset in the span of the lane's first code of this step
            const uint32_t off = (uint32_t)((b * kCompactWaves + wave) * kCell + h * kRow) + (W == 2 ? 8u * lane : 256u * step + 4u * lane);
#pragma unroll
            for (int i = 0; i < W; i++) {
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const uint32_t q = (w[i] >> (8 * k)) & 255u;
                    if (q != 0u) {
                        stage[r] = ((off + 4 * i + k) << 8) | q;
                        r++;
                    }
                }
            }
        });
        return n;
    };
    // n staged entries to list position pos and on, as far as the list reaches
    auto copy_out = [&](const uint32_t *stage, uint32_t n, int64_t pos) {
        const int64_t room = capacity - pos;
        const uint32_t m = room <= 0 ? 0u : room < (int64_t)n ? (uint32_t)room : n;
        for (uint32_t e = lane; e < m; e += 64) {
            const uint32_t entry = stage[e];
            indices_out[pos + e] = first_index + (entry >> 8);
            values_out[pos + e] = (int8_t)entry;
        }
    };
    const bool staged = span_total <= (uint32_t)STAGE;                  // uniform over the block
    if (staged) {
        static_for<0, kWaveCells>([&](auto bb) {
            constexpr int b = decltype(bb)::value;
            uint32_t at = (uint32_t)__builtin_amdgcn_readlane((int)cell_start, b * kCompactWaves + wave);
            if (__builtin_amdgcn_readlane((int)cell_count, b * kCompactWaves + wave) == 0) return;
            at += rank_row(bb, std::integral_constant<int, 0>{}, S.stage + at);
            rank_row(bb, std::integral_constant<int, 1>{}, S.stage + at);
        });
        __syncthreads();
        if (wave != 0) return;
    }
    if (wave == 0) {
        Before st = nothing_known<SPAN>(span);
        bool group_sum_out = span % kGroupSpans != kGroupSpans - 1;       // only a group's last span owes one
        // one poll; true once everything is there
        auto poll = [&]() -> bool {
            poll_before<SPAN>(span_words, group_words, span, &st);
            // the group's last span publishes the group's sum as soon as it has it, before it waits on
            if ((st.open >> kWindow & 1u) == 0u && !group_sum_out) {
                if (lane == 0 && !(kHelps && mute(span / kGroupSpans)))
                    __hip_atomic_store(group_words + span / kGroupSpans, kGroupPublished | (uint64_t)(st.in_group + span_total), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
                group_sum_out = true;
            }
            return st.open == 0u && st.next_group >= st.groups;
        };
        constexpr int kMostPolls = kHelps ? kHelpAfterPolls : kPrefixMaxPolls;
        int polls = 0;
        while (!poll() && ++polls <= kMostPolls) __builtin_amdgcn_s_sleep(4);
        bool gave_up = polls > kMostPolls;
        if constexpr (kHelps) {
            if (__builtin_expect(gave_up, 0)) {
                do help<SPAN>(span_words, group_words, span, st, count_of);
                while (!poll() && ++polls <= kPrefixMaxPolls);
                gave_up = polls > kPrefixMaxPolls;
            }
        }
        const uint64_t before = st.total;
        if (lane == 0) {
            if (gave_up) atomicMax(reinterpret_cast<unsigned long long *>(count_out), ~0ull);
            else if (span == last_span)
                atomicMax(reinterpret_cast<unsigned long long *>(count_out), (unsigned long long)(before + span_total));
            S.base = gave_up ? -1 : (int64_t)before;
        }
        if (tile_starts_out && !gave_up) {
            // where each tile of the span begins in the list (what the receiver would otherwise search for), and behind
            // the last tile the end of the list
            const int64_t ntiles = (d + kCompactTile - 1) / kCompactTile;
            const int64_t tile = span * (SPAN / kCompactTile) + lane / (kCompactTile / kCell);
            if (lane < kSpanCells && lane % (kCompactTile / kCell) == 0 && tile < ntiles) tile_starts_out[tile] = (uint32_t)before + cell_start;
            if (span == last_span && lane == 0) tile_starts_out[ntiles] = (uint32_t)before + span_total;
        }
        if (staged) {
            if (!gave_up) copy_out(S.stage, span_total, (int64_t)before);
            return;
        }
    }
    __syncthreads();
    const int64_t base = S.base;
    if (base < 0) return;                                    // uniform over the block
    uint32_t *stage = S.stage + wave * kRow;
    static_for<0, kWaveCells>([&](auto bb) {
        constexpr int b = decltype(bb)::value;
        int64_t pos = base + (uint32_t)__builtin_amdgcn_readlane((int)cell_start, b * kCompactWaves + wave);
        static_for<0, 2>([&](auto hh) {
            const uint32_t n = rank_row(bb, hh, stage);
            // the wave's own part of the staging area: its reads follow its writes in order
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            copy_out(stage, n, pos);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            pos += n;
        });
    });
}

template <int SPAN>
__global__ void __launch_bounds__(64 * kCompactWaves) __attribute__((amdgpu_num_sgpr(kCompactScalars)))
compact_onepass_kernel(const uint8_t *__restrict__ lv, int64_t d, uint64_t *__restrict__ state, int64_t nwords,
                       uint32_t *__restrict__ indices_out, int8_t *__restrict__ values_out, int64_t capacity,
                       uint64_t *__restrict__ count_out, uint32_t *__restrict__ tile_starts_out)
{
    constexpr int kWaveCells = Geometry<SPAN>::kWaveCells;
    __shared__ SpanShared<kStage> S;
    const int lane = (int)(threadIdx.x & 63u), wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t t0 = (int64_t)blockIdx.x * (SPAN / 8) + wave * (kCell / 8) + lane;
    u32x2 u[2 * kWaveCells];
    const bool whole = ((int64_t)blockIdx.x + 1) * SPAN <= d;     // uniform over the workgroup
#pragma unroll
    for (int j = 0; j < 2 * kWaveCells; j++) {
        const int64_t t = t0 + (j >> 1) * (kCompactWaves * kCell / 8) + (j & 1) * 64;
        u[j] = whole ? __builtin_nontemporal_load(reinterpret_cast<const u32x2 *>(lv) + t) : load_code_unit(lv, t, d);
    }
    uint32_t c[4 * kWaveCells];
#pragma unroll
    for (int b = 0; b < kWaveCells; b++) {
        c[4 * b] = u[2 * b].x; c[4 * b + 1] = u[2 * b].y; c[4 * b + 2] = u[2 * b + 1].x; c[4 * b + 3] = u[2 * b + 1].y;
        uint32_t cnt = 0;
#pragma unroll
        for (int i = 0; i < 4; i++) cnt += (uint32_t)__builtin_popcount(nonzero_bytes(c[4 * b + i]));
        const uint32_t sum = last_lane(wave_scan(cnt));
        if (lane == 0) S.cells[b * kCompactWaves + wave] = sum;
    }
    __syncthreads();
    emit_span<SPAN, 2>(c, S, d, state, nwords, indices_out, values_out, capacity, count_out, tile_starts_out, [&](int64_t other) {
        uint32_t n = 0;
#pragma unroll 1
        for (int i = lane; i < SPAN / 8; i += 64) {
            const u32x2 q = load_code_unit(lv, other * (SPAN / 8) + i, d);
            n += (uint32_t)(__builtin_popcount(nonzero_bytes(q.x)) + __builtin_popcount(nonzero_bytes(q.y)));
        }
        return last_lane(wave_scan(n));
    });
}

// ---------------------------------------------------------------------------------------------------------
// Sender side without the dense codes: Algorithm 1's quantisation loop for one worker feeding the list directly.
// Every wave quantises its own cells of the span, one vector of four coordinates per lane at a time, with the same
// rounding, random stream and call indices as gq_quantize, and hands the code words to emit_span: 4 d bytes read,
// 5 nnz written, and the codes never reach memory.
//   full draws   lane l owns vector l of every 64 consecutive ones
//   short draws  a lane owns vectors l and 64 + l of 128 consecutive ones and shares its Philox words with its
//                neighbour lane (one call per eight coordinates, every load contiguous over the wave)
// The loads of the next cell are issued before the current one is rounded.  A code is non-zero iff
// Round::nonzero says so, which costs about half of the full rounding rule: where it holds for no coordinate of the
// wave (most of the time under the (2,2) norm) the codes are not formed at all.
// ---------------------------------------------------------------------------------------------------------
template <int SPAN, int SCHEME, bool UNIFORM_HI, bool HALF, bool WHOLE>
__device__ __forceinline__ void quantize_cells(const float *__restrict__ x, int64_t d, const Scale &sc, bool one_level, uint64_t seed, uint32_t worker,
                                                 uint64_t call_base, uint32_t (&c)[4 * Geometry<SPAN>::kWaveCells],
                                                 uint32_t *cells)
{
    constexpr int kWaveCells = Geometry<SPAN>::kWaveCells;
    constexpr int kBatch = kCell / 256;                               // vectors per lane and cell: 4
    const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    const int64_t nfull = d >> 2;
    const int lane = (int)(threadIdx.x & 63u), wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t v0 = ((int64_t)blockIdx.x * SPAN + wave * kCell) / 4;    // scalar: the wave's first cell
    constexpr int kNextCell = kCompactWaves * kCell / 4;
    auto load_batch = [&](int b, f32x4 *g) {
#pragma unroll
        for (int i = 0; i < kBatch; i++) {
            const int64_t v = v0 + b * kNextCell + i * 64 + lane;
            if (WHOLE) g[i] = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(x) + v);
            else g[i] = load_coords(x, v, v < nfull ? 4 : (v == nfull ? (int)(d & 3) : 0));
        }
    };
    auto counter = [&](uint64_t first, int local, uint32_t &c_lo, uint32_t &c_hi) {
        if (UNIFORM_HI) {                                             // host: the launch stays below the next multiple of 2^32 calls
            c_hi = (uint32_t)(first >> 32);
            c_lo = (uint32_t)first + (uint32_t)local;
        } else {
            const uint64_t cc = first + (uint64_t)local;
            c_lo = (uint32_t)cc;
            c_hi = (uint32_t)(cc >> 32);
        }
    };
    uint32_t count = 0;                                               // scalar: non-zeros of the current cell
    // coordinates past the end were loaded as zeros, whose code is 0
    auto round_vector = [&](const f32x4 &g, const uint32_t *draw) -> uint32_t {
        uint64_t m0 = ballot(Round<SCHEME>::nonzero(g.x, sc, draw[0])), m1 = ballot(Round<SCHEME>::nonzero(g.y, sc, draw[1]));
        uint64_t m2 = ballot(Round<SCHEME>::nonzero(g.z, sc, draw[2])), m3 = ballot(Round<SCHEME>::nonzero(g.w, sc, draw[3]));
        if (one_level) {
            m0 |= ballot(__builtin_fabsf(g.x) >= sc.full); m1 |= ballot(__builtin_fabsf(g.y) >= sc.full);
            m2 |= ballot(__builtin_fabsf(g.z) >= sc.full); m3 |= ballot(__builtin_fabsf(g.w) >= sc.full);
        }
        uint32_t w = 0;
        if ((m0 | m1 | m2 | m3) != 0) {
            count += (uint32_t)(__builtin_popcountll(m0) + __builtin_popcountll(m1) + __builtin_popcountll(m2) + __builtin_popcountll(m3));
            w = Quad4<SCHEME>(g, sc, draw).signed_bytes();
        }
        return w;
    };
    f32x4 g[kBatch], gn[kBatch];
    load_batch(0, g);
    static_for<0, kWaveCells>([&](auto bb) {
        constexpr int b = decltype(bb)::value;
        if constexpr (b + 1 < kWaveCells) load_batch(b + 1, gn);
        const int64_t vb = v0 + b * kNextCell;                       // scalar
        if (HALF) {
#pragma unroll
            for (int h = 0; h < kBatch / 2; h++) {
                uint32_t c_lo, c_hi;
                counter(call_base + (uint64_t)((vb + h * 128) >> 1), (lane >> 1) + (lane & 1) * 32, c_lo, c_hi);
                const ShortDraws sd = share_short_draws(philox4x32_10(c_lo, c_hi, worker, 0u, k0, k1), (lane & 1) != 0);
                uint32_t da[4], db[4];
#pragma unroll
                for (int i = 0; i < 4; i++) { da[i] = short_draw(sd.a, i); db[i] = short_draw(sd.b, i); }
                c[b * kBatch + 2 * h] = round_vector(g[2 * h], da);
                c[b * kBatch + 2 * h + 1] = round_vector(g[2 * h + 1], db);
            }
        } else {
#pragma unroll
            for (int i = 0; i < kBatch; i++) {
                uint32_t c_lo, c_hi;
                counter(call_base + (uint64_t)(vb + i * 64), lane, c_lo, c_hi);
                const Words4 r = philox4x32_10(c_lo, c_hi, worker, 0u, k0, k1);
                c[b * kBatch + i] = round_vector(g[i], r.w);
            }
        }
        if (lane == 0) cells[b * kCompactWaves + wave] = count;
        count = 0;
        if constexpr (b + 1 < kWaveCells) {
#pragma unroll
            for (int i = 0; i < kBatch; i++) g[i] = gn[i];
        }
    });
}

template <int SPAN, int SCHEME, bool UNIFORM_HI, bool HALF>
__global__ void __launch_bounds__(64 * kCompactWaves)
quantize_compact_kernel(const float *__restrict__ x, int64_t d, const float *__restrict__ norm, int s, uint64_t seed, uint32_t worker,
                        uint64_t call_base, uint64_t *__restrict__ state, int64_t nwords, uint32_t *__restrict__ indices_out,
                        int8_t *__restrict__ values_out, int64_t capacity, uint64_t *__restrict__ count_out,
                        uint32_t *__restrict__ tile_starts_out)
{
    __shared__ SpanShared<SPAN == kMaxSpan ? 2 * kStage : kStage> S;
    const Scale sc = make_scale<SCHEME>(*norm, s);
    const bool whole = ((int64_t)blockIdx.x + 1) * SPAN <= (d & ~(int64_t)3);     // uniform over the workgroup
    uint32_t c[4 * Geometry<SPAN>::kWaveCells];
    if (whole) quantize_cells<SPAN, SCHEME, UNIFORM_HI, HALF, true>(x, d, sc, s == 1, seed, worker, call_base, c, S.cells);
    else quantize_cells<SPAN, SCHEME, UNIFORM_HI, HALF, false>(x, d, sc, s == 1, seed, worker, call_base, c, S.cells);
    __syncthreads();
    emit_span<SPAN, 1>(c, S, d, state, nwords, indices_out, values_out, capacity, count_out, tile_starts_out, NoHelp{});
}

struct SparseLists {
    const uint32_t *idx[kMaxWorkers];
    const int8_t *val[kMaxWorkers];
    const uint64_t *cnt[kMaxWorkers];
    const uint32_t *starts[kMaxWorkers];     // where every tile of kSparseTile coordinates begins in the list, or nullptr
    int64_t cap[kMaxWorkers];
};

// Receiver side.  A workgroup of 512 threads owns a span of 8192 coordinates, held as an int32 array in LDS.
// The threads are split evenly over the K workers (512 / K' lanes each, K' = K rounded up to a power of two), so
// that all K list segments of the span are walked side by side: every lane learns where its worker's segment begins
// and ends -- from the table of tile starts that gq_compact wrote beside the list, or, if the sender gave none, by
// binary search in the sorted index list -- and adds its share of the entries into the LDS array (LDS atomics),
// four loads in flight per lane.  The span is then written once with 128-bit stores.  No global atomics and no
// separate zero fill: every output word is written exactly once.
constexpr int kSparseBlock = 512;
// Long segments: four entries in a row per lane with one 128-bit and one 32-bit load (110e6 coordinates, 16 lists of 17 %:
// 0.40 -> 0.34 ms; 8e6, 64 lists of 21 %: 176 -> 128 us; single loads with eight entries in flight 0.35 ms and 319 us, most of it
// address arithmetic).  One quad in flight is 3 to 10 % slower, four are no faster and slower on short segments.
constexpr int kSparseQuads = 2;
constexpr int64_t kSparseMost = 1 << 30;                 // entries of a segment (a sorted list has at most kSparseSpan)
typedef uint32_t u32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));     // entries begin anywhere in their lists
typedef uint32_t u32_a1 __attribute__((aligned(1)));
constexpr int kSparseSpan = 2 * kCompactTile;            // two tiles of the sender's table of tile starts

template <int SCHEME>
__global__ void __launch_bounds__(kSparseBlock)
sparse_span_kernel(SparseLists S, int K, int lanes_per_worker, int64_t d, int *__restrict__ agg)
{
    __shared__ int span[kSparseSpan];
    __shared__ int64_t s_begin[kMaxWorkers], s_end[kMaxWorkers];
    const int64_t lo = (int64_t)blockIdx.x * kSparseSpan;
    const int64_t hi = lo + kSparseSpan < d ? lo + kSparseSpan : d;
    const int w = (int)threadIdx.x / lanes_per_worker;         // this thread's worker (if w < K) and its slot
    const int slot = (int)threadIdx.x - w * lanes_per_worker;
    const uint32_t *idx = S.idx[w < K ? w : 0];                // asked for before the look-up, which it does not depend on
    const int8_t *val = S.val[w < K ? w : 0];
    // the worker's entries with lo <= index < hi lie at [begin, end) of its list: lane 0 of the worker's lanes looks up
    // begin, lane 1 end (there are at least eight lanes per worker)
    if (w < K && slot < 2) {
        const uint64_t have = *S.cnt[w];
        const int64_t n = have < (uint64_t)S.cap[w] ? (int64_t)have : S.cap[w];
        const int64_t key = slot == 0 ? lo : hi;
        int64_t at;
        if (S.starts[w]) {
            const int64_t ntiles = (d + kCompactTile - 1) / kCompactTile;
            const int64_t t = (key + kCompactTile - 1) / kCompactTile;     // key is a multiple of the tile size, or d
            at = (int64_t)S.starts[w][t < ntiles ? t : ntiles];
            at = at < n ? at : n;                              // a list cut short by its capacity ends at n
        } else {
            int64_t a = 0, e = n;                              // first entry whose index is >= key
            while (a < e) {
                const int64_t mid = (a + e) >> 1;
                if ((int64_t)S.idx[w][mid] < key) a = mid + 1; else e = mid;
            }
            at = a;
        }
        if (slot == 0) s_begin[w] = at; else s_end[w] = at;
    }
    for (int i = threadIdx.x * 4; i < kSparseSpan; i += kSparseBlock * 4) *reinterpret_cast<i32x4 *>(&span[i]) = i32x4{0, 0, 0, 0};
    __syncthreads();
    if (w < K) {
        const int64_t begin = s_begin[w], left = s_end[w] - begin;
        uint32_t n = left <= 0 ? 0u : left < kSparseMost ? (uint32_t)left : (uint32_t)kSparseMost;
        idx += begin;
        val += begin;
        auto add_entry = [&](uint32_t index, int q) {
            int v = q;
            if (SCHEME == 1) {
                const int mag = (int)((1u << abs(q)) >> 1);
                v = q < 0 ? -mag : mag;
            }
            const uint32_t j = index - (uint32_t)lo;
            if (j < (uint32_t)kSparseSpan) atomicAdd(&span[j], v);     // always true for a sorted list
        };
        // four entries in a row per lane, kSparseQuads such quads in flight; a segment of no more than two entries per lane:
        // a lane's two, both asked for at once (past the end the last one again)
        if (n <= 2u * (uint32_t)lanes_per_worker) {
            if ((uint32_t)slot < n) {
                const uint32_t second = (uint32_t)slot + (uint32_t)lanes_per_worker, at = second < n ? second : n - 1u;
                const uint32_t i0 = idx[slot], i1 = idx[at];
                const int q0 = val[slot], q1 = val[at];
                add_entry(i0, q0);
                if (second < n) add_entry(i1, q1);
            }
            n = 0;
        }
        // A quad that would reach past the segment is the last four entries instead (n > lanes_per_worker >= 8), of which
        // those before `at` belong to other lanes: no second set of loads behind a branch, which would wait for the first.
        const uint32_t step = 4u * (uint32_t)lanes_per_worker;
        for (uint32_t e = 4u * (uint32_t)slot; e < n; e += kSparseQuads * step) {
            u32x4_a4 index[kSparseQuads];
            uint32_t codes[kSparseQuads], others[kSparseQuads];
#pragma unroll
            for (int u = 0; u < kSparseQuads; u++) {
                const uint32_t at = e + u * step, from = at < n - 4u ? at : n - 4u;
                others[u] = at - from;
                index[u] = *reinterpret_cast<const u32x4_a4 *>(idx + from);
                codes[u] = *reinterpret_cast<const u32_a1 *>(val + from);
            }
#pragma unroll
            for (int u = 0; u < kSparseQuads; u++) {
                if (others[u] == 0u) add_entry(index[u].x, (int8_t)codes[u]);
                if (others[u] <= 1u) add_entry(index[u].y, (int8_t)(codes[u] >> 8));
                if (others[u] <= 2u) add_entry(index[u].z, (int8_t)(codes[u] >> 16));
                if (others[u] <= 3u) add_entry(index[u].w, (int8_t)(codes[u] >> 24));
            }
        }
    }
    __syncthreads();
    for (int i = threadIdx.x * 4; i < kSparseSpan; i += kSparseBlock * 4) {
        const int64_t c = lo + i;
        if (c + 4 <= d) {
            __builtin_nontemporal_store(*reinterpret_cast<const i32x4 *>(&span[i]), reinterpret_cast<i32x4 *>(agg + c));
        } else {
            for (int u = 0; u < 4 && c + u < d; u++) agg[c + u] = span[i + u];
        }
    }
}



// words of the scan over 0 <= d <= 2^32 - 1 codes: two spare ones, one per kWordSpan codes, one per group of 64 of those
static inline int64_t span_words(int64_t d) { return (d + kWordSpan - 1) / kWordSpan; }
// Codes per workgroup.  Short spans spread a short gradient over the chip and let the workgroups end evenly; long ones pay
// the wait for the spans before them less often.  Where the lines lie (us a call on MI355X, short / long spans):
//   gq_compact            25.6e6 codes: 0.2 % non-zeros 13.6 / 13.5, 22 % 19.4 / 21.8;  50e6: 19.6 / 17.5, 31.1 / 32.7;  110e6: 39.2 / 33.8, 61 / 62
//   gq_quantize_compact   25.6e6: 25.0 / 28.8, 35.3 / 40;  110e6: 0.1 % 86.7 / 85.4, 21 % 110 / 115;  300e6: 225 / 217, 300 / 305
// (both with group sums only for what lies before the own group, kWindow = 0)
// (one pass of the earlier kernels, spans of 32768 codes on 256 threads: 16.7, 24.8, 25.8, 38.6, 43.1, 64.6 and 34.2, 41.7, 89.7,
// 115, 220, 298)
constexpr int64_t kCompactLongFrom = 1ll << 25, kQuantCompactLongFrom = 1ll << 27;
static inline int span_size(int64_t d, int64_t long_from) { return d < long_from ? kMaxSpan / 2 : kMaxSpan; }
static inline int64_t scan_words(int64_t d) { return 2 + span_words(d) + (span_words(d) + kGroupWords - 1) / kGroupWords; }

}  // namespace gq

using namespace gq;

extern "C" {

size_t gq_compact_workspace_bytes(int64_t d)
{
    if (d < 0 || d > 0xFFFFFFFFLL) return 0;
    return (size_t)scan_words(d) * sizeof(uint64_t);
}

int64_t gq_tile_starts_len(int64_t d)
{
    if (d < 0 || d > 0xFFFFFFFFLL) return 0;
    return (d + kCompactTile - 1) / kCompactTile + 1;
}

gq_status gq_compact(const void *levels, int64_t d, const gq_params *p, uint32_t *indices_out, int8_t *values_out,
                     int64_t capacity, uint64_t *count_out, uint32_t *tile_starts_out, void *workspace, size_t workspace_bytes,
                     void *hip_stream)
{
    const gq_status st = check_params(p, true, false);
    if (st != GQ_OK) return st;
    if (p->pack != GQ_PACK_I8) return GQ_ERR_UNSUPPORTED;
    if (d < 0 || d > 0xFFFFFFFFLL || capacity < 0) return GQ_ERR_INVALID_ARG;
    if (!aligned(count_out, 8)) return GQ_ERR_INVALID_ARG;
    if (d > 0 && !aligned(levels, 16)) return GQ_ERR_INVALID_ARG;
    if (capacity > 0 && (!aligned(indices_out, 4) || !values_out)) return GQ_ERR_INVALID_ARG;
    if (tile_starts_out && !aligned(tile_starts_out, 4)) return GQ_ERR_INVALID_ARG;
    if (!workspace || workspace_bytes < gq_compact_workspace_bytes(d)) return GQ_ERR_WORKSPACE;
    if (!aligned(workspace, 8)) return GQ_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)hip_stream;
    uint64_t *state = reinterpret_cast<uint64_t *>(workspace);
    const int span = span_size(d, kCompactLongFrom);
    const int64_t blocks = (d + span - 1) / span;
    if (!grid_fits(blocks, 64 * kCompactWaves)) return GQ_ERR_INVALID_ARG;
    const uint8_t *lv = reinterpret_cast<const uint8_t *>(levels);
    // the scan's words and the count start from zero (a fill kernel, so that the call can be captured in a graph)
    const int64_t words = scan_words(d);
    hipLaunchKernelGGL(compact_clear_kernel, dim3((unsigned)((words + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, state, words, count_out,
                       blocks == 0 ? tile_starts_out : nullptr);
    if (launched() != GQ_OK) return GQ_ERR_DEVICE;
    if (blocks > 0) {
#define GQ_COMPACT(SPAN) hipLaunchKernelGGL(compact_onepass_kernel<SPAN>, dim3((unsigned)blocks), dim3(64 * kCompactWaves), 0, s, lv, d, state, \
                                            span_words(d), indices_out, values_out, capacity, count_out, tile_starts_out)
        if (span == kMaxSpan) GQ_COMPACT(kMaxSpan); else GQ_COMPACT(kMaxSpan / 2);
#undef GQ_COMPACT
        if (launched() != GQ_OK) return GQ_ERR_DEVICE;
    }
    return GQ_OK;
}

gq_status gq_quantize_compact(const float *x, int64_t d, const float *norm, const gq_params *p, uint32_t worker, int64_t index_base,
                              uint32_t *indices_out, int8_t *values_out, int64_t capacity, uint64_t *count_out,
                              uint32_t *tile_starts_out, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    const gq_status st = check_params(p, true, false);
    if (st != GQ_OK) return st;
    if (p->pack != GQ_PACK_I8) return GQ_ERR_UNSUPPORTED;
    const bool half = short_draws(p);
    if (d < 0 || d > 0xFFFFFFFFLL || capacity < 0 || index_base < 0 || (index_base & (half ? 7 : 3)) != 0) return GQ_ERR_INVALID_ARG;
    if (!aligned(norm, 4) || !aligned(count_out, 8)) return GQ_ERR_INVALID_ARG;
    if (d > 0 && !aligned(x, 16)) return GQ_ERR_INVALID_ARG;
    if (capacity > 0 && (!aligned(indices_out, 4) || !values_out)) return GQ_ERR_INVALID_ARG;
    if (tile_starts_out && !aligned(tile_starts_out, 4)) return GQ_ERR_INVALID_ARG;
    if (!workspace || workspace_bytes < gq_compact_workspace_bytes(d)) return GQ_ERR_WORKSPACE;
    if (!aligned(workspace, 8)) return GQ_ERR_INVALID_ARG;
    hipStream_t hs = (hipStream_t)hip_stream;
    uint64_t *state = reinterpret_cast<uint64_t *>(workspace);
    const int span = span_size(d, kQuantCompactLongFrom);
    const int64_t blocks = (d + span - 1) / span;
    if (!grid_fits(blocks, 64 * kCompactWaves)) return GQ_ERR_INVALID_ARG;
    const int64_t words = scan_words(d);
    hipLaunchKernelGGL(compact_clear_kernel, dim3((unsigned)((words + kBlock - 1) / kBlock)), dim3(kBlock), 0, hs, state, words, count_out,
                       blocks == 0 ? tile_starts_out : nullptr);
    if (launched() != GQ_OK) return GQ_ERR_DEVICE;
    if (blocks == 0) return GQ_OK;
    const int lane_vecs = half ? 2 : 1;                                  // vectors per Philox call
    const uint64_t call_base = (uint64_t)index_base / (uint64_t)(4 * lane_vecs);
    // the high counter word is a scalar unless the gradient (rounded up to whole spans) crosses 2^32 calls
    const bool one_stretch = ((call_base & 0xFFFFFFFFull) + (uint64_t)(blocks * (span / 4) / lane_vecs)) <= ((uint64_t)1 << 32);
#define GQ_QC3(SP, SC, UH, HF) hipLaunchKernelGGL((quantize_compact_kernel<SP, SC, UH, HF>), dim3((unsigned)blocks), dim3(64 * kCompactWaves), 0, hs, x, d, \
                                             norm, p->s, p->seed, worker, call_base, state, span_words(d), indices_out, values_out, capacity, \
                                             count_out, tile_starts_out)
#define GQ_QC(SC, UH, HF) do { if (span == kMaxSpan) GQ_QC3(kMaxSpan, SC, UH, HF); else GQ_QC3(kMaxSpan / 2, SC, UH, HF); } while (0)
#define GQ_QC2(SC, UH) do { if (half) GQ_QC(SC, UH, true); else GQ_QC(SC, UH, false); } while (0)
    if (p->scheme == GQ_LINEAR) { if (one_stretch) GQ_QC2(0, true); else GQ_QC2(0, false); }
    else                        { if (one_stretch) GQ_QC2(1, true); else GQ_QC2(1, false); }
#undef GQ_QC2
#undef GQ_QC
#undef GQ_QC3
    return launched();
}

gq_status gq_sparse_aggregate(const uint32_t *const *indices, const int8_t *const *values,
                              const uint64_t *const *counts, const int64_t *capacities,
                              const uint32_t *const *tile_starts, int K, int64_t d,
                              const gq_params *p, void *agg_out, void *hip_stream)
{
    gq_status st = check_params(p, false, true);
    if (st != GQ_OK) return st;
    if (p->agg != GQ_AGG_I32) return GQ_ERR_UNSUPPORTED;
    if (!indices || !values || !counts || !capacities || K < 1 || K > GQ_MAX_WORKERS || d < 0 || d > 0xFFFFFFFFLL)
        return GQ_ERR_INVALID_ARG;
    st = gq_check_width(p, K);
    if (st != GQ_OK) return st;
    SparseLists S;
    for (int i = 0; i < K; i++) {
        if (capacities[i] < 0 || !aligned(counts[i], 8)) return GQ_ERR_INVALID_ARG;
        if (capacities[i] > 0 && (!aligned(indices[i], 4) || !values[i])) return GQ_ERR_INVALID_ARG;
        S.idx[i] = indices[i];
        S.val[i] = values[i];
        S.cnt[i] = counts[i];
        S.cap[i] = capacities[i];
        S.starts[i] = tile_starts ? tile_starts[i] : nullptr;
        if (S.starts[i] && !aligned(S.starts[i], 4)) return GQ_ERR_INVALID_ARG;
    }
    if (d > 0 && !aligned(agg_out, 16)) return GQ_ERR_INVALID_ARG;
    if (d == 0) return GQ_OK;
    hipStream_t s = (hipStream_t)hip_stream;
    const int64_t blocks = (d + kSparseSpan - 1) / kSparseSpan;
    if (!grid_fits(blocks, kSparseBlock)) return GQ_ERR_INVALID_ARG;
    const dim3 grid((unsigned)blocks);
    int kpad = 1;
    while (kpad < K) kpad <<= 1;
    const int lanes = kSparseBlock / kpad;                      // threads per worker: 512 for K = 1 ... 8 for K = 64
    if (p->scheme == GQ_LINEAR) hipLaunchKernelGGL(sparse_span_kernel<0>, grid, dim3(kSparseBlock), 0, s, S, K, lanes, d, (int *)agg_out);
    else hipLaunchKernelGGL(sparse_span_kernel<1>, grid, dim3(kSparseBlock), 0, s, S, K, lanes, d, (int *)agg_out);
    if (launched() != GQ_OK) return GQ_ERR_DEVICE;
    return GQ_OK;
}

}  // extern "C"
