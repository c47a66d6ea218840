// Device-wide soft-priority scheduler shared by the persistent kernels.
//
// The paper's asynchronous marching method (Algorithm "Asynchronous Marching
// Method", section "The Asynchronous Marching Method") pushes work with an
// integer priority floor(t / scale) into a concurrent scheduler that returns an
// approximately earliest item and tolerates priority inversions.  Here the work
// item is a grid tile and the scheduler is a window of NB bucket rings:
//
//  * a tile pushed with time t goes to bucket k = floor(t / delta), clamped to
//    the window [cur, cur + NB); the rings k mod NB hold it;
//  * a claimer takes work from the lowest bucket that has any, within a window
//    above the current bucket `cur` (Sched::lookahead, or kWide for a workgroup
//    that has been idle, unless the caller keeps it from that); `cur` moves on (to the next bucket that is not drained)
//    only once nothing is queued in it and no tile claimed from it is still
//    running.  This is the bucket discipline of delta-stepping with a window:
//    the number of premature (later lowered again) tile runs stays small;
//  * a push goes at most kRings - 1 buckets above the `cur` its run was claimed
//    under, and `cur` never decreases, so no later bucket is put into the ring of
//    an open one (an item that `cur` has passed by, see claim_with, counts as
//    kRings buckets later, which only delays it);
//  * delta = 0 puts everything in one bucket (a plain FIFO worklist);
//  * the operator is monotone and causal, so none of this changes results.
//
// Shards.  A bucket's ring is split into kShards rings, and a tile always
// goes to the one its id names (neighbouring tiles to different ones, one of
// every aligned group of 8 to each).  A workgroup claims from its own shard
// first and from the others when that one shows nothing.  The reason: the
// device completes a read-modify-write of one 64-byte line about every 12 ns
// whoever issues it (83 per us measured with 64 to 4096 waves, against 545 per
// us over 8 lines), and while such requests queue, the loads behind them in the
// compute unit wait too (staging a tile took 33 us instead of 3.2 us with 2816
// waves on unsharded rings).  The live work is one word per shard for the same
// reason; all_done() reads them twice.
//
// Each ring is a bounded MPMC array of 64-bit cells (sequence << 32 | tile),
// positions taken with fetch-add.  Its queued count and the number of runs
// claimed from it share one 64-bit word (running << 32 | count + 2^31), so a
// claim is one RMW (running + 1, count - 1) and one load shows whether the
// bucket is drained (nothing queued and nothing running at the same instant).  A cell for position p is free when its
// sequence equals p, full when it equals p + 1, and is freed for the next lap
// (sequence p + cap) by the consumer after reading: a producer never overwrites
// a cell whose item has been claimed but not yet read.  A tile is queued at most
// once at a time (tile state machine below), so a ring never holds more than
// its share of the tiles, ceil(ntiles / 8), and capacity = next_pow2(max(that, 2))
// means no producer waits on an unclaimed item.  Positions and counters are never reset between solves
// (a solve ends with every ring drained), only re-initialised after a watchdog
// expiry.
//
// Tile state word (one uint32 per tile):
//   bit0 Q  queued / needs another run       bit1 R  a wave or workgroup is running it
//   bit2 V  interior of t holds real values  bit3 S  contains a point source
// Activation = fetch_or(Q) after the writer's stores completed; whoever turns an idle word
// (no Q, no R) into Q pushes the tile.  A runner turns Q into R with an
// acquiring RMW before it reads any t, and at the end either clears R (idle) or,
// if Q was set meanwhile, keeps Q and pushes the tile again.  So every change
// of a tile's halo or interior is followed by a run that starts after it, and
// at most one of them runs a tile at any time.
//
// Memory ordering across the 8 XCDs (each with its own L2).  Every access to
// data another workgroup may touch concurrently -- arrival times, adjoint
// multipliers, tile states, queue cells and counters -- is a device-scope
// (agent) atomic, which gfx950 issues with the device-scope cache policy
// (loads and stores coherent at device scope without any cache maintenance).
// Ordering then only needs completion: a writer waits until its stores have
// been acknowledged (`stores_done`, s_waitcnt vmcnt(0) in every wave, then a
// barrier if several waves share the tile) before the RMW that hands the data over, and a reader issues its
// loads only after the RMW that took the data over has returned.  This replaces
// agent-scope release/acquire fences, whose L2 write-back / invalidate on every
// tile visit cost far more than the visit itself.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "eik_rules.hpp"

namespace eik {

// Wait until every memory operation this wave issued has completed (device
// scope for the device-scope atomics used for shared data); also a compiler
// barrier.
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

constexpr uint32_t kQ = 1u, kR = 2u, kV = 4u, kS = 8u;
// statistics words (64-bit, cleared by every reset): [0] visits [1] point
// updates [2] relax passes [3] visit-cap count [4] adjoint reference time
// [5..8] phase clocks [9] unused [10] workgroups [11] bucket advances
// [12] hand-offs [13..15] residual accumulators [16] operator evaluations
// [17] improving evaluations [18] evaluations that set the final value
constexpr int kCounters = 24;
constexpr int kRings = 32;    // buckets of the window
constexpr int kShards = 8;    // rings per bucket
constexpr int kLookEvery = 16;            // idle polls between looks at the launch's progress
// Each ring counter (head, tail, count + running) lives in its own 256-byte
// line, so polling one does not slow the atomics on the others.
constexpr int kCtrPad = 64;                 // uint32 words per counter line
constexpr int kCtrStride = 4 * kCtrPad;     // uint32 words per ring
constexpr int kCrWord = 2 * kCtrPad;        // offset of the count + running word
// words of all ring counters and, after them, the live-work counters
constexpr int kPendWord = kRings * kShards * kCtrStride;
constexpr int kCtrWords = kPendWord + kShards * kCtrPad;
constexpr uint64_t kCountBias = 1ull << 31; // count is stored biased, so it may dip below 0
constexpr uint64_t kRunOne = 1ull << 32;

// device status flags
constexpr uint32_t kFlagDomain = 1u, kFlagLimit = 2u, kFlagBadSrc = 4u, kFlagWatchdog = 8u, kFlagBadStart = 16u;

struct Sched {
    uint64_t* items;     // [kRings * kShards][cap]
    uint32_t* ctr;       // ring counters, see ring_head / ring_tail / ring_cr
    uint32_t* tstate;    // [ntiles]
    int32_t* cur;        // lowest bucket of the window
    unsigned long long* counters;  // statistics: [0] visits [1] point updates [2] relax passes ...
    uint32_t* flags;     // device status flags
    int32_t* poisoned;   // set on a watchdog expiry: the next reset re-initialises the rings
    uint32_t cap_mask;
    double inv_delta;    // 1/delta, 0 => single bucket
    long long max_visits;  // 0 => unlimited
    int lookahead;       // claims may come from buckets cur .. cur + lookahead
    int strict;          // also those of an idle worker (claim_window)
    int horizon;         // 0, or k: a run settles only values below bucket (its bucket + k)
    int track;           // ablation operators: re-activate on any change (else on decrease)
    unsigned long long* timeline;  // NULL, or [0] start, [1] end, then (time, bucket) per advance
    int timeline_cap;    // advances the timeline can hold
};

__device__ __forceinline__ uint32_t* ring_head(const Sched& s, int r) { return s.ctr + r * kCtrStride; }
__device__ __forceinline__ uint32_t* ring_tail(const Sched& s, int r) { return s.ctr + r * kCtrStride + kCtrPad; }
__device__ __forceinline__ unsigned long long* ring_cr(const Sched& s, int r) {
    return (unsigned long long*)(s.ctr + r * kCtrStride + kCrWord);
}
__device__ __forceinline__ int32_t cr_count(uint64_t w) { return (int32_t)((int64_t)(w & 0xffffffffull) - (int64_t)kCountBias); }
__device__ __forceinline__ unsigned long long ld_cr(const Sched& s, int r) {
    return __hip_atomic_load(ring_cr(s, r), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Ring of a bucket in a shard; shard of a tile and of this workgroup.
__device__ __forceinline__ int ring_of(int64_t bucket, int shard) {
    return (int)(bucket & (kRings - 1)) * kShards + shard;
}
__device__ __forceinline__ int shard_of(uint32_t tile) {
    return (int)((tile ^ (((tile >> 3) * 0x9E3779B1u) >> 29)) & (kShards - 1));
}
// A run is counted as running in the ring it was claimed from.  Its slot names
// that ring and how far above `cur` its bucket was then:
// (bucket * kShards + shard) * kRings + (bucket - cur).  A run handed on keeps it.
__device__ __forceinline__ int64_t make_slot(int64_t bucket, int shard, int above) {
    return (bucket * kShards + shard) * kRings + above;
}
__device__ __forceinline__ int64_t slot_bucket(int64_t slot) { return slot / (kShards * kRings); }
__device__ __forceinline__ int slot_above(int64_t slot) { return (int)(slot & (kRings - 1)); }
__device__ __forceinline__ int slot_ring(int64_t slot) {
    return ring_of(slot_bucket(slot), (int)(slot / kRings) & (kShards - 1));
}
__device__ __forceinline__ int my_shard() { return (int)(blockIdx.x & (kShards - 1)); }

// Live work: per shard of the counting workgroup, the tiles ever queued (high
// half) and the runs ever ended (low half).  Both only grow, so "ended" summed
// first and "queued" summed afterwards can only be equal when nothing was
// queued or running in between.
__device__ __forceinline__ unsigned long long* pend_word(const Sched& s, int shard) {
    return (unsigned long long*)(s.ctr + kPendWord + shard * kCtrPad);
}
__device__ __forceinline__ void pend_add(const Sched& s, uint32_t queued, uint32_t ended) {
    __hip_atomic_fetch_add(pend_word(s, my_shard()), ((unsigned long long)queued << 32) + ended, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}
// Tiles ever queued, or runs ever ended, over all shards.  All 64 lanes.
__device__ __forceinline__ uint32_t pend_sum(const Sched& s, bool queued) {
    const int lane = threadIdx.x & 63;
    unsigned long long w = 0;
    if (lane < kShards)
        w = __hip_atomic_load(pend_word(s, lane), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    stores_done();  // these loads return before any later one goes out
    uint32_t v = queued ? (uint32_t)(w >> 32) : (uint32_t)w;
#pragma unroll
    for (int off = 1; off < kShards; off <<= 1) v += __shfl_xor(v, off);
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}
// True when no work is left anywhere.  All 64 lanes.
__device__ __forceinline__ bool all_done(const Sched& s) {
    const uint32_t ended = pend_sum(s, false);
    return ended == pend_sum(s, true);
}
__device__ __forceinline__ void cr_add(const Sched& s, int r, uint64_t v) {
    __hip_atomic_fetch_add(ring_cr(s, r), (unsigned long long)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int32_t ld_rlx(int32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void set_flag(const Sched& s, uint32_t f) {
    __hip_atomic_fetch_or(s.flags, f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (f & kFlagWatchdog)
        __hip_atomic_store(s.poisoned, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int64_t bucket_of(const Sched& s, double t) {
    if (s.inv_delta == 0.0) return 0;
    double k = floor(t * s.inv_delta);
    if (!(k < 1.0e15)) k = 1.0e15;
    return (int64_t)k;
}

// Bucket a push with time key `t` goes to, from a run in bucket `base` that was
// `above` buckets over `cur` when claimed (0, 0 before the solve starts): not
// below the run's own, and not so far up that it would alias a bucket behind
// `cur` (which never decreases).
__device__ __forceinline__ int64_t push_bucket(const Sched& s, double t, int64_t base, int above) {
    int64_t k = bucket_of(s, t);
    if (k < base) k = base;
    if (k > base - above + kRings - 1) k = base - above + kRings - 1;
    return k;
}

// Enqueue `tile` in bucket `k` (push_bucket).  The caller has already counted it
// as live work.  With count = false the ring's queued count is left to the
// caller, which must add it when or before it ends the run (publish folds it
// into the end-of-run RMW).  Single lane.
__device__ __forceinline__ void push_tile(const Sched& s, uint32_t tile, int64_t k, bool count = true) {
    const int r = ring_of(k, shard_of(tile));
    uint32_t pos = __hip_atomic_fetch_add(ring_tail(s, r), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uint64_t* cell = s.items + (size_t)r * (s.cap_mask + 1) + (pos & s.cap_mask);
    // wait until the previous lap's consumer has read this cell (bounded: that
    // consumer has already claimed it)
    for (long long spin = 0;; ++spin) {
        uint64_t it = __hip_atomic_load(cell, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if ((uint32_t)(it >> 32) == pos) break;
        if (spin > (1ll << 24)) {
            set_flag(s, kFlagWatchdog);
            return;
        }
        __builtin_amdgcn_s_sleep(1);
    }
    // everything this wave did before (the live-work count included) completes
    // before the item becomes claimable (it has: the cell was read after it);
    // the cell itself may arrive after the count, a claimer waits for it
    stores_done();
    __hip_atomic_store(cell, ((uint64_t)(pos + 1u) << 32) | tile, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (count) cr_add(s, r, 1);
}

// End of a run: its pushes were counted first (push_tile waits for that), so the
// bucket does not look drained while work it produced is in flight.  Single lane.
__device__ __forceinline__ void end_run(const Sched& s, int64_t slot) {
    stores_done();
    cr_add(s, slot_ring(slot), 0ull - kRunOne);
}

// Count a tile and enqueue it before the solve starts.  Single lane.
__device__ __forceinline__ void activate_push(const Sched& s, uint32_t tile, double t) {
    pend_add(s, 1, 0);
    push_tile(s, tile, push_bucket(s, t, 0, 0));
}

// Try to take one item from ring r: one RMW counts the claimer as running and
// takes one queued item.  Returns the tile, -1 (empty) or -2 (watchdog).
// Single lane.
__device__ __forceinline__ int try_claim(const Sched& s, int r) {
    const uint64_t old = __hip_atomic_fetch_add(ring_cr(s, r), (unsigned long long)(kRunOne - 1),
                                                __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (cr_count(old) <= 0) {
        cr_add(s, r, 0ull - (kRunOne - 1));
        return -1;
    }
    uint32_t pos = __hip_atomic_fetch_add(ring_head(s, r), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uint64_t* cell = s.items + (size_t)r * (s.cap_mask + 1) + (pos & s.cap_mask);
    // The producer that reserved this position is about to fill the cell.
    for (long long spin = 0;; ++spin) {
        uint64_t it = __hip_atomic_load(cell, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if ((uint32_t)(it >> 32) == pos + 1u) {
            // free the cell for the next lap
            __hip_atomic_store(cell, (uint64_t)(pos + s.cap_mask + 1u) << 32, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
            return (int)(uint32_t)it;
        }
        if (spin > (1ll << 24)) {
            set_flag(s, kFlagWatchdog);
            return -2;
        }
        __builtin_amdgcn_s_sleep(1);
    }
}

// Try to take up to `want` items from ring r with one RMW, which counts as many
// runs as started.  All 64 lanes of a wave; lane i < the returned number gets an
// item in `item`.  Returns -2 on a watchdog expiry.
__device__ __forceinline__ int try_claim_many(const Sched& s, int r, int want, int& item) {
    const int lane = threadIdx.x & 63;
    int got = 0;
    uint32_t pos = 0;
    if (lane == 0) {
        const uint64_t step = (kRunOne - 1) * (uint64_t)want;
        const uint64_t old = __hip_atomic_fetch_add(ring_cr(s, r), (unsigned long long)step, __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_AGENT);
        const int32_t have = cr_count(old);
        got = have <= 0 ? 0 : (have < want ? have : want);
        if (got < want) cr_add(s, r, 0ull - (kRunOne - 1) * (uint64_t)(want - got));
        if (got)
            pos = __hip_atomic_fetch_add(ring_head(s, r), (uint32_t)got, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    got = __builtin_amdgcn_readfirstlane(got);
    pos = (uint32_t)__builtin_amdgcn_readfirstlane((int)pos) + (uint32_t)lane;
    bool bad = false;
    if (lane < got) {
        uint64_t* cell = s.items + (size_t)r * (s.cap_mask + 1) + (pos & s.cap_mask);
        // the producer that reserved this position is about to fill the cell
        for (long long spin = 0;; ++spin) {
            const uint64_t it = __hip_atomic_load(cell, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if ((uint32_t)(it >> 32) == pos + 1u) {
                __hip_atomic_store(cell, (uint64_t)(pos + s.cap_mask + 1u) << 32, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
                item = (int)(uint32_t)it;
                break;
            }
            if (spin > (1ll << 24)) {
                set_flag(s, kFlagWatchdog);
                bad = true;
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
    }
    return __ballot(bad) ? -2 : got;
}

// Idle back-off: s_sleep takes an immediate, so sleep in units of 127.
__device__ __forceinline__ void idle_sleep(int units) {
    for (int i = 0; i < units; ++i) __builtin_amdgcn_s_sleep(127);
}

// Called by all 64 lanes of one wave.  `take(ring, count)` takes items from a
// ring that showed `count` queued ones and returns > 0 (taken), 0 (none left) or
// -2.  Returns what `take` returned and the slot (*slot: bucket and shard, counted
// as running there), or -1 when no work is left anywhere, or -2 on a watchdog expiry.
//
// A poll reads the count words of 8 buckets x 8 shards, one per lane, and `cur`
// in one round trip (`cur_hint` is the window's lowest bucket as this workgroup
// last saw it; the words are used only when `cur` still equals it), and the
// words of all other buckets, in one more, only when those show nothing.  It
// takes from the lowest bucket of its own shard, else from the lowest of the
// others.  A claim that comes too late costs two read-modify-writes on the very
// line the work comes through, so where few items face many claimers only some
// of them try: eight times as many as there are items, since most that could
// are busy (twice as many: 512x512x256 11.5 -> 11.7 ms, 32 shots 58.3 -> 59.1;
// 32 times: one shot of 256x256x128 11.0 -> 11.7, 8 uneven shots 17.9 -> 18.6).
//
// A workgroup that found nothing in kPatience polls looks kWide buckets far
// (claim_window; not with Sched::strict): it has nothing to lose, while waiting
// for a bucket of few tiles to drain costs every idle one a run's time
// (160x150x100, narrow buckets, no window: 13.2 ms kept to it, 2.7 ms looking
// past it; 512x512x256 110.8 and 18.3).  Further still costs more early runs than
// it saves waiting (13601x2801, tuned window: 31 ms with 16 buckets, 65 ms with
// all 32).  Three polls: after eight, the 160x150x100 case takes 3.2 instead of
// 2.9 ms and a shot 11.6 instead of 11.0, after one a shot 11.1.
//
// Every kLookEvery idle polls it looks whether the launch still makes progress
// (StallWatch: the runs ended so far and `cur`).  The count words would not do: a
// run that is handed on again and again, a front along a channel one tile wide,
// leaves all of them as they are.
//
// kMaxSleep caps the back-off (units of s_sleep(127), about 3.4 us); with few
// workgroups polling (64 or fewer) the cap is a quarter of one, as they cannot
// flood the counters and the front's next tile waits for the poll (16x16x16, 4
// tiles: 0.23 ms, 0.27 without; hundreds of workgroups: no difference either way).
template <int kMaxSleep, class Take>
__device__ __forceinline__ int claim_with(const Sched& s, int64_t* slot, int32_t& cur_hint, Take take) {
    const int lane = threadIdx.x & 63;
    int win = claim_window(s.lookahead, s.strict, 0);
    const int wide = claim_window(s.lookahead, s.strict, kPatience);
    const int own = my_shard();
    const int lj = lane / kShards, lsh = lane % kShards;
    constexpr int kCols = 64 / kShards;  // buckets read at once
    const unsigned long long own_lanes = 0x0101010101010101ull << own;
    static_assert(kShards == 8, "the lane masks below");
    constexpr int kParts = kRings / kCols;
    uint32_t idle = 0;   // polls so far (sets the back-off; 64 bits cost 13601x2801 1%: 30.0 / 29.6 ms)
    StallWatch watch;
    uint32_t rnd = (uint32_t)wall_clock64() * 0x9E3779B1u + blockIdx.x * 0x85EBCA6Bu;
    for (;;) {
        const int32_t c = cur_hint;
        const int32_t cnow = ld_rlx(s.cur);
        unsigned long long w[kParts];
        w[0] = ld_cr(s, ring_of((int64_t)c + lj, lsh));
        if (cnow != c) {
            cur_hint = cnow;
            continue;
        }
        int first = 0;  // bucket (from c) of w[at]'s lane 0
        unsigned long long at = w[0];
        unsigned long long mask = __ballot(lj < win && cr_count(at) > 0);
        bool moved = false;
        if (!mask) {
#pragma unroll
            for (int p = 1; p < kParts; ++p) w[p] = ld_cr(s, ring_of((int64_t)c + p * kCols + lj, lsh));
            int from = 0;
            if (!__ballot(lane < kShards && w[0] != kCountBias)) {
                // bucket `cur` drained: move to the next bucket that has work
                // queued or still running.  A bucket whose runs (taken through
                // the lookahead window) are still live is not skipped: their
                // pushes may land in it, and its rings must not be reused for a
                // later bucket meanwhile.  (The words are not read at one
                // instant, so a push may be missed that goes to a word read
                // before it from a run whose end is seen: the bucket then counts
                // as kRings later, which only delays it.)
                int next = 0;
#pragma unroll
                for (int p = kParts - 1; p >= 0; --p) {
                    unsigned long long m2 = __ballot(w[p] != kCountBias);
                    if (p == 0) m2 &= ~0xFFull;
                    if (m2) next = p * kCols + (__ffsll((long long)m2) - 1) / kShards;
                }
                if (next) {
                    int32_t expect = c;
                    if (lane == 0) {
                        if (__hip_atomic_compare_exchange_strong(s.cur, &expect, c + next, __ATOMIC_RELAXED,
                                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                            expect = c + next;
                            const unsigned long long i = __hip_atomic_fetch_add(s.counters + 11, 1ull, __ATOMIC_RELAXED,
                                                                                __HIP_MEMORY_SCOPE_AGENT);
                            if (s.timeline && i < (unsigned long long)s.timeline_cap) {
                                __hip_atomic_store(s.timeline + 2 + 2 * i, (unsigned long long)wall_clock64(),
                                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                                __hip_atomic_store(s.timeline + 3 + 2 * i, (unsigned long long)(c + next),
                                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                            }
                        }
                    }
                    cur_hint = __builtin_amdgcn_readfirstlane(expect);
                    if (cur_hint != c + next) continue;  // another workgroup moved it
                    from = next;                         // the window now starts there
                    moved = true;
                } else {
                    if (all_done(s)) return -1;
                }
            }
            // lowest bucket of the window with work
#pragma unroll
            for (int p = kParts - 1; p >= 0; --p) {
                const int j = p * kCols + lj;
                const unsigned long long m = __ballot(j >= from && j < from + win && cr_count(w[p]) > 0);
                if (m) {
                    mask = m;
                    at = w[p];
                    first = p * kCols;
                }
            }
        }
        if (mask) {
            const unsigned long long mine = mask & own_lanes;
            int l;
            if (mine) {
                l = __ffsll((long long)mine) - 1;
            } else {
                // lowest bucket with work; of its shards the next after this one's
                const int jl = (__ffsll((long long)mask) - 1) & ~(kShards - 1);
                const uint32_t sh = (uint32_t)(mask >> jl) & 0xFFu;
                const uint32_t rot = ((sh | (sh << 8)) >> own) & 0xFFu;
                l = jl + ((__ffs((int)rot) - 1 + own) & (kShards - 1));
            }
            const int32_t count = cr_count(__shfl(at, l));
            // claimers this ring may have: this shard's workgroups, or all
            const uint32_t rivals = mine ? (gridDim.x + kShards - 1) / kShards : gridDim.x;
            rnd = (uint32_t)__builtin_amdgcn_readfirstlane((int)(rnd * 1664525u + 1013904223u));
            if ((uint32_t)count * 8u >= rivals || (rnd >> 16) * (uint64_t)rivals < (uint64_t)count * 8u * 65536u) {
                const int64_t bucket = (int64_t)c + first + l / kShards;
                const int got = take(ring_of(bucket, l % kShards), count);
                if (got > 0) {
                    *slot = make_slot(bucket, l % kShards, (int)(bucket - cur_hint));
                    return got;
                }
                if (got == -2) return -2;
            }
            __builtin_amdgcn_s_sleep(8);
            continue;
        }
        if (moved) continue;
        ++idle;
        if (idle >= kPatience) win = wide;
        if (idle % kLookEvery == 0) {
            const uint64_t progress = ((uint64_t)(uint32_t)c << 32) | pend_sum(s, false);
            if (watch.gives_up(progress, ld_rlx(s.poisoned) != 0, wall_clock64())) {
                if (lane == 0) set_flag(s, kFlagWatchdog);
                return -2;
            }
        }
        // exponential back-off from about 0.1 us keeps idle workgroups from
        // flooding the counters the busy ones need
        if (idle < 2) __builtin_amdgcn_s_sleep(4);
        else if (idle < 3) __builtin_amdgcn_s_sleep(16);
        else if (idle < 4) __builtin_amdgcn_s_sleep(64);
        else if (kMaxSleep == 1 && gridDim.x <= 64) __builtin_amdgcn_s_sleep(32);
        else idle_sleep(min(kMaxSleep, idle < 5 ? 1 : (idle < 6 ? 2 : (idle < 7 ? 4 : 8))));
    }
}

// One tile for a block of its own (the block-per-tile kernels).
template <int kMaxSleep>
__device__ __forceinline__ int claim(const Sched& s, int64_t* slot, int32_t& cur_hint) {
    int tile = -1;
    const int rc = claim_with<kMaxSleep>(s, slot, cur_hint, [&](int r, int32_t) {
        int got = -1;
        if ((threadIdx.x & 63) == 0) got = try_claim(s, r);
        got = __shfl(got, 0);
        tile = got;
        return got >= 0 ? 1 : (got == -2 ? -2 : 0);
    });
    return rc > 0 ? tile : rc;
}

// Work for the waves of one block that each run tiles of their own.  A wave
// without work registers as idle; one idle wave at a time polls the rings for
// all of them and takes several items with one RMW, so the shared counters see
// one poller per block (a read-modify-write of one address completes about
// every 12 ns on this device whoever issues it, so thousands of polling waves
// would slow every push and claim).
struct GroupMail {
    int lock;
    unsigned int idle;       // waves waiting for work
    int tile[16];            // per wave: kNoMail, or the tile handed to it
    int64_t slot[16];
};
constexpr int kNoMail = -3;

// As claim(), for wave `w` of the block.
__device__ __forceinline__ int claim_group(const Sched& s, GroupMail& g, int w, int64_t* slot, int32_t& cur_hint) {
    const int lane = threadIdx.x & 63;
    if (lane == 0) {
        __hip_atomic_store(&g.tile[w], kNoMail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __hip_atomic_fetch_or(&g.idle, 1u << w, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    for (;;) {
        int tile = kNoMail;
        int locked = 0;
        if (lane == 0) {
            tile = __hip_atomic_load(&g.tile[w], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (tile == kNoMail) {
                locked = __hip_atomic_exchange(&g.lock, 1, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) == 0;
                // work may have been handed over before the lock was free
                if (locked) tile = __hip_atomic_load(&g.tile[w], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        }
        tile = __builtin_amdgcn_readfirstlane(tile);
        locked = __builtin_amdgcn_readfirstlane(locked);
        if (tile != kNoMail) {
            if (locked && lane == 0)
                __hip_atomic_store(&g.lock, 0, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
            *slot = g.slot[w];
            return tile;
        }
        if (!locked) {
            __builtin_amdgcn_s_sleep(4);
            continue;
        }
        int item = -1;
        int64_t b = 0;
        unsigned int who = 0;
        const int got = claim_with<1>(s, &b, cur_hint, [&](int r, int32_t count) {
            who = (unsigned int)__builtin_amdgcn_readfirstlane(
                (int)__hip_atomic_load(&g.idle, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
            // a share of what is queued, so that the blocks' waves fill evenly (a
            // quarter or a 64th instead of a 16th: 8 uneven shots 17.9 -> 17.8 and
            // 18.4 ms, all else within 1%)
            const int want = max(1, min(__popc(who), count >> 4));
            return try_claim_many(s, r, want, item);
        });
        int mine = got;
        if (got > 0) {
            // this wave takes item 0, the next idle waves the others
            mine = __builtin_amdgcn_readfirstlane(item);
            unsigned int rest = who & ~(1u << w), gone = 1u << w;
            for (int i = 1; i < got; ++i) {
                const int o = __ffs(rest) - 1;
                rest &= rest - 1;
                gone |= 1u << o;
            }
            if (lane == 0) __hip_atomic_fetch_and(&g.idle, ~gone, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            rest = who & ~(1u << w);
            for (int i = 1; i < got; ++i) {
                const int o = __ffs(rest) - 1;
                rest &= rest - 1;
                const int t = __shfl(item, i);
                if (lane == 0) {
                    g.slot[o] = b;
                    __hip_atomic_store(&g.tile[o], t, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            }
            *slot = b;
        } else if (lane == 0) {
            __hip_atomic_fetch_and(&g.idle, ~(1u << w), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        if (lane == 0) __hip_atomic_store(&g.lock, 0, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
        return mine;
    }
}

// End of a run of `tile`, executed by the 64 lanes of wave 0 after every wave
// of the block has written its results and waited for them (stores_done).
// Lane f < 6 holds, for face f,
//   nb      bit 30 set when the neighbour across it exists,
//   nid     its tile id, face the priority key bits of the lowered values on
//           the face (kInfBits: nothing lowered there);
//   first   the run wrote this tile's interior for the first time (sets V).
// The tile's own state word drops R (and gains V); the RMW's return also says
// whether the tile was activated during the run.  Lanes 0..5 activate the
// neighbours in parallel with it.
// The live work counts the newly queued neighbours, a requeue and this run's end
// at once, before any push makes new items claimable, so it never under-counts.
// `self_key` (bits of a time, kInfBits for none) requeues the tile itself with
// at most that key: the run left points whose new values lie beyond its
// bucket.
// With `cont`, one tile that falls in this run's own bucket is not pushed: it is
// returned (state Q, counted live and counted running in this run's slot) for the
// caller to run next, which saves a push, a poll and a claim on the front's
// critical path: the tile itself if it was activated meanwhile (a front that
// runs along a face between two tiles activates them in turn), else the
// lowest-key newly activated neighbour.  With the tile itself first, before and
// after: 256x256x128 layered, corner source, 8x8x8 tiles, forward 4.94 -> 4.07 ms
// and its adjoint (16x8x8) 8.63 -> 7.46 ms; 32 such shots at once, forward
// 23.6 -> 22.2 ms, adjoint 33.5 -> 31.7 ms.  Returns that tile or -1 (the run has
// then ended), uniform across the wave.
__device__ __forceinline__ int publish_wave(const Sched& s, uint64_t* tkey, uint32_t tile, int64_t slot, bool first,
                                            uint32_t nb, uint32_t nid, unsigned long long face, bool cont,
                                            unsigned long long self_key) {
    const int lane = threadIdx.x & 63;
    const int64_t bucket = slot_bucket(slot);
    const int above = slot_above(slot);
    // lane 6 updates the tile's own word alongside the activations of lanes 0-5:
    // runs read halos without looking at V (t starts at +inf, mu at NaN), so V
    // needs no order against them
    constexpr int ol = 6;
    uint32_t own = 0;
    if (lane == ol) {
        // work of this tile left for a later bucket: activate the tile itself
        // while R still keeps everyone else from pushing it
        if (self_key != kInfBits)
            __hip_atomic_fetch_or(s.tstate + tile, kQ, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        own = __hip_atomic_fetch_xor(s.tstate + tile, kR | (first ? kV : 0u), __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_AGENT);
    }
    bool want = false;
    uint32_t n = 0;
    unsigned long long fk = kInfBits;
    if (lane < 6) {
        fk = face;
        if ((nb & 0x40000000u) && fk != kInfBits) {
            n = nid;
            uint32_t old = __hip_atomic_fetch_or(s.tstate + n, kQ, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if ((old & (kQ | kR)) == 0) {
                want = true;
            } else if (old & kR) {
                __hip_atomic_fetch_min((unsigned long long*)(tkey + n), fk, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
    own = __shfl(own, ol);
    const int64_t to = push_bucket(s, as_f64(fk), bucket, above);
    const bool requeue = (own & kQ) != 0;
    const unsigned long long wm = __ballot(want);
    const int k = __popcll(wm);
    int64_t self_to = 0;
    if (requeue) {
        if (lane == 0) {
            uint64_t kb = __hip_atomic_exchange((unsigned long long*)(tkey + tile), kInfBits, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT);
            if (self_key < kb) kb = self_key;
            self_to = push_bucket(s, kb == kInfBits ? 0.0 : as_f64(kb), bucket, above);
        }
        self_to = __shfl(self_to, 0);
    }
    const bool again = cont && requeue && self_to == bucket;
    int cl = -1;
    if (cont && wm && !again) {
        const bool cand = want && to == bucket;
        unsigned long long key = cand ? fk : ~0ull;
        // minimum over lanes 0..7 (the six face lanes)
#pragma unroll
        for (int off = 1; off < 8; off <<= 1) {
            const unsigned long long o = __shfl_xor(key, off);
            key = o < key ? o : key;
        }
        key = __shfl(key, 0);
        const unsigned long long cm = __ballot(cand && fk == key);
        if (cm) cl = __ffsll((long long)cm) - 1;
    }
    if (lane == 0) pend_add(s, (uint32_t)k + (requeue ? 1u : 0u), 1u);
    // Pushes into this run's own ring leave their queued count to the one
    // RMW below, which also ends the run, so the bucket never looks drained with
    // work of it uncounted.  Pushes to other rings count themselves, and that
    // completes before the RMW.
    const int ring = slot_ring(slot);
    const bool pushme = want && lane != cl;
    const bool same = pushme && ring_of(to, shard_of(n)) == ring;
    if (pushme) push_tile(s, n, to, !same);
    bool rq_same = false;
    if (lane == 0 && requeue && !again) {
        rq_same = ring_of(self_to, shard_of(tile)) == ring;
        push_tile(s, tile, self_to, !rq_same);
    }
    const uint64_t nsame = (uint64_t)__popcll(__ballot(same)) + (uint64_t)__popcll(__ballot(rq_same));
    const bool away = __ballot(pushme && !same) != 0 || __ballot(lane == 0 && requeue && !again && !rq_same) != 0;
    if (cl >= 0 || again) {
        if (lane == 0 && nsame) cr_add(s, ring, nsame);
        return again ? (int)tile : (int)__shfl(n, cl);
    }
    // this run's own pushes are counted: the bucket it came from may now drain
    if (away) stores_done();
    if (lane == 0) cr_add(s, ring, nsame - kRunOne);
    return -1;
}

// The same with the six faces' values in memory shared by the block.
__device__ __forceinline__ int publish(const Sched& s, uint64_t* tkey, uint32_t tile, int64_t slot, bool first,
                                       const uint32_t* nb, const uint32_t* nid,
                                       const unsigned long long* face, bool cont = false,
                                       unsigned long long self_key = kInfBits) {
    const int lane = threadIdx.x & 63;
    const bool in = lane < 6;
    return publish_wave(s, tkey, tile, slot, first, in ? nb[lane] : 0u, in ? nid[lane] : 0u,
                        in ? face[lane] : kInfBits, cont, self_key);
}

// Drop a claimed tile without running it (visit cap reached).  Lane 0.
__device__ __forceinline__ void drop_run(const Sched& s, uint32_t tile, int64_t slot) {
    const uint32_t old = __hip_atomic_fetch_xor(s.tstate + tile, kR, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    pend_add(s, (old & kQ) ? 1u : 0u, 1u);
    if (old & kQ) push_tile(s, tile, slot_bucket(slot));
    end_run(s, slot);
}

}  // namespace eik
