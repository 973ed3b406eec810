// In-kernel, deterministic combination of K-slab partial sums (no second kernel, no float atomics).
//
// Every block writes the fp32 partial sums of its (row tile, K slab) to the workspace and, when it
// has finished all its tiles, bumps each tile's arrival counter.  The block that arrives last at a
// tile adds the partials of ALL slabs in slab order - so the result does not depend on which
// block happened to be last - rounds to bf16 and stores y.  Counters live at the start of the
// workspace as 64-bit words (tag << 8 | arrivals) with a fixed 56-bit tag.  A word that does not
// carry the tag (never-initialised memory, or memory an earlier call used for something else)
// counts as zero arrivals, so the workspace needs no initialisation; the last block puts the
// counter back to (tag, 0), so every completed call leaves its counters clean - for the next call
// and for any number of replays of a captured launch.
#pragma once
#include "any4_device.h"

namespace any4 {

constexpr int kMaxSplit = 64;

__host__ __device__ inline size_t splitk_counter_bytes(int64_t tiles) { return (size_t)((tiles * 8 + 255) / 256 * 256); }

// Partial sums and counters are exchanged between blocks that may run on different XCDs (each
// with its own L2).  Instead of device-wide fences - which write back and invalidate whole caches
// and were measured to cost tens of microseconds per launch here - every access to them is a
// relaxed agent-scope atomic (coherent by itself: such accesses are served by the memory side of
// the cache hierarchy, never by a cache private to a compute unit or XCD), and ordering comes from
// waiting for the stores' completion (s_waitcnt vmcnt(0) plus a block barrier) before the counter
// is bumped: a store that has completed at that level is visible to every later agent-scope load,
// and the reader's loads are issued only after its own atomic on the counter has returned.
__device__ __forceinline__ void splitk_store(float* p, float v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float splitk_load(const float* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One arrival at a tile's counter by a single thread; true if this was the last of `ksplit`.
// The caller has made its partial sums visible (stores issued and waited for) beforehand.
// A counter word is (tag << 8 | arrivals).  The last arrival of a tile puts its counter back to
// "tag, 0", so a workspace that has served a call is clean for the next one and an arrival is ONE
// atomic add; a word without the tag (a workspace used for the first time, or memory that held
// something else) is claimed with a compare-and-swap instead.
constexpr unsigned long long kArriveTag = 0x00A4C0DE5EED17ull;          // 56 bits
__device__ __forceinline__ bool arrive_one(unsigned long long* c, int ksplit) {
    // a word is this call's own only if it carries the tag AND fewer than ksplit arrivals: a tagged word
    // with more (left by a launch that never finished, or by a call with another slab count that
    // shared the memory) is treated like memory that held something else
    auto own = [&](unsigned long long v) -> bool { return (v >> 8) == kArriveTag && (v & 0xFFull) < (unsigned long long)ksplit; };
    unsigned long long old = __hip_atomic_fetch_add(c, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    unsigned long long cnt;
    if (own(old)) {
        cnt = (old & 0xFFull) + 1ull;
    } else {
        // the add above went into a foreign word and is dropped with it
        old += 1ull;
        for (;;) {
            cnt = own(old) ? (old & 0xFFull) + 1ull : 1ull;
            const unsigned long long nv = (kArriveTag << 8) | cnt;
            if (__hip_atomic_compare_exchange_strong(c, &old, nv, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT))
                break;
        }
    }
    const bool last = cnt == (unsigned long long)ksplit;
    if (last) __hip_atomic_store(c, kArriveTag << 8, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return last;
}

// A meeting, for a tile's slabs or slices (at most 64) whose blocks share the adding.  Slabs of a tile meet at a word: arrivals (8 bits), the parts whose owners have left (8 bits), a bit that every completed
// meeting turns over, a tag.  The sums of a tile are `parts` parts; part k belongs to slab k.  A slab that has brought its sums waits a
// while for the others; if all have come it adds its part of all slabs, otherwise it leaves, and the last slab to come adds the parts
// of those that have left.  So blocks that end together share the adding, and nobody depends on anybody who may not be running.  Returns
// the parts (bits) that the block is to add.  By one thread, after the block's sums are out.
//
// The last to arrive puts the word back for the next meeting; the bit then tells those who still look at it.  A word that is not
// of this kind (memory used for the first time, or for something else) counts as no arrivals, as above.  (Marks that
// a launch which never finished has left only have a part added twice.  Arrivals that it has left, fewer than `slabs`, count for the
// next meeting, which then ends before all sums are there: a workspace is cleared or replaced after such a launch.)
//
// One block adding all the sums of a tile took 8 - 12 000 cycles (a compute unit reads 20 - 26 bytes a cycle of what others wrote; 256 KB of
// eight slabs at 64 rows of x, 1 MB at 128): 4096 x 4096 at M = 64 / 128 18.5 / 34.2 -> 16.4 / 24.3 us, 4096 x 14336 29.0 / 54.2 -> 26.5 / 39.2.
// (the words of blocks that look at them lie in cache lines of their own: packed, a sum took up to 11 000 cycles more to get out, and
// an arrival as many, however seldom the blocks looked)
constexpr int kWordBytes = 64;
constexpr unsigned long long kMeetTag = 0x24B47C5EED17ull << 17;
constexpr int kMaxParts = 8, kLooks = 10;                      // looks: about 0.4 us each
__device__ __forceinline__ uint32_t meet(unsigned long long* word, int slabs, int parts, int slab, int looks = kLooks) {
    constexpr unsigned long long kTag = kMeetTag, kTurn = 1ull << 16, kCount = 0xFFull;
    const unsigned long long all = (unsigned long long)slabs;
    auto own = [&](unsigned long long v) -> bool { return (v >> 17) == (kTag >> 17) && (v & kCount) < all; };
    unsigned long long old = __hip_atomic_fetch_add(word, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (!own(old)) {
        // the add above went into a foreign word and is dropped with it
        unsigned long long seen = old + 1ull;
        for (;;) {
            old = own(seen) ? seen : kTag;
            if (__hip_atomic_compare_exchange_strong(word, &seen, old + 1ull, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) break;
        }
    }
    const uint32_t bit = slab < parts ? 1u << slab : 0u;       // this slab's part
    if ((old & kCount) + 1ull == all) {
        __hip_atomic_store(word, kTag | (~old & kTurn), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return parts == 1 ? 1u : bit | ((uint32_t)(old >> 8) & 0xFFu);
    }
    if (parts == 1 || bit == 0u) return 0u;
    auto complete = [&](unsigned long long v) -> bool { return ((v ^ old) & kTurn) != 0ull || (v & kCount) == all; };
    for (int look = 0; look < looks; ++look) {
        if (complete(__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) return bit;
        __builtin_amdgcn_s_sleep(8);
    }
    const unsigned long long mark = (unsigned long long)bit << 8;
    const unsigned long long left = __hip_atomic_fetch_or(word, mark, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (!complete(left)) return 0u;
    // the last came in between and counts on this slab; its mark comes off the word where it went into the next meeting's
    if ((left ^ old) & kTurn) __hip_atomic_fetch_and(word, ~mark, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return bit;
}

}  // namespace any4
