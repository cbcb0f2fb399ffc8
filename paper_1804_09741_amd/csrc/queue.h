// The order in which the persistent waves of a launch take its work units:
// the index arithmetic of unit_loop (esu.h), which owns the atomics.  No
// device code, so that a host program can walk it.
#pragma once

#include <cstdint>

namespace mk {

constexpr int kQueues = 8;  // one queue per XCD of the MI355X

// Compile-time tuning knob (build flags may override it).
#ifndef MK_HEAVY_GRAB
#define MK_HEAVY_GRAB 4  // units per grab of the first sweep, in grabs of the second
#endif

// One wave's view of a launch of `grid` waves over the units [begin, begin +
// span).  The units are cut into kQueues ranges with a head each: range x is
// the units [lo_x, lo_{x+1}), or (mix) every eighth grab of all units.
struct UnitQueue {
    uint32_t begin, span;
    uint32_t chunk;     // units per grab
    uint32_t chunk0;    // and in a first sweep
    int home;           // the range the wave starts on
    int tries;          // ranges it looks into after its own
    uint32_t turn;      // which of them comes first, where it does not try all
    bool two;           // swept twice: heavy units, then the rest
    bool mix;
};

__host__ __device__ __forceinline__ UnitQueue unit_queue(uint32_t begin, uint32_t end,
                                                         uint32_t grid, uint32_t wave,
                                                         uint32_t cfg_chunk, bool heavy_first,
                                                         bool mix)
{
    UnitQueue q;
    q.begin = begin;
    q.span = end > begin ? end - begin : 0u;
    // units per grab: about 1/32 of a wave's share, 1..16
    uint32_t chunk = cfg_chunk ? cfg_chunk : q.span / (grid * 32u);
    chunk = chunk < 1u ? 1u : (chunk > 256u ? 256u : chunk);
    if (!cfg_chunk && chunk > 16u) chunk = 16u;
    // two sweeps only with at least 32 units per wave (a launch of one
    // graph's units would leave most waves idle behind a few heavy grabs);
    // the first sweep's grabs: MK_HEAVY_GRAB times as many units, at most 64
    // (a grab's marks are read by the lanes of one wave)
    q.two = heavy_first && q.span >= grid * 32u;
    q.chunk = chunk;
    q.chunk0 = chunk * MK_HEAVY_GRAB < 64u ? chunk * MK_HEAVY_GRAB : 64u;
    q.mix = mix;
    q.home = (int)(wave % (uint32_t)kQueues);
    // Ranges a wave looks into after its own.  A visit is an atomic on a head
    // that all eight XCDs share, about 10 ns one after another, and most
    // visits find the range empty.  So launches with many units a wave visit
    // every range (the walk's time hides it, and ranges of unlike graphs
    // need it); in the others a wave tries one, in turn.  8,327 units on 6,144
    // waves (k = 4, n = 2000, m = 10000): 7 visits 0.181 ms of kernel, 2
    // 0.109, 1 0.096, none 0.090; k = 5 by enumeration, n = 1000, m = 3000,
    // 26,895 units on 7,168 waves: 0.62 ms with 1 or 2, 0.64 with none.
    // (Launches of 8 waves and more have a home wave on every range, which
    // empties it whoever else comes.)
    q.tries = q.span / grid >= 16u || grid < 8u * kQueues ? kQueues - 1 : 1;
    q.turn = q.tries < kQueues - 1 ? wave / (uint32_t)kQueues : 0u;
    return q;
}

// units per grab in sweep 0 (the heavy units) or 1
__host__ __device__ __forceinline__ uint32_t queue_chunk(const UnitQueue &q, int sweep)
{
    return sweep == 0 ? q.chunk0 : q.chunk;
}

// the t-th range (0..tries) that the wave looks into
__host__ __device__ __forceinline__ int queue_range(const UnitQueue &q, int t)
{
    return t == 0 ? q.home
                  : (int)((uint32_t)(q.home + 1) +
                          (q.turn + (uint32_t)t - 1u) % (uint32_t)(kQueues - 1)) %
                        kQueues;
}

// The units [first, stop) of the grab that moved range x's head on from
// `head` in a sweep; false when the range has none left.
__host__ __device__ __forceinline__ bool queue_grab(const UnitQueue &q, int x, int sweep,
                                                    uint32_t head, uint32_t &first, uint32_t &stop)
{
    const uint32_t ch = queue_chunk(q, sweep);
    // the range, from q.begin on
    const uint32_t lo = q.mix ? (uint32_t)x * ch : (uint32_t)((uint64_t)q.span * (uint32_t)x / kQueues);
    const uint32_t hi =
        q.mix ? q.span : (uint32_t)((uint64_t)q.span * (uint32_t)(x + 1) / kQueues);
    // (compared before it is multiplied or added, so that all sums stay in 32
    // bits)
    if (q.mix && head > q.span / (uint32_t)kQueues) return false;
    const uint32_t at = q.mix ? head * (uint32_t)kQueues : head;
    if (lo >= hi || at >= hi - lo) return false;
    first = q.begin + lo + at;
    const uint32_t left = hi - lo - at;
    stop = first + (left > ch ? ch : left);
    return true;
}

}  // namespace mk
