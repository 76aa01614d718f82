// Picking the way a whole-tree schedule is served at streaming size: the
// order in which the fold kernel goes through the payload, and with it whether
// results stream past the memory-side cache.
//   1  the trees taking turns of 128 KiB of every rank (section 4.2.2; chunk by chunk where a stage
//      reads more than 8 ranks: 16 x 16 streams at a time are too many)
//   2  one front through the payload, one tree's share after the other
//   3  chunk by chunk across the trees (several trees, at most 8 ranks)
// Which is fastest depends on where the buffers lie in HBM and how far apart the
// trees' shares are, in ways addresses do not reveal.  With a standalone probe
// (8 ranks, 4 trees, buffers in allocations of their own, three sets in turn; us for
// ways 1 / 2): 64 MiB per rank 182 / 163, 114 MiB 324 / 294, 400 MiB 1119 / 1042, but
// 256 MiB, where the shares are a power of two apart, 658 / 691.  So the first calls on
// such a schedule go round the candidates, kTrialSamples times each, each call timed
// with a pair of events on the caller's stream; the next call waits for the last of
// them (the one time a call waits for the device, besides a schedule's first) and
// the candidate with the smallest minimum serves the rest.  All give the same
// bits.
//
// Only like calls are compared: sums, whose time does not depend on the element type (8 x
// 64 MiB, way 1, fp32 / int32: 184.1 / 184.3 us), and the other operators on either type
// (largest value: 189.3 / 182.8) each have a round of their own, and the first round that is
// complete decides for all.  Timed calls go to and fro like all others, so each starts on what
// the call before it left in the memory-side cache; that call was of another way.  (Timed
// all forwards, on cold data, 8 x 256 MiB in allocations of their own chose way 2: repeated in
// place 748 us a call, against 705 with way 1, which gains by what the call before it left.)
// No HIP in here.
#pragma once
#include <algorithm>
#include <cstdint>

namespace blink {

constexpr int kTrialSamples = 4;
constexpr int kMostWays = 3;
constexpr int kTrialClasses = 3;
inline int trial_class(bool sum, bool fp32) { return sum ? 0 : fp32 ? 1 : 2; }

struct WayTrial {
    int picked = 0;                    // the way once picked (1, 2 or 3); 0 = not yet
    int calls[kTrialClasses] = {};     // timed calls launched so far
};

// The ways a schedule has.  can_front, can_turns: ways 2 and 3 are among them.
struct Ways {
    int way[kMostWays] = {1, 0, 0};
    int count = 1;
    bool front = false;
};
inline Ways ways_of(bool can_front, bool can_turns) {
    Ways w;
    w.front = can_front;
    if (can_front) w.way[w.count++] = 2;
    if (can_turns) w.way[w.count++] = 3;
    return w;
}
// The way of a class's next timed call, or 0: all have been launched.
inline int timed_way(const WayTrial& t, const Ways& w, int cls) {
    return t.calls[cls] < w.count * kTrialSamples ? w.way[t.calls[cls] % w.count] : 0;
}

// Way 2, or way 1 where there is none, gets the schedule unless another beats it by more
// than the 2 % by which such minima scatter from one trial to the next: it is the fastest
// or within 1 % of it on most shapes (three sets of buffers in turn, us for ways 1 / 2 / 3:
// two servers of 8 x 64 MiB 344 / 336 / -, 6 ranks x 97.6 MiB 209 / 196 / 204, 8 x 230 MiB
// 664 / 614 / 634; the other way round 8 x 256 MiB 717 / 735 / 786).
// ms: the times of a class's calls in the order of their launch.  Each candidate's first is
// left out: it carries what happens once (the code's first launch, tables not yet in any
// cache).  Kernels of a tenth of a millisecond differ by a few percent, which is also
// what the event pair around a single launch scatters by: hence three samples each.
inline int fastest_way(const Ways& w, const float* ms) {
    float best[kMostWays] = {1e30f, 1e30f, 1e30f};
    for (int c = w.count; c < w.count * kTrialSamples; ++c) best[c % w.count] = std::min(best[c % w.count], ms[c]);
    int fastest = w.front ? 1 : 0;
    float bar = best[fastest] * 0.98f;
    for (int i = 0; i < w.count; ++i)
        if (best[i] < bar) {
            fastest = i;
            bar = best[i];
        }
    return w.way[fastest];
}

}  // namespace blink
