// Picking the way a whole-tree schedule is served at streaming size: the
// order in which the fold kernel goes through the payload, and with it whether
// results stream past the memory-side cache.
//   1  the trees taking turns of 128 KiB of every rank (section 4.2.2; chunk by chunk where a stage
//      reads more than 8 ranks: 16 x 16 streams at a time are too many)
//   2  one front through the payload, one tree's share after the other
//   3  chunk by chunk across the trees (several trees, at most 8 ranks)
// Which is fastest depends on where the buffers lie in HBM, how far apart the trees' shares are and whether a call finds
// its buffers where the one before it left them, in ways addresses do not reveal.  us for ways 1 / 2 / 3, three sets of
// buffers in turn, and repeated in place:
//   8 ranks x  40 MiB   114 / 109 / 111    94 /  94 /  94      6 ranks x  98 MiB   205 / 191 / 199   187 / 189 / 182
//              64 MiB   180 / 167 / 173   161 / 169 / 162                400 MiB   791 / 770 / 783   769 / 763 / 764
//             114 MiB   318 / 298 / 313   303 / 305 / 299      5 ranks x  98 MiB   168 / 163 / 167   147 / 145 / 147
//             230 MiB   648 / 607 / 634   630 / 604 / 607                400 MiB   713 / 662 / 700   683 / 675 / 684
//             256 MiB   673 / 747 / 879   665 / 695 / 722      4 ranks x 500 MiB   679 / 639 / 667   655 / 640 / 652
//             400 MiB  1084 /1071 /1102  1147 /1093 /1178      two servers of 8, 64 MiB  347 / 336 / -   331 / 338 / -
// (256 MiB: the shares are a power of two apart.)  So the first calls on
// such a schedule go round the candidates, kTrialSamples times each, each call timed
// with a pair of events on the caller's stream; the next call waits for the last of
// them (the one time a call waits for the device, besides a schedule's first) and
// the candidate with the smallest minimum serves the rest.  All give the same
// bits.
//
// Only like calls are compared: sums, whose time does not depend on the element type (8 x
// 64 MiB, way 1, fp32 / int32: 176 / 178 us), and the other operators on either type, which have kernels of their
// own (largest value: 177 / 177), each have a round of their own, and the first round that is
// complete decides for all.  Timed calls go to and fro like all others, so each starts on what
// the call before it left in the memory-side cache; that call was of another way.  (Timed
// all forwards, on cold data, 8 x 256 MiB in allocations of their own chose way 2 with the kernel before this one: repeated in
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
// than the 2 % by which such minima scatter from one trial to the next: on changing buffers it is 1 to 8 % ahead
// on all shapes above but the one of shares a power of two apart; in place it is the fastest or level on half of them and
// 2 to 5 % behind on the others, which the timed calls show.
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
