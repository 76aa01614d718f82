// Plays the timed choice among the ways to serve a schedule through a list of calls:
//   way_trial_check CAN_FRONT CAN_TURNS  CLASS CLASS ...
// one line per call: class, way, timed.  Every call of way 3 takes 1 ms, of way 2
// 2 ms, of way 1 3 ms.
#include <cstdio>
#include <cstdlib>

#include "way_trial.hpp"

int main(int argc, char** argv) {
    const blink::Ways ways = blink::ways_of(std::atoi(argv[1]) != 0, std::atoi(argv[2]) != 0);
    blink::WayTrial trial;
    float ms[blink::kTrialClasses][blink::kMostWays * blink::kTrialSamples] = {};
    for (int call = 0; call + 3 < argc; ++call) {
        const int cls = std::atoi(argv[call + 3]);
        bool timed = false;
        int way = trial.picked;
        if (!way) {
            way = blink::timed_way(trial, ways, cls);
            timed = way != 0;
            if (timed)
                ms[cls][trial.calls[cls]++] = static_cast<float>(4 - way);
            else
                way = trial.picked = blink::fastest_way(ways, ms[cls]);
        }
        std::printf("%d %d %d\n", cls, way, timed);
    }
    return 0;
}
