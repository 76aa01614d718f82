// Prints what the fold kernel's tables and ticket mapping make of a list of flows:
//   fold_plan_check TILE_ELEMS GRID_SHIFT EVERY_SHIFT TURN  OFF LEN  OFF LEN ...
// one line per ticket: flow (index into the arguments), first element, elements.
#include <cstdio>
#include <cstdlib>

#include "fold_plan.hpp"

int main(int argc, char** argv) {
    const uint32_t tile = static_cast<uint32_t>(std::strtoul(argv[1], nullptr, 10));
    const uint32_t shift = static_cast<uint32_t>(std::strtoul(argv[2], nullptr, 10));
    const bool every = std::atoi(argv[3]) != 0;
    const uint32_t turn = static_cast<uint32_t>(std::strtoul(argv[4], nullptr, 10));
    std::vector<blink::FoldFlow> flows;
    for (int i = 5; i + 1 < argc; i += 2) {
        blink::FoldFlow f{};
        f.off = std::strtoull(argv[i], nullptr, 10);
        f.len = std::strtoull(argv[i + 1], nullptr, 10);
        f.stores = static_cast<uint32_t>((i - 5) / 2);
        flows.push_back(f);
    }
    std::stable_sort(flows.begin(), flows.end(), [](const blink::FoldFlow& a, const blink::FoldFlow& b) { return a.len > b.len; });
    std::vector<blink::FoldLevel> levels;
    const uint64_t n = blink::fold_levels(flows, tile, shift, every, &levels);
    for (uint64_t t = 0; t < n; ++t) {
        size_t l = 0;
        while (l + 1 < levels.size() && levels[l + 1].first <= t) ++l;
        uint32_t f, k, a, b;
        int64_t org;
        blink::fold_ticket(static_cast<uint32_t>(t) - levels[l].first, levels[l].base, levels[l].tiles, levels[l].members, turn, &f, &k);
        if (f >= flows.size()) return 2;
        blink::fold_range(flows[f].off, flows[f].len, k, tile, shift, &org, &a, &b);
        std::printf("%u %lld %lld\n", flows[f].stores, static_cast<long long>(org + a), a < b ? static_cast<long long>(b - a) : 0ll);
    }
    return 0;
}
