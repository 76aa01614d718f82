// Lets the workgroups of a grid take their tickets from the fold kernel's counters in an arbitrary order:
//   fold_counters_check N_ITEMS GRID TWO SEED             one call
//   fold_counters_check calls START SEED                  many on one schedule, whose counters stand at START
// Exit status 0: every ticket was taken once, every counter was drawn from as often as the host
// counts on, every last answer lies less than the counter's workgroups past its tickets, and
// answers that make no sense (a counter that stands before or far behind its base) give no ticket.
#include <cstdio>
#include <cstdlib>
#include <random>

#include "fold_plan.hpp"

namespace {
// Calls of a schedule one after the other, each launched as fold_grid says: counters of 32 bits on the device,
// bases of 64 on the host, the number of workgroups and the size of a ticket other ones from call to call.
int calls(uint64_t start, unsigned seed) {
    std::mt19937 rng(seed);
    uint32_t counter[2] = {static_cast<uint32_t>(start), static_cast<uint32_t>(start)};
    uint64_t base[2] = {start, start};
    for (int call = 0; call < 40; ++call) {
        const uint64_t most = std::vector<uint64_t>{28, 56, 159, 160, 168, 192, 224, 256, 512}[rng() % 9];
        const uint64_t n = 1 + rng() % 3000;
        const blink::FoldGrid g = blink::fold_grid(most, n, rng() % 8 == 0, rng() % 2 ? 57344 : 131072);
        if (g.grid < 1 || g.grid > n) return 6;
        if (g.dealt) continue;   // the counters are left alone
        if (g.two && g.grid % 16) return 7;
        const uint32_t items = static_cast<uint32_t>(n), width = g.two ? g.grid / 2 : g.grid;
        std::vector<int> taken(items, 0);
        struct Workgroup { uint32_t cls, nth; };
        std::vector<Workgroup> running;
        for (uint32_t w = 0; w < g.grid; ++w) running.push_back({blink::fold_class(w, g.two), blink::fold_place(w, g.two)});
        while (!running.empty()) {
            const size_t i = rng() % running.size();
            Workgroup& wg = running[i];
            const uint32_t t = blink::fold_nth(wg.nth, wg.cls, g.two);
            if (t < items) {
                ++taken[t];
                wg.nth = counter[wg.cls]++ - static_cast<uint32_t>(base[wg.cls]) + width;
            } else {
                if (wg.nth - blink::fold_share(items, wg.cls, g.two) >= width) return 2;
                running.erase(running.begin() + static_cast<std::ptrdiff_t>(i));
            }
        }
        for (const int k : taken)
            if (k != 1) return 3;
        for (uint32_t c = 0; c < (g.two ? 2u : 1u); ++c) base[c] += blink::fold_share(items, c, g.two);
        for (int c = 0; c < 2; ++c)
            if (counter[c] != static_cast<uint32_t>(base[c])) return 4;
    }
    return 0;
}
}  // namespace

int main(int, char** argv) {
    if (argv[1][0] == 'c') return calls(std::strtoull(argv[2], nullptr, 10), static_cast<unsigned>(std::atoi(argv[3])));
    const uint32_t n = static_cast<uint32_t>(std::strtoul(argv[1], nullptr, 10));
    const uint32_t grid = static_cast<uint32_t>(std::strtoul(argv[2], nullptr, 10));
    const bool two = std::atoi(argv[3]) != 0;
    std::mt19937 rng(static_cast<unsigned>(std::atoi(argv[4])));
    const uint32_t width = two ? grid / 2 : grid;
    uint32_t counter[2] = {};
    std::vector<int> taken(n, 0);
    struct Workgroup { uint32_t cls, nth; };
    std::vector<Workgroup> running;
    for (uint32_t w = 0; w < grid; ++w) running.push_back({blink::fold_class(w, two), blink::fold_place(w, two)});
    while (!running.empty()) {
        const size_t i = rng() % running.size();
        Workgroup& g = running[i];
        const uint32_t t = blink::fold_nth(g.nth, g.cls, two);
        if (t < n) {
            ++taken[t];
            g.nth = counter[g.cls]++ + width;
        } else {
            if (g.nth - blink::fold_share(n, g.cls, two) >= width) return 2;
            running.erase(running.begin() + static_cast<std::ptrdiff_t>(i));
        }
    }
    for (const int k : taken)
        if (k != 1) return 3;
    for (uint32_t c = 0; c < (two ? 2u : 1u); ++c) {
        if (counter[c] != blink::fold_share(n, c, two)) return 4;
        for (const uint32_t off : {1u, 7u, n, 1u << 30}) {   // the counter stands this far before its base
            const uint32_t nth = width - off;
            if (off > width && (blink::fold_nth(nth, c, two) < n || nth - blink::fold_share(n, c, two) < width)) return 5;
        }
    }
    return 0;
}
