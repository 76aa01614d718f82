// Lets the workgroups of a grid take their tickets from the fold kernel's counters in an arbitrary order:
//   fold_counters_check N_ITEMS GRID TWO SEED
// Exit status 0: every ticket was taken once, every counter was drawn from as often as the host
// counts on, every last answer lies less than the counter's workgroups past its tickets, and
// answers that make no sense (a counter that stands before or far behind its base) give no ticket.
#include <cstdio>
#include <cstdlib>
#include <random>

#include "fold_plan.hpp"

int main(int, char** argv) {
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
