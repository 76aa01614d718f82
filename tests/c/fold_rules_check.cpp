// What the launch rules of the fold kernel answer:
//   fold_rules_check grid MOST N_ITEMS FOR_EVERY_TILE TICKET_BYTES      -> workgroups, dealt, two counters
#include <cstdio>
#include <cstdlib>
#include <string>

#include "fold_plan.hpp"

int main(int argc, char** argv) {
    auto number = [&](int i) { return i < argc ? std::strtoull(argv[i], nullptr, 10) : 0ull; };
    const std::string what = argv[1];
    if (what == "grid") {
        const blink::FoldGrid g = blink::fold_grid(number(2), number(3), number(4) != 0, number(5));
        std::printf("%u %d %d\n", g.grid, g.dealt, g.two);
        return 0;
    }
    return 1;
}
