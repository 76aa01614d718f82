// What the launch rules of the fold kernel answer:
//   fold_rules_check grid MOST N_ITEMS FOR_EVERY_TILE TICKET_BYTES      -> workgroups, dealt, two counters
//   fold_rules_check policy N_LOAD N_STORE PAYLOAD KERNEL_BYTES HAS_DEPS WAY ALTERNATES   -> 0 keep, 1 stream, 2 spread
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
    if (what == "policy") {
        std::printf("%d\n", blink::fold_policy(static_cast<uint32_t>(number(2)), static_cast<uint32_t>(number(3)), number(4), number(5),
                                               number(6) != 0, static_cast<int>(number(7)), number(8) != 0));
        return 0;
    }
    return 1;
}
