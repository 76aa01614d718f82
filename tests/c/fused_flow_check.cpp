// Prints what the one-pass kernel is to do with each flow of a schedule:
//   fused_flow_check OP FUSION N CHUNK K TREES  ROOT WEIGHT PARENT*K ...
// one line per flow: first element, end, final stores, then per rank consumed
// rank:push:folds, then per addition rank:written.
#include <cstdio>
#include <cstdlib>

#include "schedule.hpp"

int main(int argc, char** argv) {
    int at = 1;
    auto next = [&] { return at < argc ? argv[at++] : const_cast<char*>("0"); };
    const auto op = static_cast<blink_op_t>(std::atoi(next()));
    const auto fusion = static_cast<blink_fusion_t>(std::atoi(next()));
    const uint64_t n = std::strtoull(next(), nullptr, 10), chunk = std::strtoull(next(), nullptr, 10);
    blink::Trees trees;
    trees.k = std::atoi(next());
    const int count = std::atoi(next());
    for (int t = 0; t < count; ++t) {
        trees.root.push_back(std::atoi(next()));
        trees.weight.push_back(std::atof(next()));
        blink::ParentVec parent;
        parent.fill(-2);
        for (int v = 0; v < trees.k; ++v) parent[v] = static_cast<int8_t>(std::atoi(next()));
        trees.parent.push_back(parent);
    }
    blink::Schedule s;
    if (blink::make_schedule(trees, op, n, chunk, fusion, s) != BLINK_OK) return 1;
    for (const blink::FusedFlow& f : s.fused) {
        std::printf("%llu %llu ", static_cast<unsigned long long>(f.lo), static_cast<unsigned long long>(f.hi));
        for (int j = 0; j < f.stage.n_store; ++j) std::printf("%s%d", j ? "," : "", f.stage.store_rank[j]);
        std::printf(" ");
        for (int i = 0; i < f.stage.n_load; ++i)
            std::printf("%s%d:%d:%d", i ? "," : "", f.stage.seq_rank[i], f.stage.seq_code[i] & 1, f.stage.seq_code[i] >> 1);
        std::printf(" ");
        for (int i = 0; i + 1 < f.stage.n_load; ++i)
            std::printf("%s%d:%d", i ? "," : "", static_cast<int>(f.mid_rank >> (4 * i)) & 15, f.mid_store >> i & 1);
        std::printf("\n");
    }
    return 0;
}
