// What the launch rules of the fold kernel answer:
//   fold_rules_check grid MOST N_ITEMS FOR_EVERY_TILE TICKET_BYTES      -> workgroups, dealt, two counters
//   fold_rules_check policy N_LOAD N_STORE PAYLOAD KERNEL_BYTES HAS_DEPS WAY ALTERNATES   -> 0 keep, 1 stream, 2 spread
//   fold_rules_check columns OP FUSION N CHUNK PARENT...       -> columns of a copy along one tree
//   fold_rules_check once OP FUSION N CHUNK PARENT...          -> a workgroup per tile on 256 compute units (along one tree)
//   fold_rules_check flows OP FUSION N CHUNK PARENT...         -> that kernel's flows: first element, elements, ranks written
//   fold_rules_check counters OP FUSION N CHUNK PARENT...      -> counters per stage instance in an own and a shared block, as it is
//                                                                 served and where waiting stages are asked for
//   fold_rules_check sums OP FUSION N CHUNK PARENT...          -> additions whose sum is written on the way
//   fold_rules_check shares OP N WEIGHT...                    -> the flows of four ranks in so many stars, one per weight, root 0
//   fold_rules_check call SMALL HAS_DEPS WG_PER_CU KERNEL ALTERNATES   -> a call by that kernel
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
    if (what == "call") {
        std::printf("%d\n", blink::once_call_serves(number(2) != 0, number(3) != 0, static_cast<int>(number(4)), static_cast<int>(number(5)),
                                                    number(6) != 0));
        return 0;
    }
    if (what == "shares") {
        blink::Trees trees;
        trees.k = 4;
        for (int i = 4; i < argc; ++i) {
            blink::ParentVec parent;
            parent.fill(-2);
            for (int v = 0; v < 4; ++v) parent[v] = v ? 0 : -1;
            trees.parent.push_back(parent);
            trees.root.push_back(0);
            trees.weight.push_back(std::atof(argv[i]));
        }
        blink::Schedule s;
        if (blink::make_schedule(trees, static_cast<blink_op_t>(number(2)), number(3), 1 << 16, BLINK_FUSE_TREE, s) != BLINK_OK) return 1;
        blink::FoldTables t;
        blink::fold_tables(s, &t);
        std::printf("%zu %d\n", t.once.size(), blink::once_serves(s, t.once, 256));
        return 0;
    }
    if (what == "columns" || what == "once" || what == "flows" || what == "counters" || what == "sums") {
        blink::Trees trees;
        trees.k = argc - 6;
        trees.weight.push_back(1.0);
        blink::ParentVec parent;
        parent.fill(-2);
        for (int v = 0; v < trees.k; ++v) {
            parent[v] = static_cast<int8_t>(std::atoi(argv[6 + v]));
            if (parent[v] < 0) trees.root.push_back(v);
        }
        trees.parent.push_back(parent);
        blink::Schedule s;
        if (blink::make_schedule(trees, static_cast<blink_op_t>(number(2)), number(4), number(5),
                                 static_cast<blink_fusion_t>(number(3)), s) != BLINK_OK)
            return 1;
        if (what == "columns") {
            std::printf("%d\n", blink::fold_copy_columns(s));
        } else {
            blink::FoldTables t;
            blink::fold_tables(s, &t);
            if (what == "once") std::printf("%d\n", blink::once_serves(s, t.once, 256));
            if (what == "sums")
                for (const blink::FusedFlow& f : s.fused) std::printf("%d\n", __builtin_popcount(f.mid_store));
            if (what == "counters")
                for (bool hand_over : {false, true})
                    for (bool shared : {false, true})
                        std::printf("%u\n", blink::counters_per_stage(s, blink::served_by(s, t.fits, hand_over), 256, shared));
            if (what == "flows")
                for (const blink::FoldFlow& f : t.once)
                    std::printf("%llu %llu %d\n", static_cast<unsigned long long>(f.off), static_cast<unsigned long long>(f.len),
                                __builtin_popcount(f.stores & 0xffffu));
        }
        return 0;
    }
    return 1;
}
