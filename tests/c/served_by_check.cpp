// Which kernel serves a schedule, for schedules put together by hand: one line each.
#include <cstdio>

#include "fold_plan.hpp"

namespace {
blink::Schedule schedule(int k, uint64_t n, blink_fusion_t fusion, bool has_deps, int n_load_first, int n_load_second) {
    blink::Schedule s;
    s.k = k;
    s.n = n;
    s.fusion = fusion;
    s.has_deps = has_deps;
    uint64_t at = 0;
    for (int n_load : {n_load_first, n_load_second}) {
        blink::FusedFlow f{};
        f.lo = at;
        f.hi = at += n / 2;
        f.stage.n_load = static_cast<uint8_t>(n_load);
        f.stage.n_store = static_cast<uint8_t>(n_load);
        f.stage.seq_depth = 1;
        s.fused.push_back(f);
    }
    return s;
}
void show(const char* what, const blink::Schedule& s, bool hand_over) {
    blink::FoldTables t;
    blink::fold_tables(s, &t);
    const blink::Served served = blink::served_by(s, t.fits, hand_over);
    std::printf("%s: %s\n", what, served == blink::Served::kFold ? "fold" : served == blink::Served::kHandOver ? "hand over" : "not");
}
}  // namespace

int main() {
    using blink::kMemorySideCacheBytes;
    const uint64_t fits = kMemorySideCacheBytes / 4 / 4;   // elements on 4 ranks that fill the cache
    show("tree", schedule(4, 8 * fits, BLINK_FUSE_TREE, false, 4, 4), false);
    show("tree, asked to wait", schedule(4, 8 * fits, BLINK_FUSE_TREE, false, 4, 4), true);
    show("tree, unlike stages", schedule(4, 1024, BLINK_FUSE_TREE, false, 4, 3), false);
    show("node", schedule(4, 8 * fits, BLINK_FUSE_NODE, true, 4, 4), false);
    show("node, asked to wait", schedule(4, 1024, BLINK_FUSE_NODE, true, 4, 4), true);
    show("node, unlike stages", schedule(4, 1024, BLINK_FUSE_NODE, true, 4, 3), false);
    show("edge, fills the cache", schedule(4, fits, BLINK_FUSE_EDGE, true, 4, 4), false);
    show("edge, asked to wait", schedule(4, fits, BLINK_FUSE_EDGE, true, 4, 4), true);
    show("edge, larger", schedule(4, fits + 1, BLINK_FUSE_EDGE, true, 4, 4), false);
    show("edge without dependencies", schedule(4, 8 * fits, BLINK_FUSE_EDGE, false, 1, 1), false);
    return 0;
}
