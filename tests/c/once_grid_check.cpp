// Prints how the kernel with a workgroup per tile cuts up a list of flows:
//   once_grid_check MOST_TILE_ELEMS GRID_SHIFT CUS  OFF LEN  OFF LEN ...
// first the tile's elements, workgroups that have something to do and, where the flows are cut into tiles of the most
// elements, their number; then one line per tile and per edge element: flow, first element, elements.
#include <cstdio>
#include <cstdlib>

#include "fold_plan.hpp"

int main(int argc, char** argv) {
    const uint32_t most = static_cast<uint32_t>(std::strtoul(argv[1], nullptr, 10));
    const uint32_t shift = static_cast<uint32_t>(std::strtoul(argv[2], nullptr, 10));
    const uint32_t cus = static_cast<uint32_t>(std::strtoul(argv[3], nullptr, 10));
    std::vector<blink::FoldFlow> flows;
    for (int i = 4; i + 1 < argc; i += 2) {
        blink::FoldFlow f{};
        f.off = std::strtoull(argv[i], nullptr, 10);
        f.len = std::strtoull(argv[i + 1], nullptr, 10);
        flows.push_back(f);
    }
    const blink::OnceGrid g = blink::once_grid(flows, most, shift, cus);
    uint32_t busy = 0, whole = 0;
    for (const blink::FoldFlow& f : flows) {
        busy += blink::fold_tiles(f.off, f.len, g.tile_elems, shift);
        whole += blink::fold_tiles(f.off, f.len, most, shift);
    }
    std::printf("%u %u %u\n", g.tile_elems, busy, whole);
    const uint32_t call = blink::once_call(g.tile_elems, shift, 3, g.tiles);
    if (blink::once_tile_elems(call) != g.tile_elems || blink::once_shift(call) != shift || blink::once_redop(call) != 3 ||
        blink::once_edges(call) != g.tiles)
        return 5;
    for (size_t f = 0; f < flows.size(); ++f) {
        const blink::OnceRange r = blink::once_range(static_cast<uint32_t>(flows[f].off), static_cast<uint32_t>(flows[f].len), shift);
        if (r.origin % 16) return 2;
        for (uint32_t x = 0; x < g.columns; ++x) {
            if (x == g.tiles) {
                for (int lane = 0; lane < 64; ++lane) {
                    const int at = blink::once_edge(r, lane);
                    if (at % 4) return 3;
                    if (at != blink::kOnceNowhere) std::printf("%zu %d 1\n", f, at / 4);
                }
                continue;
            }
            int32_t from, to;
            blink::once_tile(r, x, static_cast<int32_t>(g.tile_elems * 4), &from, &to);
            if (from >= to) continue;
            if (from % 16 || to % 16 || to - from > static_cast<int32_t>(most) * 4) return 4;
            std::printf("%zu %d %d\n", f, from / 4, (to - from) / 4);
        }
    }
    return 0;
}
