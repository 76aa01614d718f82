// A schedule's work as the fold kernel (fold.hpp) sees it: flows (one tree carrying one contiguous
// range, chunk boundaries mean nothing there) cut into tiles, and the order in
// which tiles are handed out.  Plain data and the one mapping that host and device
// share; no HIP in here.
#pragma once
#include <algorithm>
#include <cstdint>
#include <vector>

#include "schedule.hpp"

namespace blink {

// One flow: its range and its stage.
struct FoldFlow {
    uint64_t off, len;                // elements
    uint8_t seq[BLINK_MAX_RANKS];     // the stack program of StageTmpl: the ranks in the order in which they
                                      // are consumed, rank | push << 4 | folds << 5
    uint32_t stores;                  // bit r: the result goes to rank r; bit 16 + i: FusedFlow::mid_store
    uint64_t mid_rank;                // FusedFlow::mid_rank
};
// What the kernel reads of a flow, 32-bit words: word w of flow f lies at
// words[w * stride + f], so that one load per word fetches it for all flows.
enum : uint32_t { kFlowOff = 0, kFlowLen = 2, kFlowSeq = 4, kFlowStores = 8, kFlowMid = 9, kFlowWords = 11 };
inline void fold_words(const std::vector<FoldFlow>& flows, uint32_t stride, uint32_t* words) {
    for (size_t f = 0; f < flows.size(); ++f) {
        const FoldFlow& fl = flows[f];
        auto put = [&](uint32_t w, uint64_t v) { words[w * static_cast<size_t>(stride) + f] = static_cast<uint32_t>(v); };
        put(kFlowOff, fl.off), put(kFlowOff + 1, fl.off >> 32);
        put(kFlowLen, fl.len), put(kFlowLen + 1, fl.len >> 32);
        for (uint32_t q = 0; q < 4; ++q)
            put(kFlowSeq + q, fl.seq[4 * q] | fl.seq[4 * q + 1] << 8 | fl.seq[4 * q + 2] << 16 |
                                  static_cast<uint32_t>(fl.seq[4 * q + 3]) << 24);
        put(kFlowStores, fl.stores);
        put(kFlowMid, fl.mid_rank), put(kFlowMid + 1, fl.mid_rank >> 32);
    }
}

// Flows are kept longest first.  A level is a stretch of `tiles` tile positions at
// which the first `members` flows, and only they, still have tiles: handing out
// a level's tiles in turns over its members leaves no ticket without a tile,
// however different the trees' weights are.
struct FoldLevel {
    uint32_t first;    // ticket number of the level's first tile
    uint32_t base;     // tile position at which the level starts
    uint32_t tiles;    // tile positions
    uint32_t members;  // flows
};

constexpr uint32_t kTurnPayload = 0xffffffffu;  // a flow's tiles of a level one after another

// Ticket -> (flow, tile of the flow).  `turn`: how many neighbouring tiles of a
// flow are handed out before the next flow has its turn (section 4.2.2): 1 = tile
// by tile across the trees, a chunk's worth = chunk by chunk, kTurnPayload = one
// front through the payload.
BLINK_HOST_DEVICE inline void fold_ticket(uint32_t w, uint32_t base, uint32_t tiles, uint32_t members, uint32_t turn,
                                          uint32_t* flow, uint32_t* tile) {
    if (turn == 1) {
        *flow = w % members;
        *tile = base + w / members;
    } else if (turn >= tiles) {
        *flow = w / tiles;
        *tile = base + w % tiles;
    } else {
        const uint32_t round = members * turn;
        const uint32_t done = w / round * turn;                               // positions of earlier rounds
        const uint32_t mine = turn < tiles - done ? turn : tiles - done;      // the last round may be shorter
        const uint32_t in_round = w - done * members;
        *flow = in_round / mine;
        *tile = base + done + in_round % mine;
    }
}

// Tile `tile` of a flow: elements [*org + *a, *org + *b), none where *a >= *b.  *org is
// where the tile would start if the flow's own start did not cut it (sub-tiles are
// counted from there; it may lie up to 255 elements before the payload).  Tiles start
// where a rank buffer whose first byte is 4 * grid_shift bytes past a 1 KiB boundary
// has such a boundary (grid_shift: a multiple of 4 in [0, 256)), so *org is a multiple of 4.
BLINK_HOST_DEVICE inline void fold_range(uint64_t off, uint64_t len, uint32_t tile, uint32_t tile_elems, uint32_t grid_shift,
                                         int64_t* org, uint32_t* a, uint32_t* b) {
    const uint32_t head = static_cast<uint32_t>(off + grid_shift) & 255u;
    const uint64_t before = static_cast<uint64_t>(tile) * tile_elems;
    const int64_t left = static_cast<int64_t>(head + len - before);   // from *org to the end of the flow
    *org = static_cast<int64_t>(off - head + before);
    *a = tile == 0 ? head : 0;
    const int32_t high = static_cast<int32_t>(left >> 32);
    const uint32_t low = static_cast<uint32_t>(left);
    *b = high < 0 ? 0 : (high > 0 || low > tile_elems) ? tile_elems : low;
}

// Drawn tickets come from two counters where the grid allows (`two`; one alone sustains about 80
// draws per microsecond): the even tickets from one, the odd ones from the other.  Workgroups
// take turns in groups of eight, so that each XCD's use both.  A workgroup starts on the ticket of its
// own place and goes on with what its counter answers, counted on from the grid's share of it.
constexpr uint32_t kTwoCountersGroup = 16;   // the grid is a multiple of it
BLINK_HOST_DEVICE inline uint32_t fold_class(uint32_t workgroup, bool two) { return two ? (workgroup >> 3) & 1u : 0u; }
BLINK_HOST_DEVICE inline uint32_t fold_place(uint32_t workgroup, bool two) {
    return two ? (workgroup >> 4) * 8u + (workgroup & 7u) : workgroup;
}
// The nth ticket of a counter; beyond all tickets where nth makes no sense.
BLINK_HOST_DEVICE inline uint32_t fold_nth(uint32_t nth, uint32_t cls, bool two) {
    return two ? (nth < 0x7fffffffu ? nth : 0x7fffffffu) * 2u + cls : nth;
}
// Of n_items tickets those of a counter; each is followed by one draw.
BLINK_HOST_DEVICE inline uint32_t fold_share(uint32_t n_items, uint32_t cls, bool two) {
    return two ? (n_items + 1u - cls) / 2u : n_items;
}

// The workgroups of a call and how they get their tickets.  most: as many workgroups as the launcher wants;
// for_every_tile: a payload that is to have one for every ticket; ticket_bytes: read and written per ticket.
struct FoldGrid {
    uint32_t grid;
    bool dealt;   // workgroup w takes tickets w, w + grid, ...
    bool two;     // two counters
};
// Two counters where one does not keep up: 224 workgroups that move tickets of 56 KiB at 6.5 TB/s draw 113 times
// per microsecond, half a draw each, and a counter serves 80, so up to 158 workgroups (a part of the card) one is
// enough.  From 128 KiB per ticket one is enough for all 256, and the front along which one hands tickets out is the
// tighter (two servers of 8, 64 MiB of zeros, with one / two 324 / 328 us).  Where the mapping of workgroups to two counters
// (fold_place) does not come out even, one serves: no workgroup is given up for it.
constexpr uint64_t kFoldOneCounterBytes = 128 * 1024;
constexpr uint32_t kTwoCountersGrid = 160;
inline FoldGrid fold_grid(uint64_t most, uint64_t n_items, bool for_every_tile, uint64_t ticket_bytes) {
    FoldGrid g{static_cast<uint32_t>(std::max<uint64_t>(1, std::min(most, n_items))), false, false};
    g.dealt = for_every_tile || g.grid == n_items;
    g.two = !g.dealt && g.grid >= kTwoCountersGrid && g.grid % kTwoCountersGroup == 0 && ticket_bytes < kFoldOneCounterBytes;
    return g;
}

inline uint32_t fold_tiles(uint64_t off, uint64_t len, uint32_t tile_elems, uint32_t grid_shift) {
    return static_cast<uint32_t>((((off + grid_shift) & 255u) + len + tile_elems - 1) / tile_elems);
}

// Bytes the fold kernel reads plus writes in rank buffers per call: every rank it takes from
// once, every rank of the result once, and (sums) the sums written on the way.
inline uint64_t fold_bytes(const Schedule& s, bool sums = true) {
    uint64_t bytes = 0;
    for (const FusedFlow& f : s.fused)
        bytes += (f.hi - f.lo) * 4u * (f.stage.n_load + f.stage.n_store + (sums ? static_cast<unsigned>(__builtin_popcount(f.mid_store)) : 0u));
    return bytes;
}

// The grid of the kernel that has a workgroup for every tile and does nothing else (fold_once.hpp): a row per flow, a
// column per tile of the longest, and one more column where some flow begins or ends within a 16-byte column of memory.
struct OnceGrid {
    uint32_t tile_elems, tiles, columns;
};
// Tiles are as small as they can be without a workgroup more on any CU than tiles of `most` elements would give it (a CU
// that has one tile more than the others decides when the call ends): 3 ranks x 3.2 MiB, 270 tiles of 12 KiB, 4.45 us, 512
// of 6.3 KiB 3.97; 6 ranks x 2.1 MiB 5.46 / 4.75; 4 ranks x 4.7 MiB 7.05 / 6.45; 8 ranks x 2.4 MiB 7.28 / 6.47.  In steps of
// 256 bytes (steps of 1 KiB: 6.47 -> 7.25, steps of less split what a channel holds together).
constexpr uint32_t kOnceTileStep = 64;   // elements
constexpr size_t kOnceMostFlows = 16;
constexpr size_t kOnceParamsBytes = 656;   // room for its arguments
inline OnceGrid once_grid(const std::vector<FoldFlow>& flows, uint32_t most, uint32_t grid_shift, uint32_t cus) {
    const auto count = [&](uint32_t tile) {
        uint64_t c = 0;
        for (const FoldFlow& f : flows) c += fold_tiles(f.off, f.len, tile, grid_shift);
        return c;
    };
    const uint64_t budget = (count(most) + cus - 1) / cus * cus;
    uint32_t low = 1, high = most / kOnceTileStep;   // in steps: the smallest that keeps the budget
    while (low < high) {
        const uint32_t mid = (low + high) / 2;
        if (count(mid * kOnceTileStep) <= budget) high = mid; else low = mid + 1;
    }
    OnceGrid g{high * kOnceTileStep, 0, 0};
    bool ragged = false;
    for (const FoldFlow& f : flows) {
        g.tiles = std::max(g.tiles, fold_tiles(f.off, f.len, g.tile_elems, grid_shift));
        ragged = ragged || (f.off & 3u) || ((f.off + f.len) & 3u);
    }
    g.columns = g.tiles + (ragged ? 1u : 0u);
    return g;
}
// Up to how much traffic per CU that kernel serves a payload (10 units: 160 MiB on 256 CUs).  Its speed relative to drawn
// tickets, on three sets of buffers in turn / on so many that none is in any cache, by units:
//                             5 to 6     6 to 7     7 to 8     8 to 9     9 to 10   10 to 13   13 to 16   16 to 20   20 to 24
//   sums to all, 2 ranks     .99 / .99  .99 / .97  .99 / .95  .98 / .94  .93 / .93
//     3 ranks                .98 / .99  .98 / .96  .97 / .95  .97 / .94  .95 / .94  .89 / .93
//     4 ranks                          1.02 / .98 1.00 / .98 1.03 / .96 1.00 / .96  .92 / .93
//     6 ranks                          1.05 / .97 1.04 / .96 1.03 / .95 1.04 / .95  .91 / .93
//     8 ranks                          1.10 /1.02 1.09 /1.01 1.07 /1.00 1.06 / .99  .96 / .98
//   to one, 3 ranks                                                                1.00 / .99 1.00 / .98 1.00 / .95  .99 / .95
//     4 ranks                                                                      1.08 /1.05 1.07 /1.04 1.06 /1.05 1.05 /1.02
//     8 ranks                                                                      1.06 /1.09 1.04 /1.05 1.03 /1.02 1.01 /1.00
//     10 and 16 ranks                                                              1.03 /1.00 1.00 /1.00  .99 / .98  .96 / .96
//   copies to one, of 8                                                            1.02 /1.05 1.05 /1.05 1.09 /1.07 1.12 /1.10
//     (further on, to 30 and 40 units: of 8 1.04 /1.02 and 1.03 /1.04, of 5 1.05 /1.04 and 1.01 /1.01, of 4 1.07 /1.06 and .99 /1.01)
//     of one to 2                      1.07 /1.10 1.05 /1.09 1.04 /1.08 1.03 /1.07 1.01 / .98
//     of one to 3                      1.10 /1.10 1.10 /1.09 1.06 /1.11 1.04 /1.08 1.02 /1.02 1.01
//     of one to 7                      1.08 /1.10 1.04 /1.04  .97 /1.02  .95 / .99  .94 / .96
//     of pieces to 7                   1.12 /1.17 1.08 /1.09 1.05 /1.07 1.04 /1.08 1.01 /1.03  .98
//     of pieces to 9 and 15                                                        1.21 /1.24 1.11 /1.15 1.00 /1.03  .99 /1.00
// Sums that all ranks get, and copies of one rank, keep the line at 10: the 3 to 6 % that drawn tickets gain there in the
// steady state (two to four ranks) cost a schedule's first call its device block (30 to 60 us) and the next ones the timed choice, and a
// call on the shared block a kernel that clears it (2 us).  Repeated on one set of buffers (where drawn tickets meet what the call
// before left in the cache, and so do these), by the same units: sums to one of 8 ranks 1.15 1.09 1.03, of 4 1.16 1.10 1.07, of 16
// 1.08 up to 12; copies to one of 8 1.06 1.04 1.04 1.02, of 4 1.04 1.02 1.02 1.01, of 3 1.01 1.00 .99 .98 (so two sources
// stop at 16); pieces to 7 1.01 up to 12, to 15 1.14 up to 13 and .87 to 1.1 up to 16 (so 13).
// (sources: ranks that something is copied from.  A Gather's root is none: its own piece stays where it is.)
//
// Sums written on the way count up to 7 ranks, and in a Reduce of 4 to 8; with more ranks, and in a Reduce of 3, they do not:
// between the two lines that makes, a workgroup per tile / drawn tickets, us by MiB without the sums:
//   per edge, all ranks   8  117  22.98 / 24.15   130  23.65 / 25.97   150  27.82 / 28.63    16  121  24.76 / 26.30   141  27.31 / 29.41
//   per node              8  137  22.08 / 23.31   150  24.40 / 25.10   159  26.35 / 27.30    16  137  23.44 / 24.98   159  28.26 / 29.82
//   per edge, to one      3  140  23.57 / 24.50   155  25.89 / 26.51                         16  120  32.43 / 34.40   155  40.17 / 43.21
// 12 ranks per edge 0.995, per node 0.996, to one 1.04 and 1.02 times as fast on average; drawn tickets faster: all ranks, 3 to 6
// of them 1 to 3 %, 7 the same, to one, 4 to 8 per node 4 to 8 %, per edge -2 to 3 %.
constexpr uint64_t kOnceLineUnit = 64 * 1024;
inline uint64_t once_bytes_per_cu(uint32_t n_load, bool all, uint32_t n_store, uint32_t sources) {
    const uint64_t units = n_load > 1 && !all           ? (n_load < 4 ? 10 : n_load <= 8 ? 20 : 12)
                           : n_load == 1 && n_store == 1 ? (sources > 2 ? 24 : sources == 2 ? 16 : 10)
                           : n_load == 1 && sources > 1  ? (n_store > 8 ? 13 : 12)
                                                         : 10;
    return units * kOnceLineUnit;
}
// The most ranks that one of the flows is copied to.
inline uint32_t once_stores(const std::vector<FoldFlow>& once) {
    int most = 0;
    for (const FoldFlow& f : once) most = std::max(most, __builtin_popcount(f.stores & 0xffffu));
    return static_cast<uint32_t>(most);
}
// Whether that kernel serves a schedule on `cus` compute units; once: its flows (see once_flows).
inline bool once_serves(const Schedule& s, const std::vector<FoldFlow>& once, uint64_t cus) {
    if (once.empty()) return false;
    const StageTmpl& st = s.fused[0].stage;
    const bool copies = st.n_load == 1;
    uint32_t from = 0;
    for (const FoldFlow& f : once)
        if (f.stores & 0xffffu) from |= 1u << (f.seq[0] & 15u);
    const bool all = !copies && st.n_store == st.n_load;
    const bool sums = all ? st.n_load < 8 : st.n_load >= 4 && st.n_load <= 8;
    return fold_bytes(s, sums) <= cus * once_bytes_per_cu(st.n_load, all, copies ? once_stores(once) : st.n_store,
                                                          static_cast<uint32_t>(__builtin_popcount(from)));
}

// Whether it serves a call on a schedule that it serves.  It has one order and one policy of stores, and as many workgroups as
// tiles: a caller who asks for a grid, for a way, or for sweeps that do not alternate gets them from the other kernel.  Except
// for the way and the sweep of a few tiles per CU (small: the other kernel has a workgroup for each there too, and all of them
// fit the memory-side cache) and of programs with dependencies, which have neither.
inline bool once_call_serves(bool small, bool has_deps, int wg_per_cu, int kernel_choice, bool alternates) {
    return wg_per_cu == 0 && (small || has_deps || (kernel_choice == 0 && alternates));
}

// What a workgroup of that kernel has: byte offsets from the start of every rank buffer.
struct OnceRange {
    int32_t origin;        // where the flow's tile 0 starts on the tile grid (see fold_range): a multiple of 16
    int32_t first, last;   // the flow's whole 16-byte columns (none where first >= last)
    int32_t begin, end;    // all of it
};
BLINK_HOST_DEVICE inline OnceRange once_range(uint32_t o, uint32_t len, uint32_t grid_shift) {
    const uint32_t e = o + len;
    return {static_cast<int32_t>((o - ((o + grid_shift) & 255u)) * 4u), static_cast<int32_t>(((o + 3) & ~3u) * 4u),
            static_cast<int32_t>((e & ~3u) * 4u), static_cast<int32_t>(o * 4u), static_cast<int32_t>(e * 4u)};
}
// The columns of tile x, [*from, *to); none where *from >= *to.
BLINK_HOST_DEVICE inline void once_tile(const OnceRange& r, uint32_t x, int32_t tile_bytes, int32_t* from, int32_t* to) {
    const int32_t tile = r.origin + static_cast<int32_t>(x) * tile_bytes;
    *from = tile > r.first ? tile : r.first;
    *to = tile + tile_bytes < r.last ? tile + tile_bytes : r.last;
}
// The element outside the whole columns that lane 0 to 7 moves (up to three at either end of a flow), or an offset
// outside every window.
constexpr int32_t kOnceNowhere = 0x7ffffff0;
BLINK_HOST_DEVICE inline int32_t once_edge(const OnceRange& r, int32_t lane) {
    const int32_t head_end = r.first < r.end ? r.first : r.end, tail = r.last > head_end ? r.last : head_end;
    const int32_t e = lane < 4 ? r.begin + lane * 4 : tail + (lane - 4) * 4;
    return lane < 8 && e < (lane < 4 ? head_end : r.end) ? e : kOnceNowhere;
}
// The rest of its arguments in one word: tile (in steps), grid_shift (in columns of 16 bytes), operator, and the column
// of the grid that moves the elements outside whole columns (none: one past the grid).
BLINK_HOST_DEVICE inline uint32_t once_call(uint32_t tile_elems, uint32_t grid_shift, uint32_t redop, uint32_t edges) {
    return tile_elems / kOnceTileStep | grid_shift / 4u << 8 | redop << 14 | edges << 16;
}
BLINK_HOST_DEVICE inline uint32_t once_tile_elems(uint32_t call) { return (call & 255u) * kOnceTileStep; }
BLINK_HOST_DEVICE inline uint32_t once_shift(uint32_t call) { return (call >> 8 & 63u) * 4u; }
BLINK_HOST_DEVICE inline uint32_t once_redop(uint32_t call) { return call >> 14 & 3u; }
BLINK_HOST_DEVICE inline uint32_t once_edges(uint32_t call) { return call >> 16; }

// The flows as that kernel is given them, in payload order; none where it cannot run them: there are more than
// kOnceMostFlows, they leave something out or overlap, a byte offset (tile grid included) does not fit 31 bits, or they differ
// so much in length that workgroups without a tile (those beyond a shorter flow's end, which end at once) would outnumber the
// others.  Copies: what goes from one rank to the same others all along is one flow, whatever trees it was split among (a
// Broadcast has one, an AllGather one per piece), and a stretch that does not move (a Gather's root's own piece) is one
// without stores, unless it lies at either end of the payload: there it is left out.  (Its workgroups end at once, but where it came
// first they were in front of all others: Gather of 2 ranks, 130 to 160 MiB moved, 24.7 us, 23.0 without them, of 3 24.0 / 23.2.)
constexpr uint64_t kOnceMostElems = (1ull << 29) - 65536;
inline std::vector<FoldFlow> once_flows(std::vector<FoldFlow> flows, uint64_t n, bool copies) {
    if (flows.empty() || n >= kOnceMostElems) return {};
    std::sort(flows.begin(), flows.end(), [](const FoldFlow& a, const FoldFlow& b) { return a.off < b.off; });
    std::vector<FoldFlow> out;
    uint64_t at = copies ? flows.front().off : 0, longest = 0;
    auto put = [&](const FoldFlow& f) {
        const bool joins = copies && !out.empty() && out.back().seq[0] == f.seq[0] && out.back().stores == f.stores;
        if (joins)
            out.back().len += f.len;
        else
            out.push_back(f);
        at += f.len;
        longest = std::max(longest, out.back().len);
    };
    for (const FoldFlow& f : flows) {
        if (f.off < at || (f.off > at && !copies)) return {};
        if (f.off > at) {
            FoldFlow hole{};
            hole.off = at, hole.len = f.off - at;
            put(hole);
        }
        put(f);
    }
    if (at > n || (at < n && !copies)) return {};
    if (out.size() > kOnceMostFlows || longest * out.size() > 2 * n) return {};
    return out;
}

// The flows of a schedule, longest first.  False where the fold kernel cannot run them
// (no program is like that): flows that read different numbers of ranks, that read
// several and write neither one nor as many, or whose stack program is missing or
// deeper than the kernel's parking space (N / 2 accumulators always suffice).
inline bool fold_flows(const Schedule& s, std::vector<FoldFlow>* out) {
    out->clear();
    if (s.fused.empty()) return false;
    const uint32_t n_load = s.fused[0].stage.n_load, n_store = s.fused[0].stage.n_store;
    if (n_load > 1 && n_store != n_load && n_store != 1) return false;
    for (const FusedFlow& one : s.fused) {
        const StageTmpl& st = one.stage;
        if (st.n_load != n_load || (n_load > 1 && st.n_store != n_store) || st.seq_depth < 1 ||
            st.seq_depth > (n_load < 4 ? 1u : n_load / 2))
            return false;
        FoldFlow fl{};
        fl.off = one.lo;
        fl.len = one.hi - one.lo;
        for (uint32_t i = 0; i < n_load; ++i)   // at most n_load / 2 - 1 folds: three bits
            fl.seq[i] = static_cast<uint8_t>(st.seq_rank[i] | (st.seq_code[i] & 1) << 4 | (st.seq_code[i] >> 1) << 5);
        for (int j = 0; j < st.n_store; ++j) fl.stores |= 1u << st.store_rank[j];
        fl.stores |= static_cast<uint32_t>(one.mid_store) << 16;
        fl.mid_rank = one.mid_rank;
        out->push_back(fl);
    }
    std::stable_sort(out->begin(), out->end(), [](const FoldFlow& a, const FoldFlow& b) { return a.len > b.len; });
    return true;
}

// The levels of flows that are sorted longest first; returns the ticket count.  A flow
// has a level of its own at most: with room for that many nothing is allocated.
// every_shift: tile counts that suffice for any grid_shift (a flow may then get a
// ticket that stands for no element).
inline uint64_t fold_levels(const std::vector<FoldFlow>& flows, uint32_t tile_elems, uint32_t grid_shift, bool every_shift,
                            std::vector<FoldLevel>* out) {
    out->clear();
    uint64_t tickets = 0;
    uint32_t base = 0;
    for (size_t m = flows.size(); m > 0; --m) {
        // a flow that is no longer than the one before it may still touch one tile more:
        // that one then gets a ticket without elements
        const uint32_t count = every_shift ? static_cast<uint32_t>((flows[m - 1].len + 255 + tile_elems - 1) / tile_elems)
                                           : fold_tiles(flows[m - 1].off, flows[m - 1].len, tile_elems, grid_shift);
        if (count <= base) continue;
        out->push_back({static_cast<uint32_t>(tickets), base, count - base, static_cast<uint32_t>(m)});
        tickets += static_cast<uint64_t>(count - base) * m;
        base = count;
    }
    return tickets;
}

constexpr uint64_t kMemorySideCacheBytes = 256ull << 20;

// One rank read and copied to n_store of them: fewer columns the more stores follow each load, and
// fewer while a payload has a workgroup for every tile.  us with 2 / 3 / 4 / 8 / 16 columns:
//   Broadcast to 15, 64 MiB        148 / 158 / 164 / - / -
//   to 7, 64 MiB                    73 /  68 /  69 / 76 / -      10 MiB  17.2 / 17.6 / 17.9 / - / -
//   to 5, 85 MiB                     - /  73 /  69 / - / -       13 MiB  14.2 / 15.1 / 15.6 / - / -
//   to 3, 300 MiB                    - /   - / 207 / 193 / 207   32 MiB  18.6 / 19.2 / 20.7 / 21.9 / 25.1
//   to 2, 107 MiB                    - /   - /  57 / 50 / 54     43 MiB  17.3 / 17.4 / 17.5 / 18.8 / 19.5
//   Gather of 4 ranks, 300 MiB       - /   - /  87 / 78 / 77     80 MiB     - /    - / 18.8 / 20.0 / 19.3
// By what the call moves (fold_bytes; not by what the stages of a per-edge or per-node program would, which the kernel does
// not): to up to three ranks the line lies at 5/8 of the memory-side cache, about where payloads cease to have a workgroup for
// every tile, to four at twice the cache.  us with 4 / 8 columns by MiB moved, chains per node and whole-tree alike:
//   to 2   163  25.5 / 25.1   210  31.9 / 31.3   250  37.9 / 37.1   300  50.4 / 46.3
//   to 3   163  26.2 / 25.5   210  32.7 / 31.5   250  38.3 / 36.9   300  45.2 / 43.6
//   to 4   163  25.5 / 25.8   210  31.7 / 32.0   425  61.1 / 61.4   512  81.7 / 79.5   1200  202 / 195
//   Gather with 4 / 16 columns: of 4 ranks, 150 MiB moved, 22.9 / 23.9, of 5, 163, 34.2 / 25.7.
constexpr int kCopyColumnsSmall = 2, kCopyColumnsMost = 2, kCopyColumnsMany = 3, kCopyColumns = 4, kCopyColumnsFew = 8,
              kCopyColumnsOne = 16;
inline int fold_copy_columns(const Schedule& s) {
    const uint32_t n_store = s.fused[0].stage.n_store;
    const bool large = fold_bytes(s) > (n_store < 4 ? kMemorySideCacheBytes / 8 * 5 : 2 * kMemorySideCacheBytes);
    return n_store > 8 ? kCopyColumnsMost
           : n_store > 6 ? kCopyColumnsMany
           : n_store > 4 || !large ? kCopyColumns
           : n_store > 1 ? kCopyColumnsFew : kCopyColumnsOne;
}

enum FoldPolicy : int {
    kFoldKeep = 0,    // results may stay in the memory-side cache: whoever reads them next finds them there
    kFoldStream = 1,  // results stream past it
    kFoldSpread = 2,  // one rank read, many written: loads by default policy, stores stream
};
// How a call's results are written.  payload: bytes of all rank buffers; kernel_bytes: what the call reads and writes
// (fold_bytes).
//
// Rank buffers that together fit the memory-side cache (256 MiB) are written so that results may stay there: whoever reads
// them next (here: the next call) finds them.  Larger ones too where calls alternate their direction: a call then starts on
// the last 256 MiB that the call before it wrote (way 1, on changing buffers / repeated in place: 3 ranks x 98 MiB 95 / 83 us,
// 8 x 256 MiB 659 / 646).
// Sums that all ranks get (the other operators have kernels that keep only) stream
//   * in way 2 from twice the cache: kept / streamed, on changing buffers 6 ranks x 98 MiB 192.1 / 190.6, 8 x 64 MiB 172.3 / 170.8,
//     8 x 230 MiB 606 / 603, 5 x 150 MiB 250 / 245, 16 x 24 MiB 132 / 128; in place 177 / 188, 159 / 173, 593 / 620, 238 / 246, 115 /
//     129 (there ways 1 and 3, which keep, are to be had);
//   * in ways 1 and 3 from twelve times.  Kept / streamed, us, on three sets of buffers in turn, and repeated in place:
//       caches   7.5  8 ranks x 240 MiB     693 / 690    672 / 700      9.5  8 ranks x 304 MiB    891 / 926    852 / 900
//               10.5  8 ranks x 336 MiB     969 / 946    923 / 926     10.5  16 ranks x 168 MiB   923 / 908    900 / 890
//                8.5  4 ranks x 544 MiB     750 / 757    735 / 775     10.3  6 ranks x 440 MiB    873 / 868    861 / 883
//               12    8 ranks x 384 MiB    1056 / 1039  1032 / 1025    12    16 ranks x 192 MiB  1049 / 1008  1032 / 1024
//               12.3  8 ranks x 392 MiB    1103 / 1072  1051 / 1034    13.7  5 ranks x 700 MiB   1208 / 1190  1161 / 1166
//               14.1  4 ranks x 900 MiB    1197 / 1177  1183 / 1184    14.4  16 ranks x 230 MiB  1264 / 1204  1250 / 1224
//     (in place, what a call finds of the one before it is worth up to 7 % at 7 to 10 caches; from twelve on streaming gains
//     1 to 5 % on changing buffers and between -1 and 2 % in place.  On one card, at twelve exactly, in place 1063 / 1091
//     and 1065 / 1128.)
// A copy to one rank moves far less than the buffers hold, a gather of 8 x 400 MiB 350 MiB each way.  What it moves decides
// whether it fits the cache (gather of 8 x 80 MiB, 140 MiB moved, kept / streamed 23.6 / 27.8, 4 x 140 MiB, 210 moved, 36.4 /
// 37.9, 3 x 180 MiB, 240 moved, 41.7 / 41.6), and what it wrote is worth keeping at every size: way 1, in place, 8 x 400 MiB 108 /
// 139, 4 x 800 MiB 180 / 215, 2 ranks x 1600 MiB 477 / 499, on changing buffers 132 / 136, 212 / 211, 500 / 499.  Way 2 streams,
// from the same line as sums: on changing buffers 8 x 200 MiB 61.5 / 60.3, 4 x 400 MiB 100 / 98.
inline FoldPolicy fold_policy(uint32_t n_load, uint32_t n_store, uint64_t payload, uint64_t kernel_bytes, bool has_deps, int way,
                              bool alternates) {
    if (n_load == 1 && n_store > 1) return kFoldSpread;
    const bool copies = n_load == 1;
    if ((copies ? kernel_bytes : payload) <= kMemorySideCacheBytes) return kFoldKeep;
    if (has_deps || !alternates) return kFoldStream;
    const bool streams = way == 2 ? payload >= 2 * kMemorySideCacheBytes : !copies && payload >= 12 * kMemorySideCacheBytes;
    return streams ? kFoldStream : kFoldKeep;
}

// Which kernel serves a schedule.  Without dependencies the fold kernel: the other one
// combines a stage's ranks in the order of load_rank, which is not that of a whole tree's
// stack program, so a schedule the fold kernel cannot run is not run at all.  With
// dependencies the fold kernel carries a tile through all its transfers in one wave and writes
// each of them to its rank buffer; the alternative is to hand chunks over from wave to wave,
// through counters and memory.  Measured on 8 ranks, fp32 sums, three sets of buffers in turn,
// us, handed over (the best of 16 KiB to 4 MiB chunks) / in one wave:
//   MiB per rank      8           16          32           64          128         256
//   per-node      57 / 26     87 / 50    168 / 92    316 / 180   599 / 355   1161 / 714
//   per-edge      60 / 29     99 / 54    179 / 101   333 / 196   635 / 384   1243 / 769
// One wave is about twice as fast at every size.  Per-edge payloads larger than the memory-side
// cache are handed over all the same, not for speed: they are the paper's pipeline of chunks,
// and its pace is what callers who tune the chunk size (section 4.2.1, blink_miad_*) measure
// there; blink_schedule_set_hand_over gives them the same on smaller ones.
// hand_over: waiting stages are asked for.
enum class Served { kFold, kHandOver, kNot };
inline Served served_by(const Schedule& s, bool fold_fits, bool hand_over) {
    if (!s.has_deps) return fold_fits ? Served::kFold : Served::kNot;
    if (hand_over || !fold_fits) return Served::kHandOver;
    const bool in_cache = static_cast<uint64_t>(s.k) * s.n * 4 <= kMemorySideCacheBytes;
    return s.fusion == BLINK_FUSE_NODE || in_cache ? Served::kFold : Served::kHandOver;
}

// Counters of finished tiles per stage instance in a block: pieces' only where chunks are handed over, the other kernels count no
// tiles.  The static block's pieces leave half of it for the tables; a schedule's own has room for more counters.
constexpr size_t kStaticBlockBytes = 4u << 20, kMostCounterBytes = 32u << 20;
inline uint32_t counters_per_stage(const Schedule& s, Served served, uint64_t counter_bytes, bool static_block) {
    return served == Served::kHandOver ? hand_over_pieces(s, counter_bytes, static_block ? kStaticBlockBytes / 2 : kMostCounterBytes) : 1u;
}

// Tile sizes a caller may ask for: powers of two.
constexpr uint32_t kLeastTileOverride = 256, kMostTileOverride = 65536;
// Sets of levels that lie on the device where a schedule's tables do: one per such tile
// size (from the smallest up) and, last, that of the tile the launcher chooses.  With all of
// them there a new tile size needs no new tables, so a call can be recorded after it.
constexpr uint32_t kLevelSets = 10;
inline uint32_t level_set(uint32_t tile_override) {
    uint32_t set = 0;
    if (tile_override == 0) return kLevelSets - 1;
    while ((kLeastTileOverride << set) < tile_override) ++set;
    return set;
}
static_assert((kLeastTileOverride << (kLevelSets - 2)) == kMostTileOverride, "a set of levels per tile size");

// What the fold kernel needs of a schedule, worked out with it: calls allocate nothing.
struct FoldTables {
    bool fits = false;               // the kernel can run the schedule
    std::vector<FoldFlow> flows;
    std::vector<FoldFlow> once;      // see once_flows
    std::vector<FoldLevel> levels;   // room for one per flow; filled by the launch plan
    // Tables on the device, copied as they are: fold_words with the number of flows as stride,
    // then the sets of levels, room for one level per flow in each.
    std::vector<uint32_t> tables;
    static constexpr size_t words_per_flow() { return kFlowWords + kLevelSets * sizeof(FoldLevel) / sizeof(uint32_t); }
    size_t level_word(uint32_t set) const {   // where a set starts
        return (kFlowWords + set * sizeof(FoldLevel) / sizeof(uint32_t)) * flows.size();
    }
    // Tile counts of the sets suffice for any distance of the buffers from a 1 KiB boundary.
    void fill_set(uint32_t set, uint32_t tile_elems) {
        fold_levels(flows, tile_elems, 0, true, &levels);
        uint32_t* to = tables.data() + level_word(set);
        for (const FoldLevel& l : levels) *to++ = l.first, *to++ = l.base, *to++ = l.tiles, *to++ = l.members;
    }
};
inline void fold_tables(const Schedule& s, FoldTables* out) {
    out->fits = fold_flows(s, &out->flows);
    if (!out->fits) out->flows.clear();
    out->once = once_flows(out->flows, s.n, s.fused.empty() || s.fused[0].stage.n_load == 1);
    out->levels.reserve(out->flows.size());
    out->tables.assign(FoldTables::words_per_flow() * out->flows.size(), 0);
    fold_words(out->flows, static_cast<uint32_t>(out->flows.size()), out->tables.data());
    for (uint32_t set = 0; set + 1 < kLevelSets; ++set) out->fill_set(set, kLeastTileOverride << set);
}

}  // namespace blink
