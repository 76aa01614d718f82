// The fold kernel: a tile is carried along its whole tree in one pass (paper sections
// 3.3, 4.1, 4.2.2): every rank buffer is read once and written once, so the kernel is
// bound by HBM at large payloads and by the latency of one pass (arguments -> rank data
// -> stores) at small ones.  It runs the whole-tree programs, and the per-node and
// small per-edge ones, in which a wave also writes every partial sum to the buffer of
// the rank that would hold it (MID; see served_by for where that is used rather than the
// hand-over of chunks between waves).
//
// How a workgroup works, and why:
//
//   * Four waves share one tile; a wave owns U columns of 1 KiB per rank, so a
//     tile is 4 * U KiB of every rank.  U falls with the number of ranks (fold_columns): where
//     all ranks are written 44 to 80 KiB of loads per workgroup are in flight (half tiles: from 28).  More in flight than HBM
//     needs to be busy only spreads the requests out (probe, 8 ranks x 64 MiB, 208 / 224 / 256 / 320 / 448
//     workgroups 160 / 160 / 168 / 178 / 188 us): one workgroup on seven of eight CUs.
//   * The number of ranks a stage reads, and whether it writes them all, are
//     template parameters: all stages of such a schedule agree on them, so the
//     launcher picks the kernel.  Loads land in registers in the order in which the
//     stack program consumes the ranks (StageTmpl), the top accumulator is in
//     registers and the others are parked in LDS.  Nothing else is staged.
//   * What decides the rate beyond that is how tight the front is along which all workgroups
//     move: HBM serves a stretch of memory best while all its requests come at one time.  So a
//     tile's results are stored as soon as they are there, in front of the next tile's loads,
//     and the next ticket is drawn late, when the first rank's data of the present tile has
//     arrived; its answer travels while the ranks are combined and the results stored.  Measured
//     against a ticket drawn a tile ahead and loads in front of the stores (us, three sets of
//     buffers in turn): 8 ranks x 64 MiB 166.5 -> 164.4, x 256 MiB 709 -> 681, x 20 MB 56.9 -> 55.8,
//     16 ranks x 1 GiB 5600 -> 5310, 3 ranks x 98 MiB 98.8 -> 97.4, Broadcast to 7 ranks, 64 MiB,
//     72.6 -> 69.7, largest value (fp32) 8 x 64 MiB 181 -> 171.  For the same reason a workgroup
//     that takes two neighbouring tiles one after the other is 10 % slower (168 -> 185) though it
//     draws half the tickets, and loads issued one by one as registers become free, which keeps
//     more in flight, are slower as well (probe, 8 x 64 MiB: 170 against 161).
//   * Tickets come from two counters, or from one where that keeps up (see fold_grid).  A payload small enough for
//     a workgroup per tile is served by fold_once.hpp; this kernel takes it, without a counter, where that one cannot: more
//     flows, shares too unequal, a tile size or a grid that the caller asks for.
#pragma once
#include "fold_plan.hpp"
#include "kernel.hpp"

namespace blink {

constexpr int kFoldWaves = 4;
constexpr int kFoldThreads = kFoldWaves * kLanes;
// At most this many flows, and levels, travel in the kernel's arguments: a schedule
// whose flows fit needs no block on the device for small payloads.
// (Copying arguments costs the host: room for 16 flows instead of 4 made a call 0.3 us
// longer.)
constexpr int kInlineFlows = 4;
// Up to this many flows a wave keeps the tables in vector registers, lane f holding
// flow f's words and lane l level l's: they are fetched beside the arguments, not
// after them, and a ticket is resolved without touching memory.  (With scalar loads
// that depended on one another a payload of one tile per workgroup spent more than
// a microsecond before its first load.)
constexpr unsigned kLaneFlows = kLanes;

struct FoldParams {
    void* buf[BLINK_MAX_RANKS];
    const unsigned* words;           // flow words (see fold_words); null: the inline ones
    const FoldLevel* levels;         // null: the inline ones
    unsigned long long* ticket;
    unsigned long long ticket_base[2];   // the counters' values when this call starts
    unsigned n_items;                // tickets
    unsigned n_flows, n_levels;
    unsigned turn;                   // see fold_ticket
    unsigned tile_elems;             // elements per ticket
    unsigned grid_shift;             // see fold_range
    unsigned redop;                  // blink_redop_t
    unsigned reverse;                // tickets walk from the last to the first
    unsigned dealt;                  // workgroup w takes tickets w, w + width, ...; no counter is used
    unsigned two;                    // tickets come from two counters (see fold_class), else from one
    unsigned width;                  // workgroups that share a counter (of all of them where tickets are dealt)
    unsigned call;                   // number of the call on its schedule
    FoldLevel inline_levels[kInlineFlows];
    unsigned inline_words[kFlowWords * kInlineFlows];
};
static_assert(sizeof(FoldParams) <= 4096, "kernel arguments");

// Columns per wave and rank for stages that read n ranks.
//
// Where all ranks are written: the less a ticket holds, the tighter the front, as long as the counters keep
// up and a tile costs little beside its loads and stores.  us with more / the columns of drawn tickets, random
// elements, three sets of buffers in turn: 3 ranks x 98 MiB, 6 / 4, 96.4 / 95.0, 4 ranks, 4 / 3, 129 / 126.5, 6 ranks, 3 / 2,
// 180 / 178.5; 8 ranks x 114 MiB with 2 / 1 columns on 224 / 256 workgroups 284 / 291.  (On buffers of zeros one
// column is 1 to 3 % faster: figures for these tables are taken with random elements.)
// A payload of about two tiles per CU or less gets a workgroup for every half tile (4 MiB per rank, whole
// / half: 8 ranks 13.3 / 11.4, 5 ranks 8.2 / 7.6, 4 ranks 7.7 / 7.2; with three tiles per CU, 8 ranks x 6 MiB,
// 16.1 / 17.8), up to five for every whole one (6 ranks x 12 MiB, with 3 columns 19.8, with 2 22.3).
//
// Where one is written a tile is hardly more than its loads, and drawn ones are larger.  Reduce with
// fewer columns and two sub-tiles per ticket / with these: 3 ranks x 64 MiB 44 / 36, 5 ranks 60 / 55,
// 6 ranks 71 / 65, 12 ranks 149 / 123; 8 ranks 88 / 83; a workgroup for every tile, 5 ranks x 5 MiB, with 3 / 4
// columns 7.0 / 7.7.
enum class FoldTile { kHalf, kWhole, kDrawn };   // a workgroup for every tile: up to two per CU, more; drawn tickets
constexpr int fold_columns(int n, bool all, FoldTile tile) {
    if (!all && tile != FoldTile::kDrawn) return n == 2 ? 8 : n == 3 ? 6 : n == 4 ? 4 : n <= 6 ? 3 : n <= 8 ? 4 : n <= 10 ? 2 : 1;
    if (!all) return n == 2 ? 8 : n == 3 ? 6 : n == 4 ? 5 : n <= 8 ? 4 : n <= 10 ? 3 : 2;
    if (tile == FoldTile::kHalf) return n == 2 ? 4 : n == 3 ? 3 : n <= 6 ? 2 : 1;
    if (tile == FoldTile::kWhole) return n == 2 ? 8 : n == 3 ? 6 : n == 4 ? 4 : n <= 6 ? 3 : n <= 10 ? 2 : 1;
    return n == 2 ? 6 : n == 3 ? 4 : n <= 5 ? 3 : n <= 10 ? 2 : 1;
}
constexpr unsigned fold_sub_elems(int columns) { return static_cast<unsigned>(columns) * kFoldWaves * 256u; }
// Cache policies of the rank buffers' loads and stores.  Measured with the probe
// (us; 8 ranks, three sets of buffers in turn; loads always nt):
//   MiB per rank       7    16    35.5   64     114
//   stores sc1       16.2  47.4   96.5  164.7  291.9
//   stores nt sc1    22.6  48.2   94.9  162.0  289.0
//   stores nt        23.2  48.6   97.9  169.4  304.9
template <int POLICY>
struct FoldPolicyBits {
    static constexpr int kLoad = POLICY == kFoldSpread ? kPolicyDefault : kPolicyStream;
    static constexpr int kStore = POLICY == kFoldKeep ? kPolicyThrough : (kPolicyStream | kPolicyThrough);
};

template <typename T>
__device__ __forceinline__ const BLINK_CONST T* as_const(const void* p) {
    return reinterpret_cast<const BLINK_CONST T*>(reinterpret_cast<unsigned long long>(p));
}

// A sub-tile: the elements a workgroup moves at a time, [org + from, org + to) of the
// payload (none where from >= to), and its flow's stage.  All wave-uniform.
template <int N>
struct FoldPiece {
    long long org;              // a multiple of 4
    unsigned from, to;
    unsigned seq[(N + 3) / 4];  // FoldFlow::seq, four to a word
    unsigned stores;            // FoldFlow::stores
    unsigned long long mid_rank;
    __device__ __forceinline__ unsigned rank(int i) const { return (seq[i / 4] >> ((i & 3) * 8)) & 15u; }
    __device__ __forceinline__ bool push(int i) const { return (seq[i / 4] >> ((i & 3) * 8)) & 16u; }
    __device__ __forceinline__ unsigned folds(int i) const { return (seq[i / 4] >> ((i & 3) * 8 + 5)) & 7u; }
};

// Up to three elements at either end of a flow that do not fill a 16-byte column,
// one per lane.
template <typename T, int N, bool SUM, bool MID, int LD, int ST>
__device__ __forceinline__ void fold_edges(RankTable ranks, const FoldPiece<N>& pc, unsigned redop, unsigned* park, int lane) {
    const unsigned head_end = min((pc.from + 3) & ~3u, pc.to);
    const unsigned tail = max(pc.to & ~3u, head_end);
    const unsigned e = lane < 4 ? pc.from + lane : tail + (lane - 4);
    const bool mine = lane < 4 ? e < head_end : (lane < 8 && e < pc.to);
    const unsigned long long byte_off = static_cast<unsigned long long>(pc.org + pc.from) * 4ull;
    const unsigned bytes = (pc.to - pc.from) * 4u;
    const unsigned at = mine ? (e - pc.from) * 4u : 0x7ffffff0u;  // outside the window: nothing happens
    unsigned acc = 0, depth = 0;
    // All loads first: they travel together (one after the other they cost a payload of
    // 16 Ki elements on 8 ranks 1 us).  After the wait nothing of this path is outstanding.
    unsigned x[N];
#pragma unroll
    for (int i = 0; i < N; ++i)
        x[i] = __builtin_amdgcn_raw_buffer_load_b32(rank_window(ranks, pc.rank(i), byte_off, bytes), at, 0, LD);
    __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8));   // vmcnt(0)
    unsigned mids = pc.stores >> 16;
    unsigned long long mid_rank = pc.mid_rank;
    auto add = [&](unsigned x) {
        acc = combine1<T>(SUM ? static_cast<unsigned>(BLINK_SUM) : redop, acc, x);
        if constexpr (MID) {
            if (mids & 1u)
                __builtin_amdgcn_raw_buffer_store_b32(
                    acc, rank_window(ranks, static_cast<unsigned>(mid_rank) & 15u, byte_off, bytes), at, 0, kPolicyThrough);
            mids >>= 1;
            mid_rank >>= 4;
        }
    };
    acc = x[0];
#pragma unroll
    for (int i = 1; i < N; ++i) {
        if (N >= 4 && pc.push(i)) {
            park[depth++ * kLanes + lane] = acc;
            acc = x[i];
        } else {
            add(x[i]);
        }
        if (N >= 4)
#pragma unroll 1
            for (unsigned f = pc.folds(i); f; --f) add(park[--depth * kLanes + lane]);
    }
#pragma unroll 1
    for (unsigned left = pc.stores & 0xffffu; left; left &= left - 1) {
        const __amdgpu_buffer_rsrc_t win = rank_window(ranks, __builtin_ctz(left), byte_off, bytes);
        __builtin_amdgcn_raw_buffer_store_b32(acc, win, at, 0, ST);
    }
}

// T: element type (float, or unsigned for wrap-around int32).  N: ranks a stage
// reads.  ALL: it writes the same ranks, else one; stages that read one write those in
// the flow's `stores`.  SUM: the operator is the sum, else params' redop (PROD, MIN or MAX).
// U: columns per wave and rank.  MID: partial sums are written on the way (see
// FusedFlow::mid_store), through the L2 like the result that overwrites them: left in the
// L2 as modified lines they cost far more (per node, 8 x 64 MiB, us: stores by default
// policy 260, nt 216, nt sc1 211, sc1 180; 8 x 5 MiB 30.6 / 22.0 / 16.3 / 16.3).
template <typename T, int N, bool ALL, bool SUM, int POLICY, int U, bool MID>
__global__ __launch_bounds__(kFoldThreads, 2) void blink_fold(const FoldParams) {
    constexpr int LD = FoldPolicyBits<POLICY>::kLoad, ST = FoldPolicyBits<POLICY>::kStore;
    constexpr unsigned kSub = fold_sub_elems(U);
    constexpr int kStores = ALL ? N : 1;   // N == 1: those in the flow's `stores` instead
    constexpr int kParked = N < 4 ? 1 : N / 2 - 1;   // a stack program over N ranks needs at most N / 2 accumulators
    __shared__ U4 parked[N < 4 ? 1 : kParked * U * kFoldThreads];
    __shared__ unsigned drawn[2];
    __shared__ unsigned edge_parked[N < 4 ? 1 : kParked * kLanes];
    const BLINK_CONST FoldParams* p = (const BLINK_CONST FoldParams*)__builtin_amdgcn_kernarg_segment_ptr();
    const int lane = threadIdx.x & (kLanes - 1);
    const unsigned wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
    const unsigned long long mine = reinterpret_cast<unsigned long long>(p->buf[lane & (BLINK_MAX_RANKS - 1)]);
    const RankTable ranks = {static_cast<unsigned>(mine), static_cast<unsigned>(mine >> 32)};
    const unsigned n_items = p->n_items, n_flows = p->n_flows, n_levels = p->n_levels, turn = p->turn;
    const unsigned tile_elems = p->tile_elems, grid_shift = p->grid_shift, redop = p->redop, width = p->width;
    const bool reverse = p->reverse != 0, dealt = p->dealt != 0, two = p->two != 0;
    unsigned long long* const ticket = p->ticket;
    // The tables in the arguments are fetched beside the other arguments; only where they are
    // elsewhere does a wave fetch them again (measured from a kernel's start, us: arguments there 0.4,
    // tables that are fetched after them 0.7).
    unsigned flow_word[kFlowWords], level_word[4];
    auto fetch_words = [&](const BLINK_CONST unsigned* words, unsigned stride, unsigned f) {
#pragma unroll
        for (unsigned w = 0; w < kFlowWords; ++w) flow_word[w] = words[w * stride + f];
    };
    auto fetch_levels = [&](const BLINK_CONST FoldLevel* levels, unsigned l) {
        level_word[0] = levels[l].first, level_word[1] = levels[l].base;
        level_word[2] = levels[l].tiles, level_word[3] = levels[l].members;
    };
    {   // (buffer loads: others would be merged with the ones below, and wait for the arguments)
        const __amdgpu_buffer_rsrc_t args = __builtin_amdgcn_make_buffer_rsrc(
            reinterpret_cast<void*>(reinterpret_cast<unsigned long long>(p)), 0, static_cast<int>(sizeof(FoldParams)), kRawDword3);
        const int mine = lane & static_cast<int>(kInlineFlows - 1);
#pragma unroll
        for (unsigned w = 0; w < kFlowWords; ++w)
            flow_word[w] = __builtin_amdgcn_raw_buffer_load_b32(
                args, mine * 4, static_cast<int>(offsetof(FoldParams, inline_words) + w * kInlineFlows * 4), 0);
        const U4 level = __builtin_amdgcn_raw_buffer_load_b128(
            args, mine * static_cast<int>(sizeof(FoldLevel)), static_cast<int>(offsetof(FoldParams, inline_levels)), 0);
        level_word[0] = level.x, level_word[1] = level.y, level_word[2] = level.z, level_word[3] = level.w;
    }
    // all of them with one wait
    asm volatile("" ::"s"(n_items), "s"(turn), "s"(tile_elems), "s"(grid_shift), "s"(redop), "s"(width), "s"(p->reverse),
                 "s"(p->dealt), "s"(p->two), "s"(ticket), "s"(p->words), "s"(p->levels));
    const BLINK_CONST unsigned* const words = as_const<unsigned>(p->words);
    const BLINK_CONST FoldLevel* const levels = p->levels ? as_const<FoldLevel>(p->levels) : p->inline_levels;
    const bool in_lanes = n_flows <= kLaneFlows;   // and with them the levels
    if (p->words) fetch_words(words, n_flows, min(static_cast<unsigned>(lane), min(n_flows, kLaneFlows) - 1));
    if (p->levels) fetch_levels(levels, min(static_cast<unsigned>(lane), min(n_levels, kLaneFlows) - 1));

    // Ticket -> its flow and elements; then its sub-tiles one after the other.
    long long org = 0;
    unsigned lo = 0, hi = 0;   // the ticket's elements, from org
    unsigned sub = 0;          // where its next sub-tile starts, from org
    unsigned seq[(N + 3) / 4], stores = 0;
    unsigned long long mid_rank = 0;
    auto resolve = [&](unsigned t) {
        if (reverse) t = n_items - 1 - t;
        unsigned l = 0, f, tile;
        unsigned word[kFlowWords];
        if (in_lanes) {
            for (unsigned above = n_levels; above - l > 1;) {
                const unsigned mid = (l + above) / 2;
                if (__builtin_amdgcn_readlane(level_word[0], mid) <= t) l = mid; else above = mid;
            }
            fold_ticket(t - __builtin_amdgcn_readlane(level_word[0], l), __builtin_amdgcn_readlane(level_word[1], l),
                        __builtin_amdgcn_readlane(level_word[2], l), __builtin_amdgcn_readlane(level_word[3], l), turn, &f, &tile);
#pragma unroll
            for (unsigned w = 0; w < kFlowWords; ++w) word[w] = __builtin_amdgcn_readlane(flow_word[w], f);
        } else {
            for (unsigned above = n_levels; above - l > 1;) {
                const unsigned mid = (l + above) / 2;
                if (levels[mid].first <= t) l = mid; else above = mid;
            }
            fold_ticket(t - levels[l].first, levels[l].base, levels[l].tiles, levels[l].members, turn, &f, &tile);
#pragma unroll
            for (unsigned w = 0; w < kFlowWords; ++w) word[w] = words[w * n_flows + f];
        }
        auto wide = [&](unsigned w) { return (static_cast<unsigned long long>(word[w + 1]) << 32) | word[w]; };
        int64_t start;
        fold_range(wide(kFlowOff), wide(kFlowLen), tile, tile_elems, grid_shift, &start, &lo, &hi);
        org = start;
        sub = 0;
#pragma unroll
        for (int q = 0; q < (N + 3) / 4; ++q) seq[q] = word[kFlowSeq + q];
        stores = word[kFlowStores];
        mid_rank = wide(kFlowMid);
    };
    auto piece = [&]() {
        FoldPiece<N> pc;
        pc.org = org;
        pc.from = max(sub, lo);
        sub += kSub;
        pc.to = min(sub, hi);
#pragma unroll
        for (int q = 0; q < (N + 3) / 4; ++q) pc.seq[q] = seq[q];
        pc.stores = stores;
        pc.mid_rank = mid_rank;
        return pc;
    };
    U4 r[N][U];
    const unsigned column = (wave * U * kLanes + lane) * 16u;
    // whole 16-byte columns of a sub-tile: where they start in every rank, and bytes
    auto vector_bytes = [&](const FoldPiece<N>& pc, unsigned long long* byte_off) {
        const unsigned a = (pc.from + 3) & ~3u, b = pc.to & ~3u;
        *byte_off = static_cast<unsigned long long>(pc.org + a) * 4ull;
        return a < b ? (b - a) * 4u : 0u;
    };
    auto load = [&](const FoldPiece<N>& pc) {
        unsigned long long byte_off;
        const unsigned bytes = vector_bytes(pc, &byte_off);
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const __amdgpu_buffer_rsrc_t win = rank_window(ranks, pc.rank(i), byte_off, bytes);
#pragma unroll
            for (int u = 0; u < U; ++u)
                r[i][u] = __builtin_amdgcn_raw_buffer_load_b128(win, column + u * kLanes * 16, 0, LD);
        }
    };

    auto store = [&](const U4 (&v)[U], unsigned rank, unsigned long long byte_off, unsigned bytes, auto policy) {
        const __amdgpu_buffer_rsrc_t win = rank_window(ranks, rank, byte_off, bytes);
#pragma unroll
        for (int u = 0; u < U; ++u)
            __builtin_amdgcn_raw_buffer_store_b128(v[u], win, column + u * kLanes * 16, 0, policy.value);
    };
    // A new accumulator, in registers of its own: where it shares those of a load the compiler
    // waits for all memory operations, the counter's answer among them, at every loop that it enters.
    auto take = [&](U4 (&acc)[U], const U4 (&x)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            acc[u] = x[u];
            asm volatile("" : "+v"(acc[u]));
        }
    };
    constexpr std::integral_constant<int, ST> final_policy;
    constexpr std::integral_constant<int, kPolicyThrough> mid_policy;
    // Every ticket is followed by one draw: a call advances its counters by n_items (32 bits of them:
    // only differences matter).  A buffer operation whose window is empty unless there is a draw to
    // make, and holds lane 0's word alone then: issued by every wave on every path, it lets the
    // compiler count what is outstanding; behind a branch it waited for the answer wherever it
    // waited for the last loads.
    const unsigned cls = fold_class(blockIdx.x, two);
    unsigned long long* const counter = ticket + cls * kCounterStride;
    auto draw = [&]() {
        const bool due = !dealt && sub >= hi && wave == 0;
        return static_cast<unsigned>(__builtin_amdgcn_raw_ptr_buffer_atomic_add_i32(
            1, __builtin_amdgcn_make_buffer_rsrc(counter, 0, due ? 4 : 0, kRawDword3), lane * 4, 0, 0));
    };
    unsigned nth = fold_place(blockIdx.x, two);   // of the counter's tickets; the grid has at most n_items workgroups
    unsigned t = fold_nth(nth, cls, two);
    unsigned slot = 0;
    resolve(t);
    FoldPiece<N> cur = piece();
    // Where tickets are drawn the status record lies in front of the counter.  If it is set
    // (see the end) the buffers are left alone.  Asked for in front of the first tile's loads, a
    // load like them (its window is empty where tickets are dealt), so that its answer is there
    // before theirs: a wave that finds it set has nothing to do of its first ticket, and the wave
    // that hands tickets on hands on that there is none.  (Waves that find different things
    // end all the same: each reaches one barrier per ticket.)
    const unsigned state = __builtin_amdgcn_raw_buffer_load_b32(
        __builtin_amdgcn_make_buffer_rsrc(ticket - kStatusWords + kStatusState, 0, dealt ? 0 : 4, kRawDword3), 0, 0, 0);
    load(cur);
    if (__builtin_amdgcn_readfirstlane(state) != 0) {
        cur.to = cur.from;
        sub = hi;
        nth = ~0u;   // the next ticket, whatever the counter says
    }
    for (;;) {
        // the tile's loads are on their way; one wave's join them
        if (((cur.from | cur.to) & 3u) && cur.from < cur.to && wave == kFoldWaves - 1)
            fold_edges<T, N, SUM, MID, LD, ST>(ranks, cur, redop, edge_parked, lane);
        unsigned long long byte_off;
        const unsigned bytes = vector_bytes(cur, &byte_off);
        U4 acc[U];
        take(acc, r[0]);
        // the first rank's data is here: time to ask for the next ticket
        const unsigned raw = draw();
        if constexpr (N > 1) {
            unsigned depth = 0;   // accumulators parked in LDS, the oldest at the bottom
            unsigned mids = cur.stores >> 16;
            unsigned long long mid_rank = cur.mid_rank;
            auto add = [&](const U4 (&x)[U]) {
                combine_columns<T, SUM, U>(redop, acc, x);
                if constexpr (MID) {
                    if (mids & 1u) store(acc, static_cast<unsigned>(mid_rank) & 15u, byte_off, bytes, mid_policy);
                    mids >>= 1;
                    mid_rank >>= 4;
                }
            };
#pragma unroll
            for (int i = 1; i < N; ++i) {
                if (N >= 4 && cur.push(i)) {
#pragma unroll
                    for (int u = 0; u < U; ++u) parked[(depth * U + u) * kFoldThreads + threadIdx.x] = acc[u];
                    ++depth;
                    take(acc, r[i]);
                } else {
                    add(r[i]);
                }
                if (N >= 4)
#pragma unroll 1
                    for (unsigned f = cur.folds(i); f; --f) {
                        --depth;
                        U4 below[U];
#pragma unroll
                        for (int u = 0; u < U; ++u) below[u] = parked[(depth * U + u) * kFoldThreads + threadIdx.x];
                        add(below);
                    }
            }
        }
        if constexpr (N > 1) {
#pragma unroll
            for (int j = 0; j < kStores; ++j) store(acc, ALL ? j : __builtin_ctz(cur.stores), byte_off, bytes, final_policy);
        } else {
            for (unsigned left = cur.stores & 0xffffu; left; left &= left - 1)
                store(acc, __builtin_ctz(left), byte_off, bytes, final_policy);
        }
        __builtin_amdgcn_sched_barrier(0);
        // the next sub-tile: of this ticket, or of the next one
        const unsigned answer = __builtin_amdgcn_readfirstlane(raw);
        if (sub >= hi) {
            if (dealt) {
                t += width;
            } else {
                if (wave == 0) drawn[slot] = nth == ~0u ? nth : answer - static_cast<unsigned>(p->ticket_base[cls]) + width;
                __syncthreads();
                nth = __builtin_amdgcn_readfirstlane(drawn[slot]);
                t = fold_nth(nth, cls, two);
                slot ^= 1;   // the other word: a wave may still be reading this one
            }
            if (t >= n_items) break;
            resolve(t);
        }
        cur = piece();
        load(cur);
    }
    // A counter's draws end less than the width of its share of the grid past its last ticket.  If these
    // did not, the counter was not where the host counted it to be when the call started, or has been
    // moved since: another call on the schedule overlaps with this one.  Both have gone wrong
    // (tickets are lost, or drawn twice).
    if (!dealt && nth - fold_share(n_items, cls, two) >= width && threadIdx.x == 0) {
        unsigned long long* const status = ticket - kStatusWords;
        if (__hip_atomic_exchange(status + kStatusState, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0) {
            const unsigned long long base = p->ticket_base[cls];
            status[kStatusStage] = status[kStatusAwaited] = ~0ull;
            status[kStatusSeen] = base + static_cast<long long>(static_cast<int>(nth - width));
            status[kStatusWanted] = base;
            status[kStatusCall] = p->call;
        }
    }
}

using FoldFn = void (*)(const FoldParams);

#define BLINK_FOLD_CASES                                                                                            \
    BLINK_CASE(2) BLINK_CASE(3) BLINK_CASE(4) BLINK_CASE(5) BLINK_CASE(6) BLINK_CASE(7) BLINK_CASE(8) BLINK_CASE(9) \
    BLINK_CASE(10) BLINK_CASE(11) BLINK_CASE(12) BLINK_CASE(13) BLINK_CASE(14) BLINK_CASE(15) BLINK_CASE(16)

// The kernel for stages that read n ranks and write them all (drawn tickets: pick_fold_drawn, others:
// pick_fold_dealt) or one (pick_fold_one); null where there is none.
template <typename T, bool SUM, int POLICY, bool MID = false>
FoldFn pick_fold_drawn(int n) {
    switch (n) {
#define BLINK_CASE(N) case N: return blink_fold<T, N, true, SUM, POLICY, fold_columns(N, true, FoldTile::kDrawn), MID>;
        BLINK_FOLD_CASES
#undef BLINK_CASE
        default: return nullptr;
    }
}
template <typename T, bool SUM, FoldTile TILE, bool MID = false>
FoldFn pick_fold_dealt(int n) {
    switch (n) {
#define BLINK_CASE(N) case N: return blink_fold<T, N, true, SUM, kFoldKeep, fold_columns(N, true, TILE), MID>;
        BLINK_FOLD_CASES
#undef BLINK_CASE
        default: return nullptr;
    }
}
template <typename T, bool SUM, FoldTile TILE, bool MID = false>
FoldFn pick_fold_one(int n) {
    switch (n) {
#define BLINK_CASE(N) case N: return blink_fold<T, N, false, SUM, kFoldKeep, fold_columns(N, false, TILE), MID>;
        BLINK_FOLD_CASES
#undef BLINK_CASE
        default: return nullptr;
    }
}
template <typename T, bool SUM, bool MID = false>
FoldFn pick_fold(int n, bool all, FoldTile tile) {
    if (!all)
        return tile == FoldTile::kDrawn ? pick_fold_one<T, SUM, FoldTile::kDrawn, MID>(n) : pick_fold_one<T, SUM, FoldTile::kWhole, MID>(n);
    return tile == FoldTile::kHalf    ? pick_fold_dealt<T, SUM, FoldTile::kHalf, MID>(n)
           : tile == FoldTile::kWhole ? pick_fold_dealt<T, SUM, FoldTile::kWhole, MID>(n)
                                      : pick_fold_drawn<T, SUM, kFoldKeep, MID>(n);
}

// Per element type and operator class, each in a translation unit of its own so
// that they compile side by side.  all: a stage writes the ranks it reads, else one;
// stream: the kernels for sums that stream their results, where tickets are drawn; mid: those that
// write partial sums on the way.
FoldFn fold_f32_sum(int n, bool all, FoldTile tile, bool stream);
FoldFn fold_f32_other(int n, bool all, FoldTile tile);
FoldFn fold_f32_mid(int n, bool all, FoldTile tile, bool sum);
FoldFn fold_i32_sum(int n, bool all, FoldTile tile, bool stream);
FoldFn fold_i32_other(int n, bool all, FoldTile tile);
FoldFn fold_i32_mid(int n, bool all, FoldTile tile, bool sum);
FoldFn fold_copy(int policy, int columns);   // one rank read: nothing is combined

}  // namespace blink
