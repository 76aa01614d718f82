// The fold kernel for payloads that have a workgroup for every tile (fold.hpp has the larger
// ones, and says what a tile and a stack program are).
//
// Such a call is bound by the latency of one pass: arguments, rank data, stores.  What lies in
// front of the loads counts in full, and so does the length of the code, which every call
// fetches anew (1.5 to 3 KB here, 5 to 9 KB in fold.hpp).  So the place in the grid says which flow (y) and
// which of its tiles (x) a workgroup has, the arguments hold each flow's buffers in the order in
// which its stack program consumes them, and one round of scalar loads stands between a wave's
// start and its rank loads: no tickets, no levels, no loop.
//
// us per call, one after the other in a graph on three sets of buffers in turn, blink_fold / this kernel
// (sums, int32): 8 ranks x 16 KiB 2.84 / 2.2, 64 KiB and a ragged end 3.48 / 2.5, 1 MiB 3.97 / 3.2, 2 MiB
// 6.6 / 5.4, 4 MiB 10 to 11 / 9.5, 8 MiB 23 / 17.5 (shares a power of two apart; at 7.3 MiB 18.5 / 16.1),
// 4 ranks x 1 MiB 3.3 / 2.7, 4 MiB 6.75 / 6.2, 3 ranks x 3.2 MiB 4.9 / 4.0.
//
// The tiles of one flow go out one after the other, one flow after the other: in turns across the flows the
// shares of a payload of 2^n elements, a power of two apart, kept asking the same channels (8 ranks x 8
// MiB 24.9 in turns, 17.9 like this, x 2 MiB 6.4 / 5.6; sizes not a power of two within 2 %).
#pragma once
#include "fold.hpp"

namespace blink {

// At most this many flows travel in the arguments of the larger of two variants (those of the
// other hold kInlineFlows); copying them takes the host 0.04 us per 100 bytes.
constexpr int kOnceMostFlows = 16;

// Where whole tiles are handed out (the upper two fifths of the range) two workgroups at a time run on a CU, by the LDS
// they ask for: more loads in flight spread the requests out.  Against as many as fit, us: 8 ranks x 9.5 MiB 24.9 / 22.9,
// 8.8 MiB 20.8 / 19.2, 4 ranks x 16 MiB 20.3 / 18.3; half tiles there 24.1, 19.5, 17.9.
constexpr int kLdsOfFew = 56 * 1024;

// A flow as a workgroup needs it.
template <int N>
struct OnceFlow {
    OnceRange range;
    unsigned code[(N + 7) / 8];  // a nibble per rank in the order of consumption: push | folds << 1
    void* buf[N];                // the ranks' buffers in that order
};
template <int N, int F>
struct OnceParams {
    OnceFlow<N> flow[F];
    unsigned edge_column;    // the column of the grid (x) that moves what fills no 16-byte column of memory
    unsigned redop;          // blink_redop_t
    int tile_bytes;          // of a rank: at most what the workgroup's columns hold
};

// What the host passes on (see fill_once): the same, before the number of ranks is a constant.
struct OnceCall {
    const FoldFlow* flows;
    unsigned n_flows;
    unsigned grid_shift;     // see fold_range
    unsigned tiles;          // of the longest flow
    unsigned tile_elems;
    unsigned redop;
    void* const* bufs;
};

// FEW: at most two workgroups at a time on a CU.
template <typename T, int N, int F, bool SUM, int U, bool FEW>
__global__ __launch_bounds__(kFoldThreads) void blink_once(const OnceParams<N, F>) {
    constexpr int kParked = N < 4 ? 0 : N / 2 - 1;   // accumulators in LDS (see blink_fold)
    constexpr int kParkedBytes = kParked * U * kFoldThreads * 16;
    constexpr int kLdsBytes = FEW ? std::max(kParkedBytes, kLdsOfFew) : std::max(kParkedBytes, 16);
    __shared__ U4 parked[kLdsBytes / 16];
    const BLINK_CONST OnceParams<N, F>* p = (const BLINK_CONST OnceParams<N, F>*)__builtin_amdgcn_kernarg_segment_ptr();
    const BLINK_CONST OnceFlow<N>* fl = p->flow + blockIdx.y;
    if constexpr (FEW && kParked == 0) asm volatile("" ::"v"(parked));   // (otherwise nothing uses the LDS)
    const int tile_bytes = p->tile_bytes;
    const unsigned edge_column = p->edge_column, redop = SUM ? static_cast<unsigned>(BLINK_SUM) : p->redop;
    const OnceRange range = {fl->range.origin, fl->range.first, fl->range.last, fl->range.begin, fl->range.end};
    unsigned code[(N + 7) / 8];
    char* buf[N];
#pragma unroll
    for (int q = 0; q < (N + 7) / 8; ++q) code[q] = fl->code[q];
#pragma unroll
    for (int i = 0; i < N; ++i) buf[i] = static_cast<char*>(fl->buf[i]);
    // all of them with one wait
    asm volatile("" ::"s"(edge_column), "s"(tile_bytes), "s"(redop), "s"(range.origin), "s"(range.first),
                 "s"(range.last), "s"(code[0]), "s"(buf[0]), "s"(buf[N - 1]));
    auto push = [&](int i) { return (code[i / 8] >> (i % 8 * 4)) & 1u; };
    auto folds = [&](int i) { return (code[i / 8] >> (i % 8 * 4 + 1)) & 7u; };
    const int lane = threadIdx.x & (kLanes - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);

    if (blockIdx.x == edge_column) {
        // up to three elements at either end of the flow, one per lane of one wave
        if (wave != 0) return;
        const int at = once_edge(range, lane);   // (past the window: nothing happens)
        const int end = range.end;
        unsigned* const park = reinterpret_cast<unsigned*>(parked);
        unsigned x[N];
#pragma unroll
        for (int i = 0; i < N; ++i)
            x[i] = __builtin_amdgcn_raw_buffer_load_b32(__builtin_amdgcn_make_buffer_rsrc(buf[i], 0, end, kRawDword3), at, 0, kPolicyDefault);
        unsigned acc = x[0];
        int depth = 0;
#pragma unroll
        for (int i = 1; i < N; ++i) {
            if (N >= 4 && push(i)) {
                park[depth++ * kLanes + lane] = acc;
                acc = x[i];
            } else {
                acc = combine1<T>(redop, acc, x[i]);
            }
            if (N >= 4)
#pragma unroll 1
                for (unsigned f = folds(i); f; --f) acc = combine1<T>(redop, acc, park[--depth * kLanes + lane]);
        }
#pragma unroll
        for (int i = 0; i < N; ++i)
            __builtin_amdgcn_raw_buffer_store_b32(acc, __builtin_amdgcn_make_buffer_rsrc(buf[i], 0, end, kRawDword3), at, 0, kPolicyThrough);
        return;
    }

    int from, to;
    once_tile(range, blockIdx.x, tile_bytes, &from, &to);
    if (from >= to) return;   // flows need not be equally long
    const int column = from + (wave * U * kLanes + lane) * 16;   // columns past `to` fall outside the windows
    U4 r[N][U];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const __amdgpu_buffer_rsrc_t win = __builtin_amdgcn_make_buffer_rsrc(buf[i], 0, to, kRawDword3);
#pragma unroll
        for (int u = 0; u < U; ++u) r[i][u] = __builtin_amdgcn_raw_buffer_load_b128(win, column + u * kLanes * 16, 0, kPolicyStream);
    }
    asm volatile("" ::: "memory");   // all of them before anything is combined
    U4 acc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) acc[u] = r[0][u];
    int depth = 0;
#pragma unroll
    for (int i = 1; i < N; ++i) {
        if (N >= 4 && push(i)) {
#pragma unroll
            for (int u = 0; u < U; ++u) parked[(depth * U + u) * kFoldThreads + threadIdx.x] = acc[u];
            ++depth;
#pragma unroll
            for (int u = 0; u < U; ++u) acc[u] = r[i][u];
        } else {
            combine_columns<T, SUM, U>(redop, acc, r[i]);
        }
        if (N >= 4)
#pragma unroll 1
            for (unsigned f = folds(i); f; --f) {
                --depth;
                U4 below[U];
#pragma unroll
                for (int u = 0; u < U; ++u) below[u] = parked[(depth * U + u) * kFoldThreads + threadIdx.x];
                combine_columns<T, SUM, U>(redop, acc, below);
            }
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const __amdgpu_buffer_rsrc_t win = __builtin_amdgcn_make_buffer_rsrc(buf[i], 0, to, kRawDword3);
#pragma unroll
        for (int u = 0; u < U; ++u) __builtin_amdgcn_raw_buffer_store_b128(acc[u], win, column + u * kLanes * 16, 0, kPolicyThrough);
    }
}

template <int N, int F>
void fill_once(const OnceCall& c, void* to) {
    OnceParams<N, F>& p = *static_cast<OnceParams<N, F>*>(to);
    for (unsigned f = 0; f < c.n_flows; ++f) {
        const FoldFlow& fl = c.flows[f];
        OnceFlow<N>& o = p.flow[f];
        o.range = once_range(fl.off, fl.len, c.grid_shift);
        for (unsigned& q : o.code) q = 0;
        for (int i = 0; i < N; ++i) {
            o.code[i / 8] |= static_cast<unsigned>(fl.seq[i] >> 4) << (i % 8 * 4);
            o.buf[i] = c.bufs[fl.seq[i] & 15];
        }
    }
    p.edge_column = c.tiles;
    p.redop = c.redop;
    p.tile_bytes = static_cast<int>(c.tile_elems * 4);
}

// A kernel and what fills its arguments.
struct OnceKernel {
    const void* fn = nullptr;
    void (*fill)(const OnceCall&, void*) = nullptr;
};
constexpr size_t kOnceParamsBytes = sizeof(OnceParams<BLINK_MAX_RANKS, kOnceMostFlows>);
static_assert(kOnceParamsBytes <= 4096, "kernel arguments");

template <typename T, bool SUM, FoldTile TILE, int F>
OnceKernel pick_once(int n) {
    switch (n) {
#define BLINK_CASE(N)                                                                                                          \
    case N:                                                                                                                    \
        return {reinterpret_cast<const void*>(blink_once<T, N, F, SUM, fold_columns(N, true, TILE), TILE == FoldTile::kWhole>), \
                fill_once<N, F>};
        BLINK_FOLD_CASES
#undef BLINK_CASE
        default: return {};
    }
}
template <typename T, bool SUM>
OnceKernel pick_once(int n, bool half, bool many) {
    if (half) return many ? pick_once<T, SUM, FoldTile::kHalf, kOnceMostFlows>(n) : pick_once<T, SUM, FoldTile::kHalf, kInlineFlows>(n);
    return many ? pick_once<T, SUM, FoldTile::kWhole, kOnceMostFlows>(n) : pick_once<T, SUM, FoldTile::kWhole, kInlineFlows>(n);
}
// Stages that read n ranks and write them all; half: tiles of half the size; many: more than kInlineFlows flows.
OnceKernel once_f32_sum(int n, bool half, bool many);
OnceKernel once_f32_other(int n, bool half, bool many);
OnceKernel once_i32_sum(int n, bool half, bool many);
OnceKernel once_i32_other(int n, bool half, bool many);

}  // namespace blink
