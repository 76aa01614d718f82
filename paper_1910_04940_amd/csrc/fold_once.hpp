// The fold kernel for payloads that have a workgroup for every tile (fold.hpp has the larger
// ones, and says what a tile and a stack program are).
//
// Such a call is bound by the latency of one pass: arguments, rank data, stores.  What lies in
// front of the loads counts in full, and so does the length of the code, which every call
// fetches anew (sums of 4 ranks 1.9 KB, of 8 3.4, against 6.8 and 8.7 in fold.hpp).  So the place in the grid says which flow (y) and
// which of its tiles (x) a workgroup has, two rounds of scalar loads, the second from
// lines that the first has fetched, stand between a wave's start and its rank loads: no tickets, no levels, no loop.
//
// us per call, one after the other in a graph on three sets of buffers in turn, blink_fold / this kernel
// (sums, int32): 8 ranks x 16 KiB 2.84 / 2.28, 64 KiB and a ragged end 3.45 / 2.36, 0.4 MiB 3.8 / 2.7, 1 MiB 3.97 / 3.56,
// 1.5 MiB 6.1 / 4.4, 4 MiB 11.1 / 9.7, 8 MiB 23 / 17.5 (shares a power of two apart; at 6.1 MiB 16.3 / 13.5),
// 4 ranks x 0.8 MiB 3.3 / 2.6, 4 MiB 6.75 / 5.5, 16 ranks x 0.8 MiB 6.5 / 5.6; 3 ranks x 3.2 MiB 4.9 / 4.0.
//
// The tiles of one flow go out one after the other, one flow after the other: in turns across the flows the
// shares of a payload of 2^n elements, a power of two apart, kept asking the same channels (8 ranks x 8
// MiB 24.9 in turns, 17.9 like this, x 2 MiB 6.4 / 5.6; sizes not a power of two within 2 %).
#pragma once
#include "fold.hpp"

namespace blink {

// Where whole tiles are handed out (from 96 MiB of traffic on 256 CUs) two workgroups at a time run on a CU, by the LDS
// they ask for: more loads in flight spread the requests out.  Against as many as fit, us: 8 ranks x 9.5 MiB 24.9 / 22.9,
// 8.8 MiB 20.8 / 19.2, 4 ranks x 16 MiB 20.3 / 18.3; half tiles there 24.1, 19.5, 17.9.
constexpr int kLdsOfFew = 56 * 1024;

// The arguments are short: a launch with at most 112 bytes of them takes the host less time (C call on one host, 3 to 7
// ranks 3.0 us, 8 ranks with 120 bytes 3.7, with 370 or more 3.8 to 4; on another host 2.24 up to 112 bytes, 2.30 beyond).
// So a buffer's address is one more scalar load away, from a line that is there by then, a flow's program is packed as tightly as
// that takes for 8 ranks, and there are two variants, for few flows and for many (kOnceMostFlows).  With sums written on the way
// the few flows take 112 bytes up to 6 ranks, 120 for 7 and 128 for 8.
constexpr int kOnceFewFlows = 4;
// Flow f's program: the ranks in the order of consumption, and for each push | folds << 1.  Up to 4 ranks: word f, four
// bits per rank, the codes from bit 16 on.  Up to 8: word f, three bits per rank, the low byte of the codes from bit 24
// on; the other two, three bits per code, are a half of word F + f / 2.  More: words 4 f and 4 f + 1, four bits per rank, and
// the codes in the next two.  Where one rank is written it stands in the place of the first code, which says nothing.
constexpr int once_words(int n, int flows) { return n <= 4 ? flows : n <= 8 ? flows + (flows + 1) / 2 : 4 * flows; }
// Where partial sums are written on the way (FusedFlow::mid_store and mid_rank), flow f's: up to 8 ranks in word f, which additions' in
// the low byte, then three bits per addition for the rank; more ranks in words 3 f (which) and 3 f + 1, 3 f + 2 (four bits).
constexpr int once_mid_words(int n, int flows, bool mid) { return !mid ? 0 : n <= 8 ? flows : 3 * flows; }
template <int N, int F, bool MID>
struct OnceParams {
    void* buf[N];
    unsigned begin[F + 1];    // flow f: elements [begin[f], begin[f + 1])
    unsigned word[once_words(N, F) + once_mid_words(N, F, MID)];
    unsigned call;            // see once_call
};
static_assert(sizeof(OnceParams<8, kOnceFewFlows, false>) <= 112 && sizeof(OnceParams<6, kOnceFewFlows, true>) <= 112, "see above");

// ALL: the ranks read are written, else one.  SUM, U, MID: see blink_fold.  FEW: at most two workgroups at a time on a CU.
template <typename T, int N, int F, bool ALL, bool SUM, bool MID, int U, bool FEW>
__global__ __launch_bounds__(kFoldThreads) void blink_once(const OnceParams<N, F, MID>) {
    constexpr int kParked = N < 4 ? 0 : N / 2 - 1;   // accumulators in LDS (see blink_fold)
    constexpr int kParkedBytes = kParked * U * kFoldThreads * 16;
    constexpr int kLdsBytes = FEW ? std::max(kParkedBytes, kLdsOfFew) : std::max(kParkedBytes, 16);
    __shared__ U4 parked[kLdsBytes / 16];
    const BLINK_CONST OnceParams<N, F, MID>* p = (const BLINK_CONST OnceParams<N, F, MID>*)__builtin_amdgcn_kernarg_segment_ptr();
    const unsigned f = blockIdx.y, call = p->call;
    if constexpr (FEW && kParked == 0) asm volatile("" ::"v"(parked));   // (otherwise nothing uses the LDS)
    unsigned order[(N + 7) / 8], codes[(N + 7) / 8];
    if constexpr (N <= 4) {
        order[0] = p->word[f];
    } else if constexpr (N <= 8) {
        order[0] = p->word[f], codes[0] = p->word[F + f / 2];
    } else {
        order[0] = p->word[4 * f], order[1] = p->word[4 * f + 1], codes[0] = p->word[4 * f + 2], codes[1] = p->word[4 * f + 3];
    }
    const unsigned begin = p->begin[f], end = p->begin[f + 1];
    unsigned which = 0;                // additions whose sum is written on the way, the next one's in bit 0
    unsigned long long sums = 0;       // their ranks, likewise
    if constexpr (MID) {
        const BLINK_CONST unsigned* mid = p->word + once_words(N, F);
        if constexpr (N <= 8) {
            which = mid[f] & 255u, sums = mid[f] >> 8;
        } else {
            which = mid[3 * f], sums = static_cast<unsigned long long>(mid[3 * f + 2]) << 32 | mid[3 * f + 1];
        }
    }
    constexpr int kSumBits = N <= 8 ? 3 : 4;
    asm volatile("" ::"s"(begin), "s"(end), "s"(order[0]), "s"(call), "s"(p->buf[0]), "s"(p->buf[N - 1]), "s"(which));   // all of them with one wait
    constexpr int kBits = N > 4 && N <= 8 ? 3 : 4;
    if constexpr (N <= 4) codes[0] = order[0] >> 16;
    else if constexpr (N <= 8) codes[0] = order[0] >> 24 | (codes[0] >> (f & 1) * 16 & 0xffffu) << 8;
    auto rank = [&](int i) { return order[i / 8] >> (i % 8 * kBits) & ((1u << kBits) - 1); };
    auto push = [&](int i) { return codes[i / 8] >> (i % 8 * kBits) & 1u; };
    auto folds = [&](int i) { return codes[i / 8] >> (i % 8 * kBits + 1) & ((1u << (kBits - 1)) - 1); };
    char* buf[N];
#pragma unroll
    for (int i = 0; i < N; ++i) buf[i] = static_cast<char*>(p->buf[rank(i)]);
    const unsigned redop = SUM ? static_cast<unsigned>(BLINK_SUM) : once_redop(call);
    const OnceRange range = once_range(begin, end - begin, once_shift(call));
    const int lane = threadIdx.x & (kLanes - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
    RankTable ranks{};
    if constexpr (MID) {   // lane r: rank r's buffer
        const unsigned long long mine = reinterpret_cast<unsigned long long>(p->buf[lane < N ? lane : 0]);
        ranks = {static_cast<unsigned>(mine), static_cast<unsigned>(mine >> 32)};
    }
    const int one = static_cast<int>(codes[0] & ((1u << kBits) - 1));   // the rank written where that is one
    auto destination = [&](int j, int limit) {
        return __builtin_amdgcn_make_buffer_rsrc(ALL ? buf[j] : static_cast<char*>(p->buf[one]), 0, limit, kRawDword3);
    };
    constexpr int kStores = ALL ? N : 1;

    if (blockIdx.x == once_edges(call)) {
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
        auto add = [&](unsigned x) {
            acc = combine1<T>(redop, acc, x);
            if constexpr (MID) {
                if (which & 1u)
                    __builtin_amdgcn_raw_buffer_store_b32(acc, rank_window(ranks, sums & ((1u << kSumBits) - 1), 0, end), at, 0, kPolicyThrough);
                which >>= 1, sums >>= kSumBits;
            }
        };
#pragma unroll
        for (int i = 1; i < N; ++i) {
            if (N >= 4 && push(i)) {
                park[depth++ * kLanes + lane] = acc;
                acc = x[i];
            } else {
                add(x[i]);
            }
            if (N >= 4)
#pragma unroll 1
                for (unsigned f = folds(i); f; --f) add(park[--depth * kLanes + lane]);
        }
#pragma unroll
        for (int j = 0; j < kStores; ++j) __builtin_amdgcn_raw_buffer_store_b32(acc, destination(j, end), at, 0, kPolicyThrough);
        return;
    }

    int from, to;
    once_tile(range, blockIdx.x, static_cast<int>(once_tile_elems(call) * 4), &from, &to);
    if (from >= to) return;   // flows need not be equally long
    const int column = from + (wave * U * kLanes + lane) * 16;   // columns past `to` fall outside the windows
    U4 r[N][U];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const __amdgpu_buffer_rsrc_t win = __builtin_amdgcn_make_buffer_rsrc(buf[i], 0, to, kRawDword3);
#pragma unroll
        for (int u = 0; u < U; ++u) r[i][u] = __builtin_amdgcn_raw_buffer_load_b128(win, column + u * kLanes * 16, 0, kPolicyStream);
    }
    asm volatile("" ::: "memory");   // all of them, in this order, before anything is combined
    if constexpr (MID) __builtin_amdgcn_sched_barrier(0);
    // Where sums are written on the way a new accumulator has registers of its own: if it shares those of a load the
    // compiler waits for all memory operations, those stores among them, at every loop that it enters (per node, 16
    // ranks x 0.9 MiB 9.5 us, 8.3 so).
    auto take = [&](U4 (&acc)[U], const U4 (&x)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            acc[u] = x[u];
            if constexpr (MID) asm volatile("" : "+v"(acc[u]));
        }
    };
    U4 acc[U];
    take(acc, r[0]);
    int depth = 0;
    auto add = [&](const U4 (&x)[U]) {
        combine_columns<T, SUM, U>(redop, acc, x);
        if constexpr (MID) {
            if (which & 1u) {
                const __amdgpu_buffer_rsrc_t win = rank_window(ranks, sums & ((1u << kSumBits) - 1), 0, to);
#pragma unroll
                for (int u = 0; u < U; ++u) __builtin_amdgcn_raw_buffer_store_b128(acc[u], win, column + u * kLanes * 16, 0, kPolicyThrough);
            }
            which >>= 1, sums >>= kSumBits;
        }
    };
#pragma unroll
    for (int i = 1; i < N; ++i) {
        if (N >= 4 && push(i)) {
#pragma unroll
            for (int u = 0; u < U; ++u) parked[(depth * U + u) * kFoldThreads + threadIdx.x] = acc[u];
            ++depth;
            take(acc, r[i]);
        } else {
            add(r[i]);
        }
        if (N >= 4)
#pragma unroll 1
            for (unsigned f = folds(i); f; --f) {
                --depth;
                U4 below[U];
#pragma unroll
                for (int u = 0; u < U; ++u) below[u] = parked[(depth * U + u) * kFoldThreads + threadIdx.x];
                add(below);
            }
    }
#pragma unroll
    for (int j = 0; j < kStores; ++j) {
        const __amdgpu_buffer_rsrc_t win = destination(j, to);
#pragma unroll
        for (int u = 0; u < U; ++u) __builtin_amdgcn_raw_buffer_store_b128(acc[u], win, column + u * kLanes * 16, 0, kPolicyThrough);
    }
}

// What of the arguments is the same for all calls on a schedule: all but the buffers and `call`.
template <int N, int F, bool MID>
void fill_once(const std::vector<FoldFlow>& flows, void* to) {
    OnceParams<N, F, MID>& p = *static_cast<OnceParams<N, F, MID>*>(to);
    constexpr int kBits = N > 4 && N <= 8 ? 3 : 4;
    for (unsigned& w : p.word) w = 0;
    for (size_t f = 0; f < flows.size(); ++f) {
        const FoldFlow& fl = flows[f];
        p.begin[f] = static_cast<unsigned>(fl.off);
        uint64_t order = 0, codes = 0;
        for (int i = 0; i < N; ++i) {
            order |= static_cast<uint64_t>(fl.seq[i] & 15u) << (i * kBits);
            codes |= static_cast<uint64_t>(fl.seq[i] >> 4) << (i * kBits);
        }
        const uint32_t stores = fl.stores & 0xffffu;
        if (!(stores & (stores - 1))) codes = (codes & ~static_cast<uint64_t>((1u << kBits) - 1)) | static_cast<unsigned>(__builtin_ctz(stores));
        if (MID) {
            unsigned* const mid = p.word + once_words(N, F);
            if (N <= 8) {
                mid[f] = fl.stores >> 16;
                for (int i = 0; i < N - 1; ++i) mid[f] |= static_cast<unsigned>(fl.mid_rank >> 4 * i & 7u) << (8 + 3 * i);
            } else {
                mid[3 * f] = fl.stores >> 16, mid[3 * f + 1] = static_cast<unsigned>(fl.mid_rank), mid[3 * f + 2] = static_cast<unsigned>(fl.mid_rank >> 32);
            }
        }
        if (N <= 4) {
            p.word[f] = static_cast<unsigned>(order | codes << 16);
        } else if (N <= 8) {
            p.word[f] = static_cast<unsigned>(order | codes << 24);
            p.word[F + f / 2] |= static_cast<unsigned>(codes >> 8 << (f & 1) * 16);
        } else {
            for (int q = 0; q < 2; ++q) {
                p.word[4 * f + q] = static_cast<unsigned>(order >> 32 * q);
                p.word[4 * f + 2 + q] = static_cast<unsigned>(codes >> 32 * q);
            }
        }
    }
    p.begin[flows.size()] = static_cast<unsigned>(flows.back().off + flows.back().len);
}

// The same where one rank is read and copied to others, up to M of them; K: ranks whose buffers are in the arguments.
// Flow f's program: four bits per rank, the source and then M destinations, the source again in the place of those it
// does not have.
template <int K, int F>
struct OnceCopyParams {
    void* buf[K];
    unsigned begin[F + 1];
    unsigned word[F * K / 8];
    unsigned call;
};
static_assert(sizeof(OnceCopyParams<8, kOnceFewFlows>) <= 112, "see OnceParams");

template <int K, int M, int F, int U>
__global__ __launch_bounds__(kFoldThreads) void blink_once_copy(const OnceCopyParams<K, F>) {
    // one load and M stores per column: what was read stays in the caches for its next reader, what is written streams;
    // a copy to one rank like a sum (see FoldPolicyBits)
    constexpr int kPolicy = M == 1 ? kFoldKeep : kFoldSpread;
    constexpr int LD = FoldPolicyBits<kPolicy>::kLoad, ST = FoldPolicyBits<kPolicy>::kStore;
    const BLINK_CONST OnceCopyParams<K, F>* p = (const BLINK_CONST OnceCopyParams<K, F>*)__builtin_amdgcn_kernarg_segment_ptr();
    const unsigned f = blockIdx.y, call = p->call;
    unsigned ranks[K / 8];
#pragma unroll
    for (int q = 0; q < K / 8; ++q) ranks[q] = p->word[f * (K / 8) + q];
    const unsigned begin = p->begin[f], end = p->begin[f + 1];
    asm volatile("" ::"s"(begin), "s"(end), "s"(ranks[0]), "s"(call), "s"(p->buf[0]), "s"(p->buf[K - 1]));   // all of them with one wait
    auto rank = [&](int i) { return ranks[i / 8] >> (i % 8 * 4) & 15u; };
    char* buf[M + 1];
#pragma unroll
    for (int i = 0; i <= M; ++i) buf[i] = static_cast<char*>(p->buf[rank(i)]);
    if (rank(1) == rank(0)) return;   // nothing of this flow moves
    const OnceRange range = once_range(begin, end - begin, once_shift(call));
    const int lane = threadIdx.x & (kLanes - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
    if (blockIdx.x == once_edges(call)) {
        if (wave != 0) return;
        const int at = once_edge(range, lane);
        const unsigned x = __builtin_amdgcn_raw_buffer_load_b32(__builtin_amdgcn_make_buffer_rsrc(buf[0], 0, range.end, kRawDword3), at, 0, LD);
#pragma unroll
        for (int i = 1; i <= M; ++i)
            if (i == 1 || rank(i) != rank(0))
                __builtin_amdgcn_raw_buffer_store_b32(x, __builtin_amdgcn_make_buffer_rsrc(buf[i], 0, range.end, kRawDword3), at, 0, ST);
        return;
    }
    int from, to;
    once_tile(range, blockIdx.x, static_cast<int>(once_tile_elems(call) * 4), &from, &to);
    if (from >= to) return;
    const int column = from + (wave * U * kLanes + lane) * 16;
    U4 r[U];
    const __amdgpu_buffer_rsrc_t source = __builtin_amdgcn_make_buffer_rsrc(buf[0], 0, to, kRawDword3);
#pragma unroll
    for (int u = 0; u < U; ++u) r[u] = __builtin_amdgcn_raw_buffer_load_b128(source, column + u * kLanes * 16, 0, LD);
#pragma unroll
    for (int i = 1; i <= M; ++i) {
        if (i > 1 && rank(i) == rank(0)) continue;
        const __amdgpu_buffer_rsrc_t win = __builtin_amdgcn_make_buffer_rsrc(buf[i], 0, to, kRawDword3);
#pragma unroll
        for (int u = 0; u < U; ++u) __builtin_amdgcn_raw_buffer_store_b128(r[u], win, column + u * kLanes * 16, 0, ST);
    }
}

template <int K, int F>
void fill_once_copy(const std::vector<FoldFlow>& flows, void* to) {
    OnceCopyParams<K, F>& p = *static_cast<OnceCopyParams<K, F>*>(to);
    for (size_t f = 0; f < flows.size(); ++f) {
        const FoldFlow& fl = flows[f];
        const unsigned source = fl.seq[0] & 15u;
        p.begin[f] = static_cast<unsigned>(fl.off);
        uint64_t ranks = 0x1111111111111111ull * source;
        int i = 1;
        for (unsigned left = fl.stores & 0xffffu; left; left &= left - 1, ++i)
            ranks ^= static_cast<uint64_t>(static_cast<unsigned>(__builtin_ctz(left)) ^ source) << (i * 4);
        for (int q = 0; q < K / 8; ++q) p.word[f * (K / 8) + q] = static_cast<unsigned>(ranks >> 32 * q);
    }
    p.begin[flows.size()] = static_cast<unsigned>(flows.back().off + flows.back().len);
}

// A kernel, what fills its arguments and where the call's own are: the buffers at the start, so many, and one word.
struct OnceKernel {
    const void* fn = nullptr;
    void (*fill)(const std::vector<FoldFlow>&, void*) = nullptr;
    int bufs = 0;
    size_t call_at = 0;
};
static_assert(sizeof(OnceParams<BLINK_MAX_RANKS, kOnceMostFlows, true>) <= kOnceParamsBytes, "the largest");

// (Two ranks form one sum, the result: no program writes it on the way.)
template <typename T, bool ALL, bool SUM, bool MID, FoldTile TILE, bool MANY>
OnceKernel pick_once(int n) {
    switch (n) {
#define BLINK_CASE(N)                                                                                                                  \
    case N:                                                                                                                            \
        if constexpr (N > 2 || !MID) {                                                                                                 \
            constexpr int kFlows = MANY ? kOnceMostFlows : kOnceFewFlows;                                                              \
            return {reinterpret_cast<const void*>(                                                                                     \
                        blink_once<T, N, kFlows, ALL, SUM, MID, fold_columns(N, ALL, TILE), ALL && TILE == FoldTile::kWhole>),         \
                    fill_once<N, kFlows, MID>, N,                                                                                      \
                    sizeof(void*) * N + 4 * (kFlows + 1 + once_words(N, kFlows) + once_mid_words(N, kFlows, MID))};                    \
        }                                                                                                                              \
        break;
        BLINK_FOLD_CASES
#undef BLINK_CASE
    }
    return {};
}
template <typename T, bool SUM, bool MID>
OnceKernel pick_once(int n, bool all, bool half, bool many) {
    constexpr FoldTile kHalf = FoldTile::kHalf, kWhole = FoldTile::kWhole;
    if (!all) return many ? pick_once<T, false, SUM, MID, kWhole, true>(n) : pick_once<T, false, SUM, MID, kWhole, false>(n);
    if (half) return many ? pick_once<T, true, SUM, MID, kHalf, true>(n) : pick_once<T, true, SUM, MID, kHalf, false>(n);
    return many ? pick_once<T, true, SUM, MID, kWhole, true>(n) : pick_once<T, true, SUM, MID, kWhole, false>(n);
}
// Stages that read n ranks; all: and write them all, else one; half: tiles of half the size; many: more than kOnceFewFlows
// flows; mid: with partial sums written on the way.
OnceKernel once_f32_sum(int n, bool all, bool half, bool many);
OnceKernel once_f32_other(int n, bool all, bool half, bool many);
OnceKernel once_f32_mid(int n, bool all, bool half, bool many, bool sum);
OnceKernel once_i32_sum(int n, bool all, bool half, bool many);
OnceKernel once_i32_other(int n, bool all, bool half, bool many);
OnceKernel once_i32_mid(int n, bool all, bool half, bool many, bool sum);
// Copies to up to m ranks among k; many: more than kOnceFewFlows flows.
OnceKernel once_copy(int k, int m, bool many);
// Columns per wave.  Against blink_fold, geometric means over random sizes with 1 / 2 / 4 columns, up to 7, and 7 to 10 tenths of the
// sizes that have a workgroup per tile: Broadcast to 7 1.13 / 1.13 / 1.12, 1.01 / 1.09 / 1.07, AllGather of 8 1.06 / 1.09 / 1.04,
// 1.00 / 1.06 / 1.02, of 5 1.07 / 1.09 / 1.07, 1.01 / 1.05 / 1.02, Broadcast to 2 1.04 / 1.06 / 1.05, 1.03 / 1.04 / 1.02,
// AllGather of 16 1.38 / 1.33 / 1.27, 1.30 / 1.25 / 1.24; Gather of 8 with 2 / 4 / 8 1.10 / 1.08 / 1.06, 1.07 / 1.06 / 1.07.
constexpr int once_copy_columns(int m) { return m > 8 ? 1 : 2; }

}  // namespace blink
