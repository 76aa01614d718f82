// The fold kernel for payloads that have a workgroup for every tile (fold.hpp has the larger
// ones, and says what a tile and a stack program are).
//
// Such a call is bound by the latency of one pass: arguments, rank data, stores.  What lies in
// front of the loads counts in full, and so does the length of the code, which every call
// fetches anew (1.5 to 3 KB here, 5 to 9 KB in fold.hpp).  So the place in the grid says which flow (y) and
// which of its tiles (x) a workgroup has, two rounds of scalar loads, the second from
// lines that the first has fetched, stand between a wave's start and its rank loads: no tickets, no levels, no loop.
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

// Where whole tiles are handed out (the upper two fifths of the range) two workgroups at a time run on a CU, by the LDS
// they ask for: more loads in flight spread the requests out.  Against as many as fit, us: 8 ranks x 9.5 MiB 24.9 / 22.9,
// 8.8 MiB 20.8 / 19.2, 4 ranks x 16 MiB 20.3 / 18.3; half tiles there 24.1, 19.5, 17.9.
constexpr int kLdsOfFew = 56 * 1024;

// The arguments are short: a launch with at most 112 bytes of them takes the host less time (C call on one host, 3 to 7
// ranks 3.0 us, 8 ranks with 120 bytes 3.7, with 370 or more 3.8 to 4; on another host 2.24 up to 112 bytes, 2.30 beyond).
// So a buffer's address is one more scalar load away, from a line that is there by then, a flow's program is packed as tightly as
// that takes for 8 ranks, and there are two variants, for few flows and for many (kOnceMostFlows).
constexpr int kOnceFewFlows = 4;
// Flow f's program: the ranks in the order of consumption, and for each push | folds << 1.  Up to 4 ranks: word f, four
// bits per rank, the codes from bit 16 on.  Up to 8: word f, three bits per rank, the low byte of the codes from bit 24
// on; the other two, three bits per code, are a half of word F + f / 2.  More: words 4 f and 4 f + 1, four bits per rank, and
// the codes in the next two.
constexpr int once_words(int n, int flows) { return n <= 4 ? flows : n <= 8 ? flows + (flows + 1) / 2 : 4 * flows; }
template <int N, int F>
struct OnceParams {
    void* buf[N];
    unsigned begin[F + 1];    // flow f: elements [begin[f], begin[f + 1])
    unsigned word[once_words(N, F)];
    unsigned call;            // see once_call
};
static_assert(sizeof(OnceParams<8, kOnceFewFlows>) <= 112, "see above");

// FEW: at most two workgroups at a time on a CU.
template <typename T, int N, int F, bool SUM, int U, bool FEW>
__global__ __launch_bounds__(kFoldThreads) void blink_once(const OnceParams<N, F>) {
    constexpr int kParked = N < 4 ? 0 : N / 2 - 1;   // accumulators in LDS (see blink_fold)
    constexpr int kParkedBytes = kParked * U * kFoldThreads * 16;
    constexpr int kLdsBytes = FEW ? std::max(kParkedBytes, kLdsOfFew) : std::max(kParkedBytes, 16);
    __shared__ U4 parked[kLdsBytes / 16];
    const BLINK_CONST OnceParams<N, F>* p = (const BLINK_CONST OnceParams<N, F>*)__builtin_amdgcn_kernarg_segment_ptr();
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
    asm volatile("" ::"s"(begin), "s"(end), "s"(order[0]), "s"(call), "s"(p->buf[0]), "s"(p->buf[N - 1]));   // all of them with one wait
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

// What of the arguments is the same for all calls on a schedule: all but the buffers and `call`.
template <int N, int F>
void fill_once(const std::vector<FoldFlow>& flows, void* to) {
    OnceParams<N, F>& p = *static_cast<OnceParams<N, F>*>(to);
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
static_assert(sizeof(OnceParams<BLINK_MAX_RANKS, kOnceMostFlows>) <= kOnceParamsBytes, "the largest");

template <typename T, bool SUM, FoldTile TILE, bool MANY>
OnceKernel pick_once(int n) {
    switch (n) {
#define BLINK_CASE(N)                                                                                                              \
    case N: {                                                                                                                      \
        constexpr int kFlows = MANY ? kOnceMostFlows : kOnceFewFlows;                                                          \
        return {reinterpret_cast<const void*>(                                                                                     \
                    blink_once<T, N, kFlows, SUM, fold_columns(N, true, TILE), TILE == FoldTile::kWhole>),                         \
                fill_once<N, kFlows>, N, sizeof(void*) * N + 4 * (kFlows + 1 + once_words(N, kFlows))};                                                  \
    }
        BLINK_FOLD_CASES
#undef BLINK_CASE
        default: return {};
    }
}
template <typename T, bool SUM>
OnceKernel pick_once(int n, bool half, bool many) {
    if (half) return many ? pick_once<T, SUM, FoldTile::kHalf, true>(n) : pick_once<T, SUM, FoldTile::kHalf, false>(n);
    return many ? pick_once<T, SUM, FoldTile::kWhole, true>(n) : pick_once<T, SUM, FoldTile::kWhole, false>(n);
}
// Stages that read n ranks and write them all; half: tiles of half the size; many: more than kOnceFewFlows flows.
OnceKernel once_f32_sum(int n, bool half, bool many);
OnceKernel once_f32_other(int n, bool half, bool many);
OnceKernel once_i32_sum(int n, bool half, bool many);
OnceKernel once_i32_other(int n, bool half, bool many);

// Copies to up to m ranks among k; many: more than kOnceFewFlows flows.
OnceKernel once_copy(int k, int m, bool many);
// Columns per wave.  Against blink_fold, geometric means over random sizes with 1 / 2 / 4 columns, up to 7, and 7 to 10 tenths of the
// sizes that have a workgroup per tile: Broadcast to 7 1.13 / 1.13 / 1.12, 1.01 / 1.09 / 1.07, AllGather of 8 1.06 / 1.09 / 1.04,
// 1.00 / 1.06 / 1.02, of 5 1.07 / 1.09 / 1.07, 1.01 / 1.05 / 1.02, Broadcast to 2 1.04 / 1.06 / 1.05, 1.03 / 1.04 / 1.02,
// AllGather of 16 1.38 / 1.33 / 1.27, 1.30 / 1.25 / 1.24; Gather of 8 with 2 / 4 / 8 1.10 / 1.08 / 1.06, 1.07 / 1.06 / 1.07.
constexpr int once_copy_columns(int m) { return m > 8 ? 1 : 2; }

}  // namespace blink
