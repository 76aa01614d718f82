// The device side of schedules whose stages wait for one another (large per-edge programs,
// and any with dependencies where the caller asks for it; fold.hpp has the others): one persistent gfx950 kernel that
// consumes the stage list of all trees concurrently (paper sections 3.3, 4.1, 4.2.1,
// 4.2.2).  kernel_{f32,i32}.hip instantiate it for the two element types, exec.hip holds
// the launcher.
//
// A workgroup is ONE 64-lane wavefront: nothing in the kernel needs a
// workgroup barrier, and a wave that waits for a dependency holds up nobody
// else.  Work unit: (stage instance, tile).  Waves draw units from ticket
// counters in the schedule's execution order, so every unit a wave might have
// to wait for has already been drawn by a running wave, or is about to be (see
// the kernel's loop): waiting can never deadlock, whatever the grid size.
//
// A tile (256..65536 elements, chosen per schedule) is cut into sub-tiles of up to U
// 128-bit columns per lane and rank; a stage reads its ranks in order, combines them one
// after the other and writes the result to its ranks.  A sub-tile's loads are issued
// before the stores of the one in front of it, whose registers are free by then, so that
// they need not wait for those.  (fold.hpp has it the other way round, measured there; here the other
// order has not been measured.)
//
// Chunk-granular hand-over (the paper's per-chunk event): a stage instance has
// a 64-bit counter of finished tiles, and a chunk of 512 KiB or more is handed on in pieces, each
// with a counter of its own (see hand_over_pieces).  Counters are never reset; call number e
// on a schedule waits for e * tiles.  Data handed from stage to stage travels
// with system-scope cache policy (see blink_consume), the counters with
// agent-scope atomics.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <cstdio>
#include <type_traits>
#include <vector>

#include "schedule.hpp"
#include "state.hpp"

namespace blink {

constexpr int kLanes = 64;        // one wavefront per workgroup
constexpr unsigned kMinTile = kLanes * 4;   // elements: one column per lane
constexpr unsigned kMaxTile = 65536;        // elements
// Progress counters sit 256 bytes apart: the few counters that are hot at any
// moment then live in different cache lines and memory channels, so thousands
// of polling waves do not pile up on one of them.
constexpr int kCounterStride = 32;  // in 8-byte words
// Tickets are dealt from several counters ("queues"), ticket t from queue
// t mod n: one counter sustains ~83 fetch-adds per microsecond however many
// waves ask, n counters in different memory channels n times that (measured:
// 540 per microsecond with 8, 1040 with 16).  4 queues and 64 KiB tickets, against one
// queue and 128 KiB: per-edge AllReduce on 8 x 256 MiB 1.336 -> 1.277 ms, per-node
// 1.169 -> 1.125 ms.
constexpr int kMaxQueues = 16;
constexpr unsigned kQueuesHandOver = 4;
constexpr unsigned kTicketBytesHandOver = 64 * 1024;
// The status record at the head of a schedule's device block, 64-bit words.
// Word kStatusState is 0 while all is well.  A wave whose wait for another stage
// outlasts the limit makes it 1 (the first such wave wins), fills in the other
// words and leaves; from then on every wave that looks leaves too, and every
// later launch on the block returns at once, until the host clears the record.
enum : int {
    kStatusState = 0,    // 0 = ok, 1 = a wait was abandoned
    kStatusStage = 1,    // the stage instance that waited
    kStatusAwaited = 2,  // the instance it waited for
    kStatusSeen = 3,     // finished tiles that instance had counted
    kStatusWanted = 4,   // finished tiles it had to reach
    kStatusCall = 5,     // number of the call on its schedule
    kStatusWords = 32,   // the record takes one 256-byte line of its own
};
// The steady counter the waits are timed with ticks at 100 MHz.
constexpr unsigned long long kTicksPerMicrosecond = 100;
constexpr unsigned long long kDefaultWaitMicroseconds = 5000000;  // 5 s: generous; only a bug waits that long

struct KParams {
    void* buf[BLINK_MAX_RANKS];
    const StageTmpl* tmpl;
    const StageInst* inst;
    unsigned long long* done;
    unsigned long long* ticket;
    unsigned long long* status;          // the status record (kStatus* words)
    unsigned long long wait_ticks;       // longest wait for another stage, in ticks of the steady counter
    unsigned long long ticket_base[kMaxQueues];  // value of each queue's counter when this call starts
    unsigned n_queues;
    unsigned long long n_items;
    unsigned long long epoch;
    unsigned tiles_per_chunk;
    unsigned tile_shift;  // a tile is 2^tile_shift elements
    unsigned redop;       // blink_redop_t
    unsigned max_naps;  // longest pause between two looks at a dependency, in units of ~0.2 us
    unsigned n_inst;    // stage instances
    unsigned pieces;    // counters per instance (see hand_over_pieces)
};

// Address spaces: the kernel arguments and the schedule tables are never
// written by the kernel, so they are read through the constant address space,
// which lets wave-uniform reads use the scalar unit.
#define BLINK_CONST __attribute__((address_space(4)))
using ConstParams = const BLINK_CONST KParams*;
using ConstTmpl = const BLINK_CONST StageTmpl*;
using ConstInst = const BLINK_CONST StageInst*;

typedef float F4 __attribute__((ext_vector_type(4)));
typedef unsigned U4 __attribute__((ext_vector_type(4)));  // one 128-bit access, as raw bits

// Element-wise a (+) b on raw bits; `op` is wave-uniform.  fp32 SUM / PROD: one
// IEEE operation per element (round to nearest even, subnormals kept).  int32
// SUM / PROD: unsigned arithmetic, i.e. wrap-around modulo 2^32 without
// signed-overflow UB.  MIN / MAX: signed comparison for int32; for fp32 the
// bits are mapped to keys whose signed order is the IEEE total order (-0 below
// +0; the map is its own inverse), so min and max commute bit for bit.
template <typename T>
__device__ __forceinline__ unsigned combine1(unsigned op, unsigned a, unsigned b);
template <>
__device__ __forceinline__ unsigned combine1<float>(unsigned op, unsigned a, unsigned b) {
    if (op == BLINK_SUM)
        return __builtin_bit_cast(unsigned, __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b));
    if (op == BLINK_PROD)
        return __builtin_bit_cast(unsigned, __builtin_bit_cast(float, a) * __builtin_bit_cast(float, b));
    const int ka = static_cast<int>(a) ^ ((static_cast<int>(a) >> 31) & 0x7fffffff);
    const int kb = static_cast<int>(b) ^ ((static_cast<int>(b) >> 31) & 0x7fffffff);
    const int k = op == BLINK_MIN ? min(ka, kb) : max(ka, kb);
    return static_cast<unsigned>(k ^ ((k >> 31) & 0x7fffffff));
}
template <>
__device__ __forceinline__ unsigned combine1<unsigned>(unsigned op, unsigned a, unsigned b) {
    if (op == BLINK_SUM) return a + b;
    if (op == BLINK_PROD) return a * b;
    const int sa = static_cast<int>(a), sb = static_cast<int>(b);
    return static_cast<unsigned>(op == BLINK_MIN ? min(sa, sb) : max(sa, sb));
}
template <typename T>
__device__ __forceinline__ U4 combine4(unsigned op, U4 a, U4 b) {
    if (op == BLINK_SUM) {  // the common case, kept free of per-element selects
        if constexpr (std::is_same<T, float>::value)
            return __builtin_bit_cast(U4, __builtin_bit_cast(F4, a) + __builtin_bit_cast(F4, b));
        else
            return a + b;
    }
    U4 r;
    r.x = combine1<T>(op, a.x, b.x);
    r.y = combine1<T>(op, a.y, b.y);
    r.z = combine1<T>(op, a.z, b.z);
    r.w = combine1<T>(op, a.w, b.w);
    return r;
}

// acc (+)= in, U columns at a time; `redop` is wave-uniform: one branch per operand, not
// per element (dispatched per column, minima and maxima took twice as long as sums).
template <typename T, bool SUM, int U>
__device__ __forceinline__ void combine_columns(unsigned redop, U4 (&acc)[U], const U4 (&in)[U]) {
    if constexpr (SUM) {
#pragma unroll
        for (int u = 0; u < U; ++u) acc[u] = combine4<T>(BLINK_SUM, acc[u], in[u]);
    } else if (redop == BLINK_MAX) {
#pragma unroll
        for (int u = 0; u < U; ++u) acc[u] = combine4<T>(BLINK_MAX, acc[u], in[u]);
    } else if (redop == BLINK_MIN) {
#pragma unroll
        for (int u = 0; u < U; ++u) acc[u] = combine4<T>(BLINK_MIN, acc[u], in[u]);
    } else {
#pragma unroll
        for (int u = 0; u < U; ++u) acc[u] = combine4<T>(BLINK_PROD, acc[u], in[u]);
    }
}

// Byte `field_offset + i` of a stage template, fetched as part of a 32-bit word
// so that the scalar unit can do it.
__device__ __forceinline__ unsigned tmpl_byte(ConstTmpl st, unsigned byte_index) {
    const BLINK_CONST uint32_t* w = reinterpret_cast<const BLINK_CONST uint32_t*>(st);
    return (w[byte_index >> 2] >> ((byte_index & 3u) * 8u)) & 0xffu;
}
#define BLINK_TMPL(st, field, i) tmpl_byte(st, static_cast<unsigned>(offsetof(StageTmpl, field)) + (i))

// Rank buffers are accessed through buffer descriptors that cover exactly the
// bytes still to be processed: lanes past the end read zeros and their stores
// are dropped by the hardware range check, so ragged ends need no branches.
// The cache-policy bits of each access are chosen per kernel flavour (below).
constexpr int kRawDword3 = 0x00020000;  // raw 32-bit data format, no swizzle (gfx9 family)
constexpr int kPolicyDefault = 0;
constexpr int kPolicyStream = 2;        // nt: streamed once, do not keep in cache
constexpr int kPolicyThrough = 16;      // sc1: agent scope, stores written through
constexpr int kPolicySystem = 17;       // sc0 sc1: bypass / write through every cache level

// Where stages hand chunks over to one another loads and stores bypass the caches
// (see blink_consume); the loads also carry the streaming hint, which changes no
// scope.  Per-edge AllReduce, 8 x 256 MiB (load policy, store policy -> ms): (sc0 sc1,
// sc0 sc1) 1.417, (sc0 sc1 nt, sc0 sc1) 1.337, nt on stores 1.65-1.72.
constexpr int kPolicyLoadHandOver = kPolicySystem | kPolicyStream;
constexpr int kPolicyStoreHandOver = kPolicySystem;

// The rank buffers' addresses live in a vector register pair, lane r holding rank
// r's (loaded once per wave): a rank's pointer is then one readlane away instead
// of a scalar load that depends on another scalar load (the rank's number from
// the stage's table), twice per rank and sub-tile.
struct RankTable {
    unsigned lo, hi;
};
__device__ __forceinline__ RankTable load_rank_table(ConstParams p, int lane) {
    const unsigned long long mine = reinterpret_cast<unsigned long long>(p->buf[lane & (BLINK_MAX_RANKS - 1)]);
    return {static_cast<unsigned>(mine), static_cast<unsigned>(mine >> 32)};
}
__device__ __forceinline__ unsigned long long rank_base(RankTable t, unsigned rank) {
    const unsigned lo = __builtin_amdgcn_readlane(t.lo, rank);
    const unsigned hi = __builtin_amdgcn_readlane(t.hi, rank);
    return (static_cast<unsigned long long>(hi) << 32) | lo;
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rank_window(RankTable t, unsigned rank,
                                                              unsigned long long byte_off, unsigned bytes) {
    char* base = reinterpret_cast<char*>(rank_base(t, rank) + byte_off);
    return __builtin_amdgcn_make_buffer_rsrc(base, 0, static_cast<int>(bytes), kRawDword3);
}

// A stage that reads N ranks over `bytes` bytes (a multiple of 16) at byte_off, U
// columns per lane and sub-tile.  Columns past the end of a ragged tile fall outside
// the window: such loads return zeros and such stores are dropped.
template <typename T, int N, int U>
__device__ __forceinline__ void run_stage(ConstParams p, RankTable ranks, ConstTmpl st, unsigned long long byte_off,
                                          unsigned bytes, int lane) {
    constexpr unsigned kSubBytes = kLanes * U * 16;
    const unsigned redop = p->redop;
    const int n_store = BLINK_TMPL(st, n_store, 0);
    U4 r[N][U];
    auto load = [&](unsigned at) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const __amdgpu_buffer_rsrc_t win = rank_window(ranks, BLINK_TMPL(st, load_rank, i), byte_off, bytes);
#pragma unroll
            for (int u = 0; u < U; ++u)
                r[i][u] = __builtin_amdgcn_raw_buffer_load_b128(win, at + (u * kLanes + lane) * 16, 0, kPolicyLoadHandOver);
        }
    };
    load(0);
    for (unsigned at = 0; at < bytes; at += kSubBytes) {
        U4 acc[U];
#pragma unroll
        for (int u = 0; u < U; ++u) acc[u] = r[0][u];
#pragma unroll
        for (int i = 1; i < N; ++i) {
            if (redop == BLINK_SUM)
                combine_columns<T, true, U>(redop, acc, r[i]);
            else
                combine_columns<T, false, U>(redop, acc, r[i]);
        }
        if (at + kSubBytes < bytes) load(at + kSubBytes);
        for (int j = 0; j < n_store; ++j) {
            const __amdgpu_buffer_rsrc_t win = rank_window(ranks, BLINK_TMPL(st, store_rank, j), byte_off, bytes);
#pragma unroll
            for (int u = 0; u < U; ++u)
                __builtin_amdgcn_raw_buffer_store_b128(acc[u], win, at + (u * kLanes + lane) * 16, 0, kPolicyStoreHandOver);
        }
    }
}

// The same for any number of ranks, one after the other: the fan-ins of per-node programs,
// which only come here where the caller asks for it (see blink_schedule_set_hand_over).
template <typename T>
__device__ __forceinline__ void run_stage_any(ConstParams p, RankTable ranks, ConstTmpl st, unsigned long long byte_off,
                                              unsigned bytes, int lane) {
    constexpr int U = 4;
    const unsigned redop = p->redop;
    const int n_load = BLINK_TMPL(st, n_load, 0), n_store = BLINK_TMPL(st, n_store, 0);
    for (unsigned at = 0; at < bytes; at += kLanes * U * 16) {
        U4 acc[U], in[U];
        for (int i = 0; i < n_load; ++i) {
            const __amdgpu_buffer_rsrc_t win = rank_window(ranks, BLINK_TMPL(st, load_rank, i), byte_off, bytes);
#pragma unroll
            for (int u = 0; u < U; ++u)
                in[u] = __builtin_amdgcn_raw_buffer_load_b128(win, at + (u * kLanes + lane) * 16, 0, kPolicyLoadHandOver);
            if (i == 0) {
#pragma unroll
                for (int u = 0; u < U; ++u) acc[u] = in[u];
            } else if (redop == BLINK_SUM) {
                combine_columns<T, true, U>(redop, acc, in);
            } else {
                combine_columns<T, false, U>(redop, acc, in);
            }
        }
        for (int j = 0; j < n_store; ++j) {
            const __amdgpu_buffer_rsrc_t win = rank_window(ranks, BLINK_TMPL(st, store_rank, j), byte_off, bytes);
#pragma unroll
            for (int u = 0; u < U; ++u)
                __builtin_amdgcn_raw_buffer_store_b128(acc[u], win, at + (u * kLanes + lane) * 16, 0, kPolicyStoreHandOver);
        }
    }
}

// The same for up to kLanes single 4-byte elements: the ragged end of a payload
// whose length is not a multiple of 4 elements, and chunks that do not start on
// a 16-byte boundary.  Slow path; one element per lane.
template <typename T>
__device__ __forceinline__ void run_scalar(ConstParams p, RankTable ranks, ConstTmpl st, unsigned long long byte_off,
                                           unsigned bytes, int lane) {
    const int n_load = BLINK_TMPL(st, n_load, 0), n_store = BLINK_TMPL(st, n_store, 0);
    unsigned acc = 0;
    for (int i = 0; i < n_load; ++i) {
        const __amdgpu_buffer_rsrc_t win = rank_window(ranks, BLINK_TMPL(st, load_rank, i), byte_off, bytes);
        const unsigned x = __builtin_amdgcn_raw_buffer_load_b32(win, lane * 4, 0, kPolicyLoadHandOver);
        acc = i == 0 ? x : combine1<T>(p->redop, acc, x);
    }
    for (int j = 0; j < n_store; ++j) {
        const __amdgpu_buffer_rsrc_t win = rank_window(ranks, BLINK_TMPL(st, store_rank, j), byte_off, bytes);
        __builtin_amdgcn_raw_buffer_store_b32(acc, win, lane * 4, 0, kPolicyStoreHandOver);
    }
}

// T: element type (float, or unsigned for wrap-around int32).  Stages hand chunks over
// to each other, possibly across XCDs whose L2 caches are not coherent with one another:
// all rank-buffer accesses use system-scope cache policy (loads bypass, stores write
// through; the loads also carry the streaming hint, which changes no scope), so the
// hand-over needs no L2 write-back or invalidate, only "my stores have completed" before
// the counter is bumped.
// Programs whose stages wait for one another combine their ranks in the order of
// load_rank (edge_stages, node_stages in schedule.cpp): the micro-program is not looked at.
// Bound by the memory side, which serves 140 bytes per element for 8 ranks: 8 x 64 MiB
// per edge in 1 MiB chunks 345 us, 6.8 TB/s of requests (through LDS slots and the
// micro-program, sub-tiles not overlapped: fp32 376, int32 410 us).
// The by-value argument is only there to size the kernel-argument segment; it is
// read through the constant address space (see ConstParams).
template <typename T>
__global__ __launch_bounds__(kLanes, 1) void blink_consume(const KParams) {
    const int lane = threadIdx.x;
    ConstParams p = (ConstParams)__builtin_amdgcn_kernarg_segment_ptr();
    const RankTable ranks = load_rank_table(p, lane);
    unsigned long long* const ticket = p->ticket;
    unsigned long long* const done = p->done;
    ConstTmpl const tmpl = reinterpret_cast<ConstTmpl>(reinterpret_cast<unsigned long long>(p->tmpl));
    ConstInst const inst = reinterpret_cast<ConstInst>(reinterpret_cast<unsigned long long>(p->inst));
    const unsigned long long n_items = p->n_items, epoch = p->epoch;
    const unsigned n_queues = p->n_queues;
    const unsigned tiles_per_chunk = p->tiles_per_chunk;
    const unsigned tile_shift = p->tile_shift;
    const unsigned tile_elems = 1u << tile_shift;
    const unsigned n_inst = p->n_inst, pieces = p->pieces;

    // Lane-dependent regions.  readfirstlane needs lane 0 present, so the
    // compiler must never get the chance to let some lanes run ahead of lane 0
    // around the loop: a version with a lane-0 region at the tail of the loop
    // (completion signal) and one at its head (ticket draw) had the two merged
    // across the back edge and hung.  Hence the completion signal of a tile is
    // posted together with the next ticket draw, in ONE lane-0 region at the
    // head, and the back edges are wave-uniform.  The only other lane-dependent
    // region is the wait for dependencies in the middle of the body (lanes
    // below n_dep poll one counter each).  It cannot be merged with the region
    // at the head in either direction: between the two, on both sides, lies
    // wave-uniform code with effects of its own (the readfirstlane pair and the
    // ticket arithmetic after the head; the tile's loads and stores after the
    // wait), and the wait ends in a ballot over all lanes, which the lanes can
    // only reach together.  All other branches are wave-uniform.
    //
    // Ticket j * n_queues + q is the j-th of queue q.  A wave starts on queue (its
    // number mod n_queues), stays with it until it is empty and then goes round the
    // others, so every wave draws exactly one ticket past the end of every queue.
    // The grid has at least n_queues waves, so each queue has waves of its own; this
    // keeps the schedule free of deadlock: take the first unfinished ticket t in
    // schedule order.  Everything it waits for is finished.  If t is drawn its
    // holder runs; if not, its queue is not empty, the queue's own waves hold
    // only earlier tickets of that queue, which are finished, so one of them
    // draws t next.
    //
    // A block whose status record is set (an earlier call gave up a wait, so its
    // counters no longer mean anything) is left alone.
    unsigned long long* const status = p->status;
    if (__hip_atomic_load(status + kStatusState, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return;
    unsigned queue = blockIdx.x % n_queues, empty_queues = 0;
    long long pending = -1;  // counter in which a finished tile still has to be counted
    for (;;) {
        unsigned long long raw = 0;
        if (lane == 0) {
            if (pending >= 0)
                __hip_atomic_fetch_add(done + pending * kCounterStride, 1ull, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
            raw = __hip_atomic_fetch_add(ticket + queue * kCounterStride, 1ull, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
        }
        pending = -1;
        const unsigned lo = __builtin_amdgcn_readfirstlane(static_cast<unsigned>(raw));
        const unsigned hi = __builtin_amdgcn_readfirstlane(static_cast<unsigned>(raw >> 32));
        const unsigned long long nth = ((static_cast<unsigned long long>(hi) << 32) | lo) - p->ticket_base[queue];
        const unsigned long long t = nth * n_queues + queue;
        if (t >= n_items) {  // this queue is empty: on to the next, or done
            if (++empty_queues == n_queues) break;
            queue = queue + 1 == n_queues ? 0 : queue + 1;
            continue;
        }
        // ticket -> (instance, tile), instance by instance
        unsigned ii, tile;
        ticket_to_tile(t, 1, tiles_per_chunk, n_inst, &ii, &tile);
        ConstInst in = inst + ii;
        // Tiles lie on the absolute grid of tile_elems-element blocks of the
        // payload, so tile starts are 128-byte (indeed tile-size) aligned even
        // when a tree's share starts at an odd multiple of 16 bytes; the first
        // and last tile of an instance are the ragged ones.
        const unsigned long long off = in->off, end = off + in->len;
        const unsigned long long block_lo = ((off >> tile_shift) + tile) << tile_shift;
        const unsigned long long lo_e = max(off, block_lo);
        const unsigned long long hi_e = min(end, block_lo + tile_elems);
        if (lo_e < hi_e) {  // instances have at most tiles_per_chunk tiles, some fewer
            const unsigned tlen = static_cast<unsigned>(hi_e - lo_e);
            ConstTmpl st = tmpl + in->tmpl;

            // the tile's piece of the instance: its counter and its ends
            unsigned long long piece = 0, piece_lo = off, piece_hi = end;
            if (pieces > 1) {
                const unsigned long long block = block_lo >> kPieceShift;
                piece = block - (off >> kPieceShift);
                piece_lo = max(off, block << kPieceShift);
                piece_hi = min(end, (block + 1) << kPieceShift);
            }
            const int n_dep = in->n_dep;
            if (n_dep) {
                bool gave_up = false;
                if (lane < n_dep) {
                    const unsigned long long want =
                        epoch * (((piece_hi + tile_elems - 1) >> tile_shift) - (piece_lo >> tile_shift));
                    const unsigned long long* f =
                        done + (static_cast<unsigned long long>(in->dep[lane]) * pieces + piece) * kCounterStride;
                    // poll, backing off (up to ~0.8 us between looks for large
                    // schedules) so that waiting waves leave the memory system
                    // to the working ones.  Every 64th look also checks the
                    // clock and the status record: a wait that outlasts the
                    // limit, or any wait once another wave has given up, ends
                    // here, and the wave leaves the kernel.
                    const unsigned max_naps = p->max_naps;
                    unsigned naps = 1, looks = 0;
                    unsigned long long since = 0, seen;
                    while ((seen = __hip_atomic_load(f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) < want) {
                        for (unsigned i = 0; i < naps; ++i) __builtin_amdgcn_s_sleep(8);
                        if (naps < max_naps) naps *= 2;
                        if ((++looks & 63u) != 0) continue;
                        const unsigned long long now = wall_clock64();
                        if (since == 0) since = now;
                        const bool late = now - since > p->wait_ticks;
                        if (late && __hip_atomic_exchange(status + kStatusState, 1ull, __ATOMIC_RELAXED,
                                                          __HIP_MEMORY_SCOPE_AGENT) == 0) {
                            status[kStatusStage] = ii;
                            status[kStatusAwaited] = static_cast<unsigned long long>(in->dep[lane]);
                            status[kStatusSeen] = seen;
                            status[kStatusWanted] = want;
                            status[kStatusCall] = epoch;
                        }
                        if (late || __hip_atomic_load(status + kStatusState, __ATOMIC_RELAXED,
                                                      __HIP_MEMORY_SCOPE_AGENT) != 0) {
                            gave_up = true;
                            break;
                        }
                    }
                }
                if (__builtin_amdgcn_ballot_w64(gave_up) != 0) break;  // wave-uniform: leave the kernel
                // orders the polls before the data loads; the loads themselves bypass the caches
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
            }

            const unsigned long long e0 = lo_e;  // first element of the tile
            if ((e0 & 3ull) == 0) {
                const unsigned vec_bytes = (tlen >> 2) * 16u;
                if (vec_bytes) {
                    const unsigned n_load = BLINK_TMPL(st, n_load, 0);
                    if (n_load == 1)
                        run_stage<T, 1, 16>(p, ranks, st, e0 * 4ull, vec_bytes, lane);
                    else if (n_load == 2)
                        run_stage<T, 2, 16>(p, ranks, st, e0 * 4ull, vec_bytes, lane);
                    else
                        run_stage_any<T>(p, ranks, st, e0 * 4ull, vec_bytes, lane);
                }
                const unsigned rem = tlen & 3u;  // only where the payload itself ends off a 16-byte boundary
                if (rem) run_scalar<T>(p, ranks, st, e0 * 4ull + vec_bytes, rem * 4u, lane);
            } else {
                // chunk size not a multiple of 4 elements: element-wise, slow but correct
                for (unsigned b = 0; b < tlen * 4u; b += kLanes * 4u)
                    run_scalar<T>(p, ranks, st, e0 * 4ull + b, min(static_cast<unsigned>(kLanes) * 4u, tlen * 4u - b), lane);
            }

            if (BLINK_TMPL(st, signals, 0)) {
                // every store of this wave has reached memory before the counter moves
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                __builtin_amdgcn_s_waitcnt(0);
                pending = static_cast<long long>(static_cast<unsigned long long>(ii) * pieces + piece);
            }
        }
    }
}

// ---- what the launcher sees ---------------------------------------------------------
using KernelFn = void (*)(const KParams);

// Per element type, each in a translation unit of its own, so that they compile side by
// side.
KernelFn kernel_f32();
KernelFn kernel_i32();

}  // namespace blink
