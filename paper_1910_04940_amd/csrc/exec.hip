// The launcher of the kernels (kernel.hpp: stages that wait for one another;
// fold.hpp: the others, fold_once.hpp: small payloads of those): the device block of a schedule (status record, progress
// counters, tables), the launch plan, the launch and its bookkeeping.
#include "fold_once.hpp"

#include <atomic>
#include <cstring>
#include <mutex>

namespace blink {

// ---- a device block that needs no allocation ------------------------------------------
// For callers that may not allocate (a stream under HIP graph capture, a tight
// serving loop, a harness that forbids it): a block of fixed size in the
// library's own device image.  Every GPU the library runs on holds its own copy
// of the array, at its own address, until the process ends; host code reaches
// it only through the address hipGetSymbolAddress returns with that GPU current
// (the array's name in host code is a host-side stand-in, not a device address).
// All calls of blink_allreduce_noalloc on one GPU share that GPU's block.
static __device__ __align__(256) unsigned char scratch[kStaticBlockBytes];

namespace {
constexpr int kMaxDevices = 64;
struct StaticBlock {
    char* ptr = nullptr;   // device address of `scratch` on this GPU
    uint64_t owner = 0;    // id of the schedule whose tables the block holds (0 = none)
    bool fold = false;     // they are the fold kernel's, not those of stages that wait
};
StaticBlock g_static[kMaxDevices];
std::mutex g_static_mutex;
std::atomic<uint64_t> g_next_id{1};

// Zeroes `words` 64-bit words (a fill kernel rather than hipMemsetAsync, which
// must not be recorded into a captured graph).
__global__ __launch_bounds__(256) void blink_clear(unsigned long long* p, unsigned long long words) {
    for (unsigned long long i = blockIdx.x * 256ull + threadIdx.x; i < words; i += gridDim.x * 256ull) p[i] = 0;
}
}  // namespace

uint64_t next_schedule_id() { return g_next_id.fetch_add(1); }

// ---- host side ------------------------------------------------------------------------
namespace {

#define BLINK_HIP(call)                                                                   \
    do {                                                                                  \
        hipError_t err__ = (call);                                                        \
        if (err__ != hipSuccess) {                                                        \
            std::fprintf(stderr, "blink: %s failed: %s\n", #call, hipGetErrorString(err__)); \
            return err__ == hipErrorOutOfMemory ? BLINK_ENOMEM : BLINK_EHIP;              \
        }                                                                                 \
    } while (0)

KernelFn pick_kernel(blink_dtype_t dtype) { return dtype == BLINK_FP32 ? kernel_f32() : kernel_i32(); }

size_t round_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// The status record and the ticket counters, at the head of a block whatever follows.
constexpr size_t kLine = static_cast<size_t>(kCounterStride) * sizeof(unsigned long long);
constexpr size_t kTicketAt = static_cast<size_t>(kStatusWords) * sizeof(unsigned long long);   // the fold kernel relies on it
constexpr size_t kHeadBytes = kTicketAt + kMaxQueues * kLine;

BlockLayout layout_of(const Schedule& s, Served served, bool static_block) {
    BlockLayout l;
    l.ticket = kTicketAt;
    l.done = kHeadBytes;
    l.pieces = counters_per_stage(s, served, kLine, static_block);
    l.counters_end = l.done + s.inst.size() * l.pieces * kLine;
    l.tmpl = round_up(l.counters_end, 256);
    l.inst = round_up(l.tmpl + s.tmpl.size() * sizeof(StageTmpl), 256);
    l.bytes = round_up(l.inst + s.inst.size() * sizeof(StageInst), 256);
    l.words = l.done;   // a flow has an instance at least, hence kLine bytes
    static_assert(kLine >= FoldTables::words_per_flow() * sizeof(uint32_t), "the tables fit the space of the counters");
    return l;
}

// Bytes at the head of a block that are zero when a schedule is new.
size_t cleared_bytes(const LaunchPlan& pl, const BlockLayout& l) { return pl.fold ? l.done : l.counters_end; }

// What of a fold plan travels in the kernel's arguments.  Tables that do not are the same for
// every tile size (see kLevelSets) and every distance past a 1 KiB boundary.
bool words_inline(const blink_schedule& h) { return h.fold.flows.size() <= kInlineFlows; }
bool levels_inline(const blink_schedule& h) { return h.fold.levels.size() <= kInlineFlows; }

// Copy a schedule's tables into a block on the current device.  Synchronous.
blink_status_t copy_tables(const blink_schedule& h, const BlockLayout& l, char* block) {
    const LaunchPlan& pl = h.plan;
    const Schedule& s = h.s;
    if (!pl.fold) {
        BLINK_HIP(hipMemcpy(block + l.tmpl, s.tmpl.data(), s.tmpl.size() * sizeof(StageTmpl), hipMemcpyHostToDevice));
        BLINK_HIP(hipMemcpy(block + l.inst, s.inst.data(), s.inst.size() * sizeof(StageInst), hipMemcpyHostToDevice));
    } else if (!words_inline(h)) {
        const std::vector<uint32_t>& t = h.fold.tables;
        BLINK_HIP(hipMemcpy(block + l.words, t.data(), t.size() * sizeof(uint32_t), hipMemcpyHostToDevice));
    }
    return BLINK_OK;
}

// A schedule belongs to the device of its first call.
blink_status_t bind_device(blink_schedule* h) {
    int dev = -1;
    BLINK_HIP(hipGetDevice(&dev));
    if (h->device >= 0 && h->device != dev) return BLINK_EMISMATCH;
    h->device = dev;
    return BLINK_OK;
}

// The schedule's own block: one allocation, made at the first call that needs it and
// made anew where a plan needs a larger one (chunks that are handed on in pieces, on a caller's request).
// Synchronously zeroed and filled, then and when a new plan needs other tables.
// Nothing is left behind when a step fails.
blink_status_t upload(blink_schedule* h, const BlockLayout& l) {
    if (h->d_block && !h->tables_stale) return BLINK_OK;
    void* block = h->d_block;
    if (block) BLINK_HIP(hipDeviceSynchronize());   // calls under the old plan
    const bool anew = h->block_bytes < l.bytes;
    if (anew) BLINK_HIP(hipMalloc(&block, l.bytes));
    blink_status_t st = BLINK_OK;
    const hipError_t zeroed = hipMemset(block, 0, cleared_bytes(h->plan, l));
    if (zeroed != hipSuccess) {
        std::fprintf(stderr, "blink: hipMemset failed: %s\n", hipGetErrorString(zeroed));
        st = BLINK_EHIP;
    }
    if (st == BLINK_OK) st = copy_tables(*h, l, static_cast<char*>(block));
    if (st != BLINK_OK) {
        if (anew) (void)hipFree(block);
        return st;
    }
    if (anew) {
        if (h->d_block) (void)hipFree(h->d_block);
        h->d_block = block;
        h->block_bytes = l.bytes;
    }
    BLINK_HIP(hipDeviceSynchronize());
    h->tables_stale = false;
    return BLINK_OK;
}

// The current device's static block, holding the tables of `h`.  The address is
// looked up once per device.  The tables are copied in when the block last
// held another schedule's (synchronously, after waiting for `stream`, whose
// earlier calls may still be reading the old ones).  Allocates nothing.
blink_status_t claim_static_block(blink_schedule* h, const BlockLayout& l, hipStream_t stream, char** out) {
    int dev = -1;
    BLINK_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return BLINK_ELIMIT;
    if (l.bytes > kStaticBlockBytes) {
        std::fprintf(stderr, "blink: the schedule needs a device block of %zu bytes, the static one has %zu\n",
                     l.bytes, kStaticBlockBytes);
        return BLINK_ELIMIT;
    }
    std::lock_guard<std::mutex> lock(g_static_mutex);
    StaticBlock& sb = g_static[dev];
    if (!sb.ptr) {
        char* ptr = nullptr;
        BLINK_HIP(hipGetSymbolAddress(reinterpret_cast<void**>(&ptr), HIP_SYMBOL(scratch)));
        if (!ptr) return BLINK_EHIP;
        sb.ptr = ptr;
    }
    if (sb.owner != h->id || sb.fold != h->plan.fold) {
        // waiting and copying are not things a capturing stream can record
        hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(stream, &capture) != hipSuccess) {
            (void)hipGetLastError();
        } else if (capture != hipStreamCaptureStatusNone) {
            std::fprintf(stderr, "blink: the stream is capturing and the static block holds another schedule's tables; "
                                 "call blink_allreduce_noalloc on this schedule once before the capture\n");
            return BLINK_EINVAL;
        }
        sb.owner = 0;
        BLINK_HIP(hipStreamSynchronize(stream));
        if (const blink_status_t st = copy_tables(*h, l, sb.ptr)) return st;
        sb.owner = h->id;
        sb.fold = h->plan.fold;
    }
    h->last_static_device = dev;
    *out = sb.ptr;
    return BLINK_OK;
}

// The plan where stages wait for one another.  Tickets move about
// kTicketBytesHandOver bytes.
void plan_hand_over(blink_schedule* h) {
    LaunchPlan& pl = h->plan;
    const Schedule& s = h->s;
    uint64_t work = 0;  // elements x stages
    for (const StageInst& in : s.inst) work += in.len;
    const uint64_t bytes_per_elem = std::max<uint64_t>(1, s.traffic_bytes / std::max<uint64_t>(1, work));
    // the power of two nearest (in ratio) to ticket bytes / bytes_per_elem
    const uint64_t ticket_bytes = kTicketBytesHandOver;
    unsigned tile = kMinTile;
    while (tile < kMaxTile && 2ull * tile * tile * bytes_per_elem * bytes_per_elem < ticket_bytes * ticket_bytes)
        tile *= 2;
    if (h->tile_override) tile = h->tile_override;
    pl.tile_elems = tile;
    pl.tile_shift = 0;
    while ((1u << pl.tile_shift) < tile) ++pl.tile_shift;
    pl.n_items = ticket_count(s, 1, pl.tile_shift, &pl.tiles_per_chunk);
}

// The plan where the fold kernel runs the schedule.  A drawn ticket is one sub-tile of the
// kernel, or as many as make it move 56 KiB, which two counters keep up with (see fold_grid).
// A payload of at most five tiles (of 128 KiB read and written) per CU gets a workgroup for every tile, and no ticket has to
// be drawn, unless blink_once can serve such schedules and no longer does at this size (see once_bytes_per_cu).  Where ranks are
// combined they are all resident at once or nearly so; the
// small tiles of a copy need not be (to two ranks a CU gets up to 27 workgroups and holds eight) (probe, 8 ranks,
// workgroup per tile against 224 that draw: 2 MiB per rank 5.1 / 7.2 us, 4 MiB 9.6 /
// 10.8, 7 MiB (3.5 tiles per CU) 14.4 / 16.2, 10.4 MiB (5.2) 25 / 25, 16 MiB 51 / 47).  Larger ones that blink_once
// serves draw tickets where a caller's wish takes them to this kernel (see once_call_serves).
constexpr unsigned kFoldTicketBytes = 56 * 1024;
constexpr unsigned kFoldRunElems = 32 * 1024;
constexpr uint64_t kFoldSmallBytesPerCu = 5 * 128 * 1024;
constexpr uint64_t kOnceHalfBytesPerCu = 3 * 128 * 1024;   // up to here half tiles in the kernel that does nothing else (see kLdsOfFew)
constexpr unsigned kFoldHalfTilesPerCu = 2;   // up to here half tiles are faster (see fold_columns)

FoldTile fold_tile(const LaunchPlan& pl) { return pl.half ? FoldTile::kHalf : pl.small ? FoldTile::kWhole : FoldTile::kDrawn; }

void plan_fold(blink_schedule* h) {
    LaunchPlan& pl = h->plan;
    const Schedule& s = h->s;
    pl.n_load = s.fused[0].stage.n_load;
    const uint32_t n_store = s.fused[0].stage.n_store;
    pl.all = pl.n_load > 1 && n_store == pl.n_load;
    for (const FusedFlow& f : s.fused) pl.mid = pl.mid || f.mid_store != 0;
    pl.kernel_bytes = fold_bytes(s);
    const int n = static_cast<int>(pl.n_load);
    pl.copy_columns = n == 1 ? fold_copy_columns(s) : 0;
    const unsigned sub = fold_sub_elems(n == 1 ? pl.copy_columns : fold_columns(n, pl.all, FoldTile::kWhole));
    uint64_t tiles = 0;
    for (const FoldFlow& f : h->fold.flows) tiles += (f.len + sub - 1) / sub;
    const uint64_t cus = static_cast<uint64_t>(h->n_cu);
    if (n == 1) pl.once_stores = static_cast<int>(once_stores(h->fold.once));
    const bool once_can = h->tile_override == 0 && !h->fold.once.empty();
    pl.once = once_can && once_serves(s, h->fold.once, cus);
    pl.once_half = pl.kernel_bytes <= kOnceHalfBytesPerCu * cus;
    pl.small = (pl.once || !once_can) && tiles * sub * 4 * (pl.n_load + n_store) <= kFoldSmallBytesPerCu * cus;
    // a tile per flow more than that: shares need not be whole tiles
    pl.half = pl.small && pl.all && tiles <= kFoldHalfTilesPerCu * cus + h->fold.flows.size();
    if (pl.small && n == 1 && n_store > 1 && tiles > cus) pl.copy_columns = kCopyColumnsSmall;   // (one tile per CU at most: no difference)
    const unsigned least = fold_sub_elems(n == 1 ? pl.copy_columns : fold_columns(n, pl.all, fold_tile(pl)));
    unsigned tile = least;
    while (!pl.small && tile * 4 * (pl.n_load + n_store) < kFoldTicketBytes) tile += least;
    if (!words_inline(*h)) h->fold.fill_set(level_set(0), tile);
    if (h->tile_override) tile = h->tile_override;
    pl.tile_elems = tile;
    pl.grid_shift = 0;
    pl.n_items = fold_levels(h->fold.flows, tile, 0, !words_inline(*h), &h->fold.levels);
}

blink_status_t make_plan(blink_schedule* h) {
    LaunchPlan& pl = h->plan;
    if (pl.made) return BLINK_OK;
    if (h->n_cu == 0) {
        int dev = -1, n_cu = 0;
        BLINK_HIP(hipGetDevice(&dev));
        BLINK_HIP(hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev));
        if (n_cu < 1) return BLINK_EHIP;
        h->n_cu = n_cu;
    }
    const Served served = served_by(h->s, h->fold.fits, h->must_wait());
    if (served == Served::kNot) return BLINK_EINVAL;
    pl.fold = served == Served::kFold;
    if (pl.fold)
        plan_fold(h);
    else
        plan_hand_over(h);
    pl.own = layout_of(h->s, served, false);
    pl.shared = layout_of(h->s, served, true);
    pl.made = true;
    return BLINK_OK;
}

}  // namespace

// Forget all progress and the status record, and let the next call plan its
// launch afresh (used when the tile size changes: counters of earlier calls were
// counted in other units; and to recover after a wait was abandoned).  Waits for
// the device first.
blink_status_t reset_progress(blink_schedule* h) {
    h->epoch = 0;
    for (uint64_t& b : h->ticket_base) b = 0;
    h->tables_stale = true;
    h->plan = LaunchPlan();
    h->call_skipped = false;
    h->static_record = false;
    h->occupancy[0] = h->occupancy[1] = 0;
    forget_trial(h);
    if (h->device < 0) return BLINK_OK;
    BLINK_HIP(hipDeviceSynchronize());
    if (!h->d_block) return BLINK_OK;
    // the next call's counters and tables go in with it (see upload); the status record is read before
    BLINK_HIP(hipMemset(h->d_block, 0, kHeadBytes));
    BLINK_HIP(hipDeviceSynchronize());
    return BLINK_OK;
}

// Wait for the device, then report what the status record of the block says.
blink_status_t read_status(blink_schedule* h, blink_progress_t* out) {
    *out = blink_progress_t{};
    out->stage = out->awaited_stage = -1;
    const void* block = h->d_block;
    if (h->last_static_device >= 0) {  // the latest call ran on a static block: report on that one
        int dev = -1;
        BLINK_HIP(hipGetDevice(&dev));
        std::lock_guard<std::mutex> lock(g_static_mutex);
        // no record of this schedule's: its latest call kept none or a reset has dropped it, or the
        // block has passed to another schedule or to tables for the other kernel
        if (!h->static_record || dev != h->last_static_device) return BLINK_OK;
        const StaticBlock& sb = g_static[dev];
        if (sb.owner != h->id || sb.fold != h->plan.fold) return BLINK_OK;
        block = sb.ptr;
    } else if (h->device < 0) {
        return BLINK_OK;  // never ran: nothing can have gone wrong
    }
    unsigned long long rec[kStatusWords] = {};
    BLINK_HIP(hipDeviceSynchronize());
    if (!block) return BLINK_OK;  // no stage waits for another, no ticket is drawn: nothing can have gone wrong
    BLINK_HIP(hipMemcpy(rec, block, sizeof rec, hipMemcpyDeviceToHost));
    out->state = static_cast<int32_t>(rec[kStatusState]);
    if (rec[kStatusState] == 0) return BLINK_OK;
    out->stage = static_cast<int32_t>(rec[kStatusStage]);
    out->awaited_stage = static_cast<int32_t>(rec[kStatusAwaited]);
    out->seen = rec[kStatusSeen];
    out->wanted = rec[kStatusWanted];
    out->call = rec[kStatusCall];
    return BLINK_ESTUCK;
}

// Calls with less traffic are too short to time against one another.  (On all 256 CUs a payload
// that does not get a workgroup for every tile moves more; on a part of them it need not.)
constexpr uint64_t kTrialMinBytes = 64ull << 20;

namespace {
// The pair of events around a timed call; index < 0: the call is not timed.
struct Timed {
    int cls = 0, index = -1;
};

void drop_trial_events(blink_schedule* h) {
    for (auto& per_class : h->trial_event)
        for (void*& e : per_class) {
            if (e) (void)hipEventDestroy(static_cast<hipEvent_t>(e));
            e = nullptr;
        }
}
hipEvent_t trial_event(const blink_schedule* h, Timed t, int which) {
    return static_cast<hipEvent_t>(h->trial_event[t.cls][2 * t.index + which]);
}

// No more timed calls: `way` serves from now on.
int pick(blink_schedule* h, int way) {
    drop_trial_events(h);
    h->trial.picked = way;
    return way;
}

// How this call is served (1, 2 or 3, see way_trial.hpp); *timed: the events to put around
// it.  can_front, can_turns: the schedule has ways 2, 3.
// A caller who asks for way 2 gets it for sums only, as the interface says; picked by
// the trial it serves every operator.
int choose_way(blink_schedule* h, bool static_block, blink_dtype_t dtype, bool sum, bool can_front, bool can_turns, Timed* timed) {
    if (h->kernel_choice == 2) return can_front && sum ? 2 : 1;
    if (h->kernel_choice == 3) return can_turns ? 3 : 1;
    if (h->kernel_choice) return 1;
    if (h->trial.picked) return h->trial.picked;
    const Ways ways = ways_of(can_front, can_turns);
    // no trial: one way only / nothing may be created here / too short
    if (ways.count == 1 || static_block || h->s.traffic_bytes < kTrialMinBytes) return 1;
    const int cls = trial_class(sum, dtype == BLINK_FP32);
    const int n = ways.count * kTrialSamples;
    if (const int way = timed_way(h->trial, ways, cls)) {
        for (int e = 0; e < 2 * n; ++e) {
            if (h->trial_event[cls][e]) continue;
            hipEvent_t ev = nullptr;
            if (hipEventCreate(&ev) != hipSuccess) {
                (void)hipGetLastError();
                return pick(h, 1);
            }
            h->trial_event[cls][e] = ev;
        }
        *timed = {cls, h->trial.calls[cls]};
        return way;
    }
    // All of this class's timed calls are launched: wait for the last of them (once per
    // schedule) and compare.
    float ms[kMostWays * kTrialSamples] = {};
    bool ok = hipEventSynchronize(trial_event(h, {cls, n - 1}, 1)) == hipSuccess;
    for (int c = 0; ok && c < n; ++c)
        ok = hipEventElapsedTime(&ms[c], trial_event(h, {cls, c}, 0), trial_event(h, {cls, c}, 1)) == hipSuccess;
    if (!ok) (void)hipGetLastError();
    return pick(h, ok ? fastest_way(ways, ms) : can_front ? 2 : 1);
}
}  // namespace

// Forget the picked way and the times so far: later calls are timed afresh.
void forget_trial(blink_schedule* h) {
    drop_trial_events(h);
    h->trial = WayTrial();
}

void release_device_state(blink_schedule* h) {
    drop_trial_events(h);
    if (h->d_block) (void)hipFree(h->d_block);
    h->d_block = nullptr;
    h->block_bytes = 0;
    h->device = -1;
}

namespace {

// One launch on `stream`.  Its own status decides whether the call counts: an error
// some earlier HIP call of this thread left behind is not this launch's, and a
// launch that failed must not consume a call number or move the ticket bases
// (the next call would wait for tiles that nobody ever counted).  timed: the events to
// record around it.
blink_status_t launch(blink_schedule* h, const void* fn, dim3 grid, unsigned threads, void* params, hipStream_t stream,
                      Timed timed) {
    if (timed.index >= 0 && hipEventRecord(trial_event(h, timed, 0), stream) != hipSuccess) {
        (void)hipGetLastError();  // e.g. a capturing stream: give the trial up
        pick(h, 1);
        timed = Timed();
    }
    void* args[] = {params};
    const hipError_t launched = hipLaunchKernel(fn, grid, dim3(threads), args, 0, stream);
    if (launched != hipSuccess) {
        std::fprintf(stderr, "blink: kernel launch failed: %s\n", hipGetErrorString(launched));
        (void)hipGetLastError();  // the failed launch's error is reported here, not left for later calls
        return BLINK_EHIP;
    }
    if (timed.index >= 0) {
        if (hipEventRecord(trial_event(h, timed, 1), stream) == hipSuccess) {
            h->trial.calls[timed.cls] += 1;
        } else {
            (void)hipGetLastError();
            pick(h, 1);
        }
    }
    h->last_grid = grid.x * grid.y;
    return BLINK_OK;
}

// Clears the head of the static block before a call on it.
blink_status_t launch_clear(char* block, size_t bytes, hipStream_t stream) {
    unsigned long long* words = reinterpret_cast<unsigned long long*>(block);
    unsigned long long n_words = bytes / sizeof(unsigned long long);
    void* args[] = {&words, &n_words};
    const unsigned grid = static_cast<unsigned>(std::min<unsigned long long>((n_words + 255) / 256, 1024));
    const hipError_t cleared = hipLaunchKernel(reinterpret_cast<const void*>(blink_clear), dim3(grid), dim3(256), args, 0, stream);
    if (cleared != hipSuccess) {
        std::fprintf(stderr, "blink: kernel launch failed: %s\n", hipGetErrorString(cleared));
        (void)hipGetLastError();
        return BLINK_EHIP;
    }
    return BLINK_OK;
}

FoldFn pick_fold(blink_dtype_t dtype, bool sum, const LaunchPlan& pl, int policy) {
    const int n = static_cast<int>(pl.n_load);
    const bool stream = policy == kFoldStream;
    const FoldTile tile = fold_tile(pl);
    if (n == 1) return fold_copy(policy, pl.copy_columns);
    if (pl.mid) return dtype == BLINK_FP32 ? fold_f32_mid(n, pl.all, tile, sum) : fold_i32_mid(n, pl.all, tile, sum);
    if (dtype == BLINK_FP32) return sum ? fold_f32_sum(n, pl.all, tile, stream) : fold_f32_other(n, pl.all, tile);
    return sum ? fold_i32_sum(n, pl.all, tile, stream) : fold_i32_other(n, pl.all, tile);
}

// A call on the fold kernel for a workgroup per tile.
blink_status_t run_once(blink_schedule* h, void* const* bufs, blink_dtype_t dtype, blink_redop_t redop, hipStream_t stream,
                        uint32_t grid_shift) {
    LaunchPlan& pl = h->plan;
    const std::vector<FoldFlow>& flows = h->fold.once;
    const int n = static_cast<int>(pl.n_load);
    if (pl.once_shift != grid_shift) {
        const int columns = n == 1 ? once_copy_columns(pl.once_stores) : fold_columns(n, pl.all, pl.once_half && pl.all ? FoldTile::kHalf : FoldTile::kWhole);
        pl.once_grid = once_grid(flows, fold_sub_elems(columns), grid_shift, static_cast<uint32_t>(h->n_cu));
        pl.once_shift = grid_shift;
    }
    const OnceGrid& g = pl.once_grid;
    const bool many = flows.size() > kOnceFewFlows;
    const bool fp32 = dtype == BLINK_FP32, sum = redop == BLINK_SUM;
    const OnceKernel kernel = n == 1   ? once_copy(h->s.k, pl.once_stores, many)
                              : pl.mid ? (fp32 ? once_f32_mid : once_i32_mid)(n, pl.all, pl.once_half, many, sum)
                              : sum    ? (fp32 ? once_f32_sum : once_i32_sum)(n, pl.all, pl.once_half, many)
                                       : (fp32 ? once_f32_other : once_i32_other)(n, pl.all, pl.once_half, many);
    if (!kernel.fn) return BLINK_EINVAL;
    if (!pl.once_filled) {
        kernel.fill(flows, pl.once_params);   // the same for all element types and operators
        pl.once_filled = true;
    }
    alignas(16) unsigned char params[kOnceParamsBytes];
    std::memcpy(params, pl.once_params, kernel.call_at);
    void** const buf = reinterpret_cast<void**>(params);
    for (int i = 0; i < kernel.bufs; ++i) buf[i] = bufs[std::min(i, h->s.k - 1)];
    const uint32_t call = once_call(g.tile_elems, grid_shift, static_cast<uint32_t>(redop), g.tiles);
    std::memcpy(params + kernel.call_at, &call, sizeof call);
    return launch(h, kernel.fn, dim3(g.columns, static_cast<unsigned>(flows.size())), kFoldThreads, params, stream, Timed());
}

// A call on the fold kernel.  block: the static block, or null for the schedule's own, which is only made where tickets are drawn or the tables
// do not travel with the launch.
blink_status_t run_fold(blink_schedule* h, void* const* bufs, blink_dtype_t dtype, blink_redop_t redop, hipStream_t stream,
                        const BlockLayout& l, char* block) {
    const Schedule& s = h->s;
    LaunchPlan& pl = h->plan;
    const bool static_block = block != nullptr;
    // Rank buffers that all start the same distance past a 1 KiB boundary (views
    // into larger buffers, allocations at 512-byte granularity): the tile grid
    // is moved down by that distance, so that tiles, and with them the 1 KiB
    // accesses of a wave, start on such boundaries in memory.
    uint32_t grid_shift = 0;
    const uintptr_t past = reinterpret_cast<uintptr_t>(bufs[0]) & 1023u;
    bool common = true;
    for (int i = 1; i < s.k; ++i) common = common && (reinterpret_cast<uintptr_t>(bufs[i]) & 1023u) == past;
    if (common) grid_shift = static_cast<uint32_t>(past / 4);
    const FoldTables& t = h->fold;
    if (pl.once && once_call_serves(pl.small, s.has_deps, h->wg_per_cu, h->kernel_choice, h->sweep_alternates)) {
        if (static_block) h->static_record = false;
        if (blink_status_t st = run_once(h, bufs, dtype, redop, stream, grid_shift)) return st;
        h->last_kernel = 1;
        h->handed_over = 0;
        if (!static_block) h->epoch += 1;
        return BLINK_OK;
    }
    if (words_inline(*h) && grid_shift != pl.grid_shift) {
        pl.n_items = fold_levels(t.flows, pl.tile_elems, grid_shift, false, &h->fold.levels);
        pl.grid_shift = grid_shift;
    }

    const bool sum = redop == BLINK_SUM;
    const bool by_tile = pl.n_load <= 8 && t.flows.size() <= 64;
    Timed timed;
    // Programs with dependencies have way 1 only.  Way 2 is offered up to four accumulators, as the
    // interface says; the kernel has no such limit, and what it gives deeper stages was not measured.
    const bool choice = !pl.small && !s.has_deps;
    const int way = choose_way(h, static_block, dtype, sum, choice && s.max_stack <= 4, choice && by_tile && t.flows.size() > 1, &timed);
    const uint64_t chunk_tiles = std::max<uint64_t>(1, s.chunk / pl.tile_elems);
    const uint32_t chunk_turn = static_cast<uint32_t>(std::min<uint64_t>(chunk_tiles, kTurnPayload));

    const uint64_t payload_bytes = static_cast<uint64_t>(s.k) * s.n * 4;
    const uint32_t n_store = s.fused[0].stage.n_store;
    const FoldPolicy policy = fold_policy(pl.n_load, n_store, payload_bytes, pl.kernel_bytes, s.has_deps, way, h->sweep_alternates);
    const FoldFn fn = pick_fold(dtype, sum, pl, policy);
    if (!fn) return BLINK_EINVAL;

    // Workgroups: all tiles of a small payload; otherwise 7 on 8 CUs (see fold.hpp), one on each where one
    // rank is written (Reduce of 8 ranks, 64 MiB, with 224 / 256 workgroups 84.5 / 83 us, of 4 48 / 46).  Copies
    // have few loads per workgroup and n_store times that of stores in flight: one workgroup on each CU
    // where one, two, five or six ranks are written, 7 on 8 CUs where three, four, seven or eight are, 6 on 8
    // with more; and one on eight CUs more than that from seven ranks and four times the memory-side cache on (us with
    // 192 / 224 / 256 workgroups: Gather of 3 ranks, 400 MiB, - / 89 / 90; Broadcast to 2, 400 MiB, 197 /
    // 192 / 190; to 3, 300 MiB, 195 / 193 / 194; to 5, 85 MiB, 72 / 70 / 70, 200 MiB, 207 / 192 / 190; to 15,
    // 64 MiB 148 / 155 / -, 150 MiB 424 / 408 / -; to 7 by payload in times the cache, two - / 72.0 (AllGather 72.3) / 72.1
    // (73.3), three - / 125.8 (127.8) / 123.8 (125.9), four and a half - / 184 (185) / 180 (180), six - / 262 / 255,
    // nine - / 396 / 389, sixteen - / 653 / 642: to seven ranks the line could lie a little lower).
    const uint64_t cus = static_cast<uint64_t>(h->n_cu);
    const bool copy_many = pl.n_load == 1 && n_store > 6;
    const uint64_t eighths = pl.n_load > 1 ? (pl.all ? 7 : 8)
                             : copy_many   ? (n_store > 8 ? 6 : 7) + (payload_bytes > 4 * kMemorySideCacheBytes ? 1 : 0)
                             : n_store == 3 || n_store == 4 ? 7 : 8;
    uint64_t most = pl.small ? pl.n_items : cus * eighths / 8;
    if (h->wg_per_cu > 0) most = h->wg_per_cu * cus;
    const auto [grid, dealt, two] = fold_grid(most, pl.n_items, pl.small, 4ull * pl.tile_elems * (pl.n_load + n_store));

    if (static_block) {
        h->static_record = !dealt;
        if (!dealt)
            if (blink_status_t st = launch_clear(block, l.done, stream)) return st;
    } else if (!dealt || !words_inline(*h)) {
        if (blink_status_t st = upload(h, l)) return st;
        block = static_cast<char*>(h->d_block);
    }
    FoldParams p;   // every field that is read is set
    for (int i = 0; i < BLINK_MAX_RANKS; ++i) p.buf[i] = i < s.k ? bufs[i] : nullptr;
    const unsigned* const tables = reinterpret_cast<const unsigned*>(block + l.words);
    p.words = words_inline(*h) ? nullptr : tables;
    p.levels = levels_inline(*h) ? nullptr : reinterpret_cast<const FoldLevel*>(tables + t.level_word(level_set(h->tile_override)));
    if (!p.words) fold_words(t.flows, kInlineFlows, p.inline_words);
    if (!p.levels) std::copy(t.levels.begin(), t.levels.end(), p.inline_levels);
    p.ticket = block ? reinterpret_cast<unsigned long long*>(block + l.ticket) : nullptr;
    for (int c = 0; c < 2; ++c) p.ticket_base[c] = static_block ? 0 : h->ticket_base[c];
    p.n_items = static_cast<unsigned>(pl.n_items);
    p.n_flows = static_cast<unsigned>(t.flows.size());
    p.n_levels = static_cast<unsigned>(t.levels.size());
    // Programs with dependencies go through one tree's share after the other: with partial sums
    // written on the way the trees' turns cost up to a tenth (per node, us on the same buffers,
    // one front / turns: 8 ranks x 8 MiB 26.1 / 24.0, 20 MiB 60.8 / 62.3, 64 MiB 175 / 192, 128 MiB
    // 351 / 388, 256 MiB 738 / 735; 6 ranks x 98 MiB 200 / 216).
    // Way 1 gives a tree 128 KiB of every rank at a turn: HBM serves a stretch like that best in one go
    // (8 ranks, us in turns of a tile / 64 / 128 / 256 KiB, on one set of buffers: 230 MiB 663 / 658 / 642 / 646,
    // 256 MiB 675 / 671 / 658 / 668, on another 729 / 724 / 707 / 734, 400 MiB 1127 / 1116 / 1094 / 1098; of a tile / 128 KiB,
    // 7 ranks x 200 MiB 478 / 476, 6 x 98 MiB 201 / 196, 5 x 98 MiB 161 / 162, x 300 MiB 504 / 522, 4 x 98 MiB 130 / 130,
    // 4 x 300 MiB 405 / 410, 3 x 98 MiB 95 / 95, AllGather 8 x 64 MiB 74 / 75, 8 x 256 MiB 455 / 418, Broadcast 333 / 333:
    // it helps where there are many trees, and what it costs to five ranks and less a schedule's timed choice avoids).
    const uint32_t run_turn = pl.small ? 1u : std::max(1u, kFoldRunElems / pl.tile_elems);
    p.turn = way == 2 || s.has_deps ? kTurnPayload : (way == 3 || !by_tile) ? chunk_turn : run_turn;
    p.tile_elems = pl.tile_elems;
    p.grid_shift = grid_shift;
    p.redop = static_cast<unsigned>(redop);
    // Calls sweep the payload in alternating directions (the second, fourth, ... call
    // backwards), unless switched off.
    p.reverse = !s.has_deps && !static_block && h->sweep_alternates && (h->epoch & 1) != 0;
    p.dealt = dealt;
    p.two = two;
    p.width = two ? grid / 2 : grid;
    p.call = static_block ? 1 : static_cast<unsigned>(h->epoch + 1);
    if (blink_status_t st = launch(h, reinterpret_cast<const void*>(fn), dim3(grid), kFoldThreads, &p, stream, timed)) return st;
    h->last_kernel = way;
    h->handed_over = 0;
    if (static_block) return BLINK_OK;
    h->epoch += 1;
    if (!dealt)   // every ticket is followed by one draw
        for (uint32_t c = 0; c < (two ? 2u : 1u); ++c) h->ticket_base[c] += fold_share(p.n_items, c, two);
    return BLINK_OK;
}

// A call whose stages wait for one another.
blink_status_t run_hand_over(blink_schedule* h, void* const* bufs, blink_dtype_t dtype, blink_redop_t redop, hipStream_t stream,
                             const BlockLayout& l, char* block) {
    const Schedule& s = h->s;
    const LaunchPlan& pl = h->plan;
    const bool static_block = block != nullptr;
    if (!static_block) {
        if (blink_status_t st = upload(h, l)) return st;
        block = static_cast<char*>(h->d_block);
    }
    KernelFn fn = pick_kernel(dtype);
    int& occ = h->occupancy[dtype == BLINK_FP32];
    if (occ == 0) {
        BLINK_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, fn, kLanes, 0));
        if (occ < 1) {
            occ = 0;
            return BLINK_EHIP;
        }
    }
    // Waves per CU: 3 (some always wait), with more than 8 ranks, whose programs have more
    // stages that can run at a time, 4.  Per-edge AllReduce, us with 2 / 3 / 4: 8 ranks x
    // 64 MiB in 1 MiB chunks 337 / 345 / 368, in 64 KiB chunks 342 / 325 / 331, in 16 KiB
    // chunks 420 / 342 / 328; 16 ranks, one-hop trees, 64 MiB - / 694 / 670.
    const int per_cu = std::min(occ, h->wg_per_cu > 0 ? h->wg_per_cu : (s.k > 8 ? 4 : 3));
    unsigned long long max_grid = static_cast<unsigned long long>(per_cu) * h->n_cu;
    const unsigned long long n_items = pl.n_items;
    // no more waves than three time slots' worth of tickets can be busy
    max_grid = std::min(max_grid, std::max<unsigned long long>(64, 3 * (n_items / s.n_slots + 1)));
    const unsigned long long grid = std::min<unsigned long long>(max_grid, n_items);

    KParams p{};
    for (int i = 0; i < s.k; ++i) p.buf[i] = bufs[i];
    p.tmpl = reinterpret_cast<const StageTmpl*>(block + l.tmpl);
    p.inst = reinterpret_cast<const StageInst*>(block + l.inst);
    p.done = reinterpret_cast<unsigned long long*>(block + l.done);
    p.ticket = reinterpret_cast<unsigned long long*>(block + l.ticket);
    p.status = reinterpret_cast<unsigned long long*>(block);
    p.wait_ticks = (h->wait_limit_us ? h->wait_limit_us : kDefaultWaitMicroseconds) * kTicksPerMicrosecond;
    const unsigned n_queues = static_cast<unsigned>(std::min<unsigned long long>(kQueuesHandOver, grid));
    p.n_queues = n_queues;
    // A static block is shared by every schedule used on the GPU and keeps the
    // last call's contents: each call on it starts from cleared counters, as
    // call number 1.  The schedule's own block counts on from call to call.
    for (unsigned q = 0; q < n_queues; ++q) p.ticket_base[q] = static_block ? 0 : h->ticket_base[q];
    p.n_items = n_items;
    p.epoch = static_block ? 1 : h->epoch + 1;
    p.tiles_per_chunk = pl.tiles_per_chunk;
    p.tile_shift = pl.tile_shift;
    p.redop = static_cast<unsigned>(redop);
    p.n_inst = static_cast<unsigned>(s.inst.size());
    p.pieces = l.pieces;
    p.max_naps = 4;   // looks at a dependency back off to ~0.8 us apart

    if (static_block) {
        h->static_record = true;
        if (blink_status_t st = launch_clear(block, l.counters_end, stream)) return st;
    }
    if (blink_status_t st = launch(h, reinterpret_cast<const void*>(fn), dim3(static_cast<unsigned>(grid)), kLanes, &p, stream, Timed())) return st;
    h->last_kernel = 1;
    h->handed_over = 1;
    if (static_block) return BLINK_OK;
    h->epoch += 1;
    // queue q holds the tickets q, q + n_queues, ...; every wave draws exactly one
    // ticket past the end of every queue
    for (unsigned q = 0; q < n_queues; ++q) h->ticket_base[q] += (n_items + n_queues - 1 - q) / n_queues + grid;
    return BLINK_OK;
}

}  // namespace

blink_status_t execute(blink_schedule* h, void* const* bufs, int k, size_t n, blink_dtype_t dtype,
                       blink_op_t op, blink_redop_t redop, void* stream, bool static_block) {
    if (!h || !bufs) return BLINK_EINVAL;
    if (dtype != BLINK_FP32 && dtype != BLINK_INT32) return BLINK_EINVAL;
    if (redop != BLINK_SUM && redop != BLINK_PROD && redop != BLINK_MIN && redop != BLINK_MAX) return BLINK_EINVAL;
    const Schedule& s = h->s;
    if (k != s.k || n != s.n || op != s.op) return BLINK_EMISMATCH;
    if (n == 0) return BLINK_OK;  // nothing to move: the buffer pointers are not looked at
    for (int i = 0; i < k; ++i) {
        if (!bufs[i] || (reinterpret_cast<uintptr_t>(bufs[i]) & 15u)) return BLINK_EINVAL;
        for (int j = 0; j < i; ++j) {
            const char* a = static_cast<const char*>(bufs[i]);
            const char* b = static_cast<const char*>(bufs[j]);
            if (a < b + n * 4 && b < a + n * 4) return BLINK_EINVAL;
        }
    }
    if (s.inst.empty()) return BLINK_OK;
    if (blink_status_t st = make_plan(h)) return st;
    const BlockLayout& l = static_block ? h->plan.shared : h->plan.own;
    char* block = nullptr;   // the static block, or null: the schedule's own
    if (static_block) {
        if (blink_status_t st = claim_static_block(h, l, static_cast<hipStream_t>(stream), &block)) return st;
    } else {
        // A launch carries the call's number on its schedule and the place its
        // ticket counters have reached; replayed from a HIP graph it would carry
        // them again and find the counters elsewhere: waves would draw nothing
        // and stages would not wait.  Say so instead of recording such a launch.
        hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(static_cast<hipStream_t>(stream), &capture) != hipSuccess) {
            (void)hipGetLastError();  // not this call's business: the launch will report a bad stream
        } else if (capture != hipStreamCaptureStatusNone) {
            std::fprintf(stderr, "blink: the stream is capturing; only blink_allreduce_noalloc can be recorded into a HIP graph\n");
            return BLINK_EINVAL;
        }
        if (blink_status_t st = bind_device(h)) return st;
        h->last_static_device = -1;
    }
    return h->plan.fold ? run_fold(h, bufs, dtype, redop, static_cast<hipStream_t>(stream), l, block)
                        : run_hand_over(h, bufs, dtype, redop, static_cast<hipStream_t>(stream), l, block);
}

}  // namespace blink
