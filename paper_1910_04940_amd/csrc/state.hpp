// The schedule handle: host-side schedule, the launch plan derived from it, and
// the device-side block (status record, progress counters, tables) the kernel uses.
#pragma once
#include <cstddef>
#include <cstdint>

#include "fold_plan.hpp"
#include "way_trial.hpp"

namespace blink {

// Layout of the device block of a schedule, in bytes from its start:
//   status record (kStatusWords 64-bit words), ticket counters, a counter of
//   finished tiles per stage instance, or per piece of it (counters kCounterStride words apart),
//   stage templates, stage instances.  The fold kernel counts no finished tiles and
//   knows neither templates nor instances: its
//   tables, where they do not travel in the kernel's arguments, lie where the counters
//   of finished tiles would (they need 204 of every 256 bytes there).
struct BlockLayout {
    size_t ticket = 0, done = 0, tmpl = 0, inst = 0, bytes = 0;
    uint32_t pieces = 1;      // counters per stage instance (see counters_per_stage)
    size_t counters_end = 0;  // status record and counters are [0, counters_end)
    size_t words = 0;         // FoldTables::tables
};

// What a launch needs besides the schedule itself.  It depends only on the
// schedule, the device and the caller's overrides, so it is worked out once, at
// the first call, and kept until an override changes (the progress counters
// count tiles, so the tile size may not change while they hold progress).
struct LaunchPlan {
    bool made = false;
    unsigned tile_elems = 0;       // elements per tile (ticket)
    BlockLayout own, shared;       // of the schedule's own block and of a device's static one
    // stages that wait for one another (kernel.hpp)
    unsigned tile_shift = 0;       // log2 of tile_elems
    uint32_t tiles_per_chunk = 1;  // most tiles any stage instance has
    uint64_t n_items = 0;          // tickets per call
    // what the fold kernel runs (fold.hpp)
    bool fold = false;
    bool small = false;            // a few tiles per CU: a workgroup for every one
    bool half = false;             // tiles of half the size (where small)
    bool once = false;             // served by the kernel that does nothing else (fold_once.hpp), see once_call_serves
    bool once_half = false;        // there: tiles of half the size
    int once_stores = 0;           // copies there: the most ranks a flow is copied to
    OnceGrid once_grid{};          // made for once_shift
    uint32_t once_shift = ~0u;
    bool once_filled = false;
    alignas(16) unsigned char once_params[kOnceParamsBytes] = {};   // what of them all calls share
    bool all = false;              // every stage writes all the ranks it reads
    bool mid = false;              // partial sums are written on the way
    uint32_t n_load = 0;           // ranks a stage reads
    int copy_columns = 0;          // where it reads one: columns per wave
    uint64_t kernel_bytes = 0;     // read and written per call (fold_bytes)
    uint32_t grid_shift = 0;       // the tile grid the levels were made for
};

}  // namespace blink

struct blink_schedule {
    blink::Schedule s;
    blink::FoldTables fold;       // of s; the levels, and the last of the sets, belong to the plan
    blink::LaunchPlan plan;
    int device = -1;              // HIP device the schedule has run on; -1 = none yet
    void* d_block = nullptr;      // its block there (see BlockLayout); null = not needed so far
    size_t block_bytes = 0;       // of that block
    bool tables_stale = true;     // the block's tables are not those of the plan
    uint64_t id = 0;              // names, with the kernel the tables are for, the owner of a device's static block
    uint64_t epoch = 0;           // calls made so far on d_block; its counters hold epoch * tiles
    uint64_t ticket_base[16] = {};  // value of each ticket counter when the next call starts
    bool call_skipped = false;    // blink_schedule_test_skip_call was used: stages wait for one another
    bool hand_over = false;       // so does the caller want it (blink_schedule_set_hand_over)
    int handed_over = -1;         // whether the latest call's stages waited; -1 = none yet
    bool must_wait() const { return call_skipped || hand_over; }
    uint64_t wait_limit_us = 0;   // longest wait for another stage; 0 = default
    int n_cu = 0;
    int wg_per_cu = 0;            // launch override (0 = automatic)
    unsigned tile_override = 0;   // elements per tile requested by the caller (0 = automatic)
    int occupancy[2] = {};        // waves per CU of the kernel in use, per dtype (schedules with dependencies)
    unsigned last_grid = 0;
    int last_kernel = 0;          // the way the latest call ran (see choose_way), 0 = none yet
    int last_static_device = -1;  // device whose static block the latest call used; -1 = it used d_block
    bool static_record = false;   // that call cleared the block's status record and may have set it; no reset since
    int kernel_choice = 0;        // the caller's wish: 0 = pick the fastest way, else one of the three
    bool sweep_alternates = true; // calls on a schedule without dependencies walk the tiles in alternating directions
    blink::WayTrial trial;        // the timed calls so far and the pick
    void* trial_event[blink::kTrialClasses][2 * blink::kMostWays * blink::kTrialSamples] = {};   // hipEvent_t pairs around them
};

namespace blink {
// static_block: run on the device's file-scope block instead of the schedule's own.
blink_status_t execute(blink_schedule* h, void* const* bufs, int k, size_t n, blink_dtype_t dtype,
                       blink_op_t op, blink_redop_t redop, void* stream, bool static_block = false);
uint64_t next_schedule_id();
blink_status_t reset_progress(blink_schedule* h);
void forget_trial(blink_schedule* h);
blink_status_t read_status(blink_schedule* h, blink_progress_t* out);
void release_device_state(blink_schedule* h);
}  // namespace blink
