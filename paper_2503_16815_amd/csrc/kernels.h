// Internal interface between the C ABI (api.hip) and the kernel files.
// Nothing here is visible to users of include/deft_knapsack.h.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <functional>

#include "../../include/deft_knapsack.h"

namespace deft {

// Arguments of one solve call as the kernels see them (all device pointers).
struct BatchArgs {
    int32_t mode;  // DEFT_MODE_*
    int32_t batch, item_stride, knap_stride;
    int32_t max_capacity, max_c1, max_c2;  // create-time limits (per-instance LIMIT status)
    const int32_t *n_items, *n_knapsacks, *weights, *values, *capacities, *fill_order;
    const int32_t *drop_time;  // recursive mode only
    int64_t *total_value;
    int32_t *knap_value, *knap_load, *assignment, *status;
    // [batch] or null.  The bit-set kernels write 1 for an instance whose values are not all its
    // weights and leave it alone, 0 for one they answered; the LDS-row kernels then skip those.  The
    // enumeration ahead of rows in global memory does the same for the streamed sweep.
    int32_t *left;
};

// ---- sequential mode, capacity row resident in LDS (seq_lds.hip) ------------
// One instance is owned by `threads` lanes (64 = one wavefront, several
// instances per workgroup; otherwise one workgroup).  Each lane keeps
// `cells_per_thread` row cells in registers.
struct SeqLdsPlan {
    int32_t variant;           // index into the compiled (threads, cells_per_thread) table
    int32_t threads;           // T
    int32_t cells_per_thread;  // K
    int32_t keep_words;        // 32-bit keep words per lane and item: ceil(K / 32)
    int32_t guard_cells;       // cells below the row: 8 scratch words, then INT_MIN
    int32_t row_cells;         // LDS row length (multiple of 64, covers max_capacity)
    int32_t n_pad;             // entries per offered-item list (multiple of 8, >= max_items)
    int32_t lds_bytes;         // dynamic LDS per workgroup
    int32_t wg_threads;        // workgroup size
    int32_t inst_per_wg;       // instances per workgroup
    int32_t wg_per_cu;         // co-resident workgroups: the runtime's answer, capped by LDS granules
    int64_t keep_words_per_inst;  // max_items * keep_words * T
    int64_t keep_bytes;        // keep table of the whole batch
    int64_t scratch_bytes;     // keep table + one offered-item list per instance and stage
};

// Picks the variant for the limits; returns false when no LDS variant fits.
bool seq_lds_plan(int32_t max_capacity, int32_t max_items, int32_t max_knapsacks, int32_t max_batch,
                  int32_t lds_per_wg_bytes, SeqLdsPlan *plan);
// Sets the kernel's dynamic-LDS attribute and queries occupancy.
hipError_t seq_lds_prepare(SeqLdsPlan *plan);
// `swept_cells` (device, may be null): every stage adds the cell-updates its sweep evaluated.
hipError_t seq_lds_launch(const SeqLdsPlan &plan, const BatchArgs &args, void *scratch,
                          hipStream_t stream, unsigned long long *swept_cells);
// Its kernels that try a stage by enumeration first (seq_lds_pool.hip); seq_lds_prepare and seq_lds_launch see to them.
hipError_t seq_lds_pool_prepare(const SeqLdsPlan &plan);
hipError_t seq_lds_pool_launch(const SeqLdsPlan &plan, const BatchArgs &args, void *scratch,
                               hipStream_t stream, unsigned long long *swept_cells);
// Algorithm 1 (recursive mode) under the same plan and scratch (seq_lds_rec.hip).
hipError_t seq_lds_rec_prepare(const SeqLdsPlan &plan);
hipError_t seq_lds_rec_launch(const SeqLdsPlan &plan, const BatchArgs &args, void *scratch,
                              hipStream_t stream, unsigned long long *swept_cells);

// Arguments of one simulation call as the kernels see them (all device pointers).
struct ScheduleArgs {
    int32_t batch, n_buckets, iterations, max_capacity;
    const int32_t *comm_time, *drop_time, *forward_time, *backward_time;
    int32_t *stage_case, *stage_count, *stage_time, *update_k, *tail, *status;
};

// ---- sequential layout, value = weight, one bit per cell (seq_bits_kernel.h) -----
// One wavefront per instance; the reachable sums as a bit set in registers and LDS, the
// selection from a bit-sliced "first item that reached this sum" table in registers.  No scratch.
struct SeqBitsPlan {
    int32_t variant;         // index into the compiled (words per lane, planes) table; it, planes and n_pad are those of
                             // the longest lists: a launch takes those of the call's
    int32_t words_per_lane;  // K: capacities up to 2048 K - 1
    int32_t planes;          // NP: lists of up to 2^NP items
    int32_t row_words;       // 64 x the slots max_capacity needs
    int32_t n_pad;           // entries of the stage's item list in LDS
    int32_t lds_limit;       // most dynamic LDS a workgroup may ask for
    int32_t lds_bytes;       // what one instance on its own takes
    int32_t compute_units;
};
bool seq_bits_plan(int32_t max_capacity, int32_t max_items, int32_t lds_per_wg_bytes, int32_t compute_units, SeqBitsPlan *plan);
hipError_t seq_bits_prepare(const SeqBitsPlan &plan);
// DEFT_MODE_SEQUENTIAL, DEFT_MODE_RECURSIVE and DEFT_MODE_CAPACITY_SWEEP.
// `swept_cells` (device, may be null): every stage that is swept adds the cell-updates this evaluates, to one of
// kBitsCounters counters a cache line apart (all to one: 16384 instances of 38 items 0.06 -> 0.21 ms).
constexpr int kBitsCounters = 64, kBitsCounterStride = 16;
hipError_t seq_bits_launch(const SeqBitsPlan &plan, const BatchArgs &args, hipStream_t stream, unsigned long long *swept_cells);
// The two task queues over several iterations (schedule_sim.hip has them for rows in global memory), one launch.
hipError_t seq_bits_queues_launch(const SeqBitsPlan &plan, const ScheduleArgs &args, hipStream_t stream, unsigned long long *swept_cells);
// The kernels that other translation units compile: of the longer rows, of the task queues, and of both.
const void *seq_bits_long_kernel(int variant, bool queues);
const void *seq_bits_queues_kernel(int variant);
const void *seq_bits_long_queues_kernel(int variant);

// ---- sequential mode by enumeration, ahead of rows in global memory (seq_enum.hip) ----------
// Answers the instances it can (args.left 0) and flags the others (1).  No scratch.
hipError_t seq_enum_prepare();
hipError_t seq_enum_launch(const BatchArgs &args, int32_t compute_units, hipStream_t stream);

// ---- per-call HIP-event timing (profile.hip) ---------------------------------
class Profiler {
public:
    void reset() { ncall_ = nsweep_ = 0; failed_ = counted_ = false; }
    bool begin(hipStream_t st);        // start of a profiled call
    void sweep_begin(hipStream_t st);  // brackets one launch of the DP sweep kernel
    void sweep_end(hipStream_t st);
    void end(hipStream_t st);
    void counted(hipStream_t st);      // behind what counts a profiled call's cells
    // waits for the last recorded call, sums every call since reset(), resets
    deft_status_t read(deft_knapsack_profile_t *out);
    void destroy();

private:
    struct Pool {
        hipEvent_t *ev = nullptr;
        int cap = 0;
        hipEvent_t get(int i);  // event i, created on demand; nullptr on failure
        void destroy();
    };
    void record(Pool &p, int idx, hipStream_t st);
    Pool call_, sweep_, count_;
    int ncall_ = 0, nsweep_ = 0;  // events used (two per call / per launch)
    bool failed_ = false, counted_ = false;
};

// Adds to `cells` (device) what the job's sweeps go through, or would, of the instances of a call that the bit-set
// kernels answered (profile.hip).
hipError_t bits_count_launch(const BatchArgs &args, hipStream_t stream, unsigned long long *cells);

// ---- sequential mode, rows in global memory (seq_global.hip) -------------------
// For capacities whose row does not fit LDS: the row streams through LDS rings, several items per
// pass, one workgroup per instance, which idle compute units help where instances are few (Algorithm 1:
// one launch per item, rows in two buffers).
struct SeqGlobalPlan {
    int32_t threads, cells_per_thread;  // of the launch per item
    int32_t row_len;           // int32 cells per row buffer (multiple of the tile)
    int32_t keep_words;        // 64-bit keep words per item
    int32_t max_items, max_batch;
    int32_t ring_cells;        // streamed sweep: cells of its rings in LDS
    int32_t lds_bytes;         // its dynamic LDS
    int32_t compute_units;
    int64_t scratch_bytes;     // rows + keep + item lists + per-instance state
};
void seq_global_plan(int32_t max_capacity, int32_t max_items, int32_t max_batch, int32_t lds_per_wg_bytes,
                     int32_t compute_units, SeqGlobalPlan *plan);
// Sets the kernels' dynamic-LDS attribute and clears what calls expect cleared in the scratch.
hipError_t seq_global_prepare(const SeqGlobalPlan &plan, void *scratch);
// `streamed_cells` (device, may be null): the streamed sweep adds the row cells it reads and writes.
hipError_t seq_global_launch(const SeqGlobalPlan &plan, const BatchArgs &args, void *scratch,
                             hipStream_t stream, Profiler *prof, unsigned long long *streamed_cells);

// ---- joint two-link mode, table in global memory (joint2.hip) -----------------
struct JointPlan {
    int32_t pitch;             // int32 cells per table row (multiple of 64)
    int32_t rows;              // max_c1 + 1
    int32_t lds_pitch;         // int32 cells per LDS row: max_c2 + 1
    int32_t ring_rows;         // old rows resident in LDS
    int32_t lds_bytes;         // dynamic LDS of the sweep kernel
    int32_t max_items, max_batch;
    int64_t scratch_bytes;
};
void joint_plan(int32_t max_c1, int32_t max_c2, int32_t max_items, int32_t max_batch, int32_t lds_per_wg_bytes,
                JointPlan *plan);
hipError_t joint_prepare(const JointPlan &plan, void *scratch);
// `swept_cells` (device, may be null): every instance that is answered from its table adds the table's cells, an item.
hipError_t joint_launch(const JointPlan &plan, const BatchArgs &args, void *scratch, hipStream_t stream,
                        Profiler *prof, unsigned long long *swept_cells);

// ---- the two task queues over several iterations (schedule_sim.hip) -------------
// Bytes of the handle-owned buffers (queue state and the per-stage solver problem).
int64_t schedule_sim_bytes(int32_t max_batch, int32_t max_items);
// Enqueues the whole simulation: per stage a set-up kernel, the solver (`solve` enqueues one
// batch in args.mode = DEFT_MODE_SEQUENTIAL or DEFT_MODE_RECURSIVE on the handle's path), a
// kernel that applies the answer.
hipError_t schedule_sim_launch(const ScheduleArgs &args, void *sim_buffers, hipStream_t stream,
                               const std::function<hipError_t(const BatchArgs &)> &solve);

// ---- the paper's greedy heuristic (greedy.hip) ----------------------------------
// No scratch memory.  per_link: the two-link weight layout.
hipError_t greedy_prepare(int32_t max_items);
hipError_t greedy_launch(const BatchArgs &args, bool per_link, hipStream_t stream);

}  // namespace deft
