// Sequential multiple-knapsack solve for capacities whose row does not fit LDS
// (Sec. III.B, Problem 1 per window): the row lives in global memory.
//
// The streamed sweep (sg_stream; the sequential mode, for the instances that the enumeration ahead of it leaves, and
// the capacity sweep): one launch, one workgroup per instance for all stages, lists and walks included.
//
// What is kept of a cell is how far it falls short: D[c] = (value of the items so far) - row[c], so
//   D'[c] = min(D[c] + v, D[c - w]),   item taken where D[c - w] < D[c] + v,   D[c < 0] = infinity.
// Every cell at or above the weight of the items so far holds all of them: D = 0 there, in no need of
// being stored or computed, and its keep bit is known to be set.  And a walk that starts at C has at
// most the items behind q to lower it: cells of the row after item q below C - (their weight) are
// never looked at.  What is swept of a row is the band between the two, at most the smaller of C and
// (weight offered) - C wide: on the GPT-2 shape 30 % of the cells up to C.
//
// The band streams through LDS in ascending blocks of R cells, and a pass over it serves up to
// seven consecutive items.  Level l (item q + l) has a ring in LDS with the row before its item, long
// enough to reach w cells back; at step t it computes block t - l from its ring into level l + 1's, the
// last level stores to global memory, in place, behind the loads, and one wavefront keeps the loads
// of level 0 two or three blocks ahead.  The levels work on different blocks, so one barrier per step
// is all the ordering there is, and a step is one task of 512 cells for each of up to fifteen
// wavefronts.  The shifted operand of an item of at least a block's weight lies in blocks that were
// complete a step ago: it is read one step ahead, while the step's own cells are computed.  A cell-update
// costs 8 / levels + 1/8 bytes of global traffic, 12 bytes of LDS, four vector instructions and a share
// of about thirty vector and forty scalar instructions per task.
// Measured on the GPT-2 shape (256 instances, C = 381000, one window swept): 2.34 ms; one persistent workgroup per instance over all cells up to C, three items per pass,
// and launches of their own for lists and walks took 11.5 ms, one launch per item 3.55 ms.  What bounds
// it: a step is read, compute, write, barrier for all wavefronts at once (counters: vector units busy 41 % of
// the cycles, LDS 39 %, a wavefront waiting 52 % of its own).
//
// Teams.  A batch of at most half as many instances as there are compute units, on long rows (kTeamRows), is
// launched with helpers: workgroups behind the batch's own, as many per instance as fill the chip.
// An instance's own workgroup (the owner) runs everything above; where that is expected to be quicker
// (kTeamJobNs and its like) it cuts the next item's band into tiles instead, every workgroup of the team
// takes some, both operands straight from global memory, from one row buffer into the other, and the owner
// waits for the tiles that helpers took.  Nobody waits for a workgroup that has not begun: a tile is
// asked for by whoever is there (the owner would do them all), an owner waits only for helpers that are at a
// tile, and a helper waits only for an owner that has begun, else it leaves after a few
// milliseconds.  So no order or number of workgroups on the chip, another team's included, can hold one up.
// The helpers hold their compute units until the owner dismisses them: before its last walk, or when a
// list shows that no band worth a job is left (kTeamMinBand).
// Row cells go out as device-scope stores, which leave nothing in an XCD's L2 for the release to write
// back (2000000 cells, 4 instances of 148 items: 3.06 ms, with plain stores 3.56); counters
// are striped (see TeamStripe; one instance of that: 2.24 ms, one counter for all 3.40).
// Measured, 148 items in two windows, lists twice the first window: one instance of 381000 cells 1.38 ms,
// alone 3.68, a launch per item over all compute units 3.26; 2000000 cells 2.42, 34.5 and 3.63 ms; sixteen of
// 381000 cells 2.37, 3.82 and 4.17 ms.  A call with nothing to sweep pays 3 to 5 us for its helpers.
//
// Algorithm 1 reads a cell of every intermediate row, so it takes sweeps that leave each of them in
// global memory: one launch per offered-item rank, two row buffers, the row cut into tiles over
// many workgroups (sg_sweep), keep bits by wavefront ballots.
#include <limits.h>

#include "instance_check.h"

namespace deft {

namespace {

constexpr int kMaxItemsPlaced = 4096;  // longest item list (create-time limit)

constexpr int kThreads = 256;
constexpr int kIter = 32;                       // 64-cell groups per wavefront
constexpr int kWaveCells = 64 * kIter;          // 2048
constexpr int kTileCells = kWaveCells * (kThreads / 64);

// per-instance state kept between launches
struct InstState {
    int32_t status, n_act, knap, cap;
    // Algorithm 1: the best level met so far (its value, the length of its list, its remaining time)
    int32_t best_value, best_length, best_remain;
};

// One offered item of the streamed sweep.
struct alignas(8) StreamItem {
    int32_t w, v;
    int64_t upto;  // weight of the stage's list up to and with this item
    int32_t index, pad;
};

// What the workgroups of a team tell each other (see the head of this file).  Every access is an atomic one
// of the whole device.  A team of some size has kTeamStripes counters of each kind, a cache line to itself,
// with every kTeamStripes-th tile and workgroup: 255 workgroups at one address wait 20 ns for each other.
constexpr int kTeamStripes = 8;
struct alignas(128) TeamStripe {
    // 0: the owner has not begun.  Else the tiles of the job in the upper half (none: there is no job)
    // and how often a tile was asked for in the lower; kTeamOver: there will be no more jobs.
    unsigned long long ticket;
    uint32_t done;  // tiles that helpers have finished, all jobs
    uint32_t gone;  // workgroups that have left the team
};
struct alignas(128) TeamJob {
    TeamStripe stripe[kTeamStripes];
    uint32_t word[8];  // the job: w, v, low, top, top_in, q, buffer read, tasks per wavefront and tile
    uint32_t gone;     // stripes whose workgroups have all left; the last one leaves all at 0 for the next call
};

struct Scratch {
    int32_t *rows;      // [batch][2][row_len]
    uint64_t *keep;     // [batch][max_items][keep_words]
    int32_t *act;       // [batch][max_items]
    int32_t *probe;     // [batch][max_items]  Algorithm 1: remaining time of the level that ends before entry q
    InstState *state;   // [batch]
    StreamItem *items;  // [batch][max_items]  the streamed sweep's lists
    TeamJob *jobs;      // [batch]  the streamed sweep's teams
};

__host__ __device__ inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

Scratch carve(const SeqGlobalPlan &p, void *base, int32_t max_batch)
{
    char *c = static_cast<char *>(base);
    Scratch s;
    s.rows = reinterpret_cast<int32_t *>(c);
    c += align256((size_t)max_batch * 2 * p.row_len * 4);
    s.keep = reinterpret_cast<uint64_t *>(c);
    c += align256((size_t)max_batch * p.max_items * p.keep_words * 8);
    s.act = reinterpret_cast<int32_t *>(c);
    c += align256((size_t)max_batch * p.max_items * 4);
    s.probe = reinterpret_cast<int32_t *>(c);
    c += align256((size_t)max_batch * p.max_items * 4);
    s.state = reinterpret_cast<InstState *>(c);
    c += align256((size_t)max_batch * sizeof(InstState));
    s.items = reinterpret_cast<StreamItem *>(c);
    c += align256((size_t)max_batch * p.max_items * sizeof(StreamItem));
    s.jobs = reinterpret_cast<TeamJob *>(c);
    return s;
}

__global__ void __launch_bounds__(kThreads) sg_init(BatchArgs a, InstState *state)
{
    const int inst = blockIdx.x;
    const int status = check_instance(a, inst, false);
    clear_outputs(a, inst, status);
    if (threadIdx.x == 0) {
        state[inst].status = status;
        state[inst].n_act = 0;
    }
}

// Algorithm 1 (one stage): the whole list is offered in its order, and entry q gets the
// remaining time of the level that ends before it, R - sum of drop_time over the entries
// from q on (-1 if negative), from a suffix sum taken 64 entries at a time from the end.
__global__ void __launch_bounds__(64) sg_levels_setup(BatchArgs a, InstState *state, int32_t *act, int32_t *probe,
                                                      int max_items)
{
    const int inst = blockIdx.x, lane = threadIdx.x;
    InstState *st = &state[inst];
    if (st->status != DEFT_OK) {
        if (lane == 0) st->n_act = 0, st->knap = -1;
        return;
    }
    const int n = a.n_items[inst];
    const int C = a.capacities[(size_t)inst * a.knap_stride];
    const int32_t *drop = a.drop_time + (size_t)inst * a.item_stride;
    long long behind = 0;
    for (int i0 = (n - 1) & ~63; i0 >= 0 && n > 0; i0 -= 64) {
        const int i = i0 + lane;
        long long x = i < n ? drop[i] : 0;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const long long y = __shfl_down(x, off);
            if (lane + off < 64) x += y;
        }
        if (i < n) {
            const long long left = (long long)C - (x + behind);
            act[(size_t)inst * max_items + i] = i;
            probe[(size_t)inst * max_items + i] = left < 0 ? -1 : (int)left;
        }
        behind += __shfl(x, 0);
    }
    if (lane == 0) {
        st->n_act = n; st->knap = 0; st->cap = C;
        st->best_value = 0; st->best_length = 0; st->best_remain = 0;
    }
}

// Offered item q of every instance: one pass over the row.
__global__ void __launch_bounds__(kThreads)
sg_sweep(BatchArgs a, int q, InstState *state, const int32_t *__restrict__ act, const int32_t *__restrict__ probe,
         int32_t *rows, uint64_t *keep, int row_len, int keep_words, int max_items, int tiles)
{
    const int inst = blockIdx.x / tiles, tile = blockIdx.x % tiles;
    const InstState st = state[inst];
    if (q >= st.n_act) return;
    const int C = st.cap;
    if (tile == 0 && threadIdx.x == 0 && q > 0) {
        // Algorithm 1: the row before item q is the row of the level that ends here; a
        // shallower level replaces the best one only when strictly greater.  (Nobody else
        // touches the instance's best level during this launch; before the first item the
        // row is all zero and cannot win.)
        const int at = probe[(size_t)inst * max_items + q];
        if (at >= 0) {
            const int level_value = rows[((size_t)inst * 2 + (q & 1)) * row_len + at];
            if (level_value > st.best_value) {
                state[inst].best_value = level_value;
                state[inst].best_length = q;
                state[inst].best_remain = at;
            }
        }
    }
    const int lane = threadIdx.x & 63;
    const int wave_base = (tile * (kThreads / 64) + (threadIdx.x >> 6)) * kWaveCells;
    if (wave_base > C) return;
    const int t = act[(size_t)inst * max_items + q];
    const int w = a.weights[(size_t)inst * a.item_stride + t];
    const int v = a.values[(size_t)inst * a.item_stride + t];
    const int32_t *__restrict__ src = rows + ((size_t)inst * 2 + (q & 1)) * row_len;
    int32_t *__restrict__ dst = rows + ((size_t)inst * 2 + ((q & 1) ^ 1)) * row_len;
    uint64_t *kw = keep + ((size_t)inst * max_items + t) * keep_words + wave_base / 64;
    const bool first = q == 0;

    unsigned long long mine = 0;
#pragma unroll 8
    for (int i = 0; i < kIter; ++i) {
        const int c = wave_base + i * 64 + lane;
        const int own = first ? 0 : src[c];
        int cand = INT_MIN;
        if (c >= w) cand = (first ? 0 : src[c - w]) + v;
        const bool take = cand > own;
        dst[c] = take ? cand : own;
        const unsigned long long mask = __ballot(take);
        if (lane == i) mine = mask;
    }
    if (lane < kIter) kw[lane] = mine;
}

// Algorithm 1: one thread per instance walks the keep words back from the best level's last item and
// remaining time.
__global__ void __launch_bounds__(64)
sg_traceback(BatchArgs a, InstState *state, const int32_t *__restrict__ act, const int32_t *rows,
             const uint64_t *keep, int row_len, int keep_words, int max_items)
{
    const int inst = blockIdx.x * 64 + threadIdx.x;
    if (inst >= a.batch) return;
    InstState *st = &state[inst];
    if (st->status != DEFT_OK || st->knap < 0) return;
    const int nact = st->n_act, C = st->cap, j = st->knap;
    const int32_t *W = a.weights + (size_t)inst * a.item_stride;
    const int32_t *list = act + (size_t)inst * max_items;
    int value = 0;
    if (nact > 0) value = rows[((size_t)inst * 2 + (nact & 1)) * row_len + C];
    // the whole list is the last level met
    if (value > st->best_value) { st->best_value = value; st->best_length = nact; st->best_remain = C; }
    value = st->best_value;
    const int length = st->best_length, start = st->best_remain;
    int c = start;
    for (int q = length - 1; q >= 0; --q) {
        const int t = list[q];
        const int w = W[t];
        if (w <= c) {
            const uint64_t word = keep[((size_t)inst * max_items + t) * keep_words + (c >> 6)];
            if ((word >> (c & 63)) & 1ull) {
                a.assignment[(size_t)inst * a.item_stride + t] = j;
                c -= w;
            }
        }
    }
    a.knap_value[(size_t)inst * a.knap_stride + j] = value;
    a.knap_load[(size_t)inst * a.knap_stride + j] = start - c;
    // slot 1 reports the level: items left off the list, its remaining time
    a.knap_value[(size_t)inst * a.knap_stride + 1] = a.n_items[inst] - length;
    a.knap_load[(size_t)inst * a.knap_stride + 1] = value > 0 ? start : 0;
    a.total_value[inst] = value;
}

// ---- the streamed sweep -----------------------------------------------------------------

constexpr int kStreamThreads = 1024;  // one workgroup per instance, all stages
constexpr int kStreamWaves = kStreamThreads / 64;  // the last one moves old cells from global memory into LDS
constexpr int kTaskCells = 512;       // what a wavefront computes at a time: eight cells per lane
constexpr int kTaskSlots = kTaskCells / 64;
constexpr int kMaxLevels = 7;         // items per pass over the row
// Teams: a job is cut into tiles of one task per wavefront.
constexpr int kTeamCells = kStreamWaves * kTaskCells;
// Which launches get helpers: rows of kTeamRows cells, or of kTeamRowsHeavy and kTeamCellsPerItem cells per item
// listed (heavy items, for which a team does most).  The host cannot see how wide a band will be; what decides is that
// a call whose bands are too narrow for a team loses 4 to 7 us to the larger kernel.  One window, then two fifths of
// it, lists 1.2 and 1.7 times the first (narrow and wide), 1 to 64 instances, gain by the team: 140000 cells
// and 20 items 0.98-1.05 and 1.10-1.39, 24 items 0.96-1.03 and 1.08-1.23; 160000 and 12 1.08-1.18 and 1.34-1.61, 24
// 0.97 and 1.12-1.43, 60 0.98 and 1.01-1.18; 200000 and 24 1.03-1.13 and 1.20-1.63, 60 0.98 and 1.05-1.44; 300000 and
// 60 1.02-1.13 and 1.18-2.1, 148 0.995-1.01 and 1.00-1.72.  On 80000 cells 0.9 and 1.1 with 12 items.
constexpr int kTeamRows = 1 << 18, kTeamRowsHeavy = 1 << 17, kTeamCellsPerItem = 7000;
// The narrowest band in which the estimate below can favour the team: where passes serve seven items, and where
// items are so heavy that a pass serves one (lists of more than kTeamHeavy on average are taken for such).
// 160000 cells with 33000 of band: 148 items gain nothing, 12 go from 141 to 121 us.
constexpr int kTeamMinBand = 60000, kTeamMinBandHeavy = 9500, kTeamHeavy = 4000;
constexpr int kTeamStartPolls = 1 << 12;     // how often a helper looks for an owner that has not begun
constexpr unsigned long long kTeamOver = 1ull << 63;
// What is expected, in ns, of a job (besides its tiles), of a task of every wavefront of the team, of a step of
// a pass and of a step of an item too heavy for the rings.  All items by the team or none (148 items, two
// windows, lists twice the first window): one instance of 160000 cells 1.52 and 1.58 ms, by this
// estimate 1.25; 64 of them 3.13 and 1.70, so 1.67; one of 381000 1.72 and 3.67, so 1.33.
constexpr int kTeamJobNs = 5000, kTeamTileNs = 2500, kStepNs = 780, kHeavyStepNs = 1400;
constexpr int kMiscBytes = 1024;      // LDS in front of the rings: StreamShared and the placed-item bits

typedef __attribute__((address_space(3))) int32_t lds_i32;
typedef const __attribute__((address_space(1))) int32_t global_ci32;

struct StreamShared {
    int32_t cnt, knap, cap, cap_min;
    int64_t weight;            // of the whole list
    int32_t value;             // of the whole list
    int32_t settled;
    unsigned long long ticket;  // of the team's job
    int32_t job[8], stripe, team;
    uint32_t placed[kMaxItemsPlaced / 32];
};
static_assert(sizeof(StreamShared) <= kMiscBytes, "fits in front of the rings");

// How a pass is cut: `levels` items over blocks of `block` cells, `ahead` blocks of the old row in flight.
struct PassShape {
    int16_t levels, block, ahead;
};
// Fifteen computing wavefronts, block / 512 tasks per level and step: the shapes that keep most of them
// busy.  A cell costs 8 / levels bytes of global traffic, which is what bounds a pass of few
// items, so more levels come before larger blocks; the rings limit both.
constexpr PassShape kShapes[] = {{7, 1024, 3}, {6, 1024, 3}, {5, 1536, 2}, {5, 1024, 3}, {4, 1536, 2}, {4, 1024, 3},
                                 {3, 2560, 2}, {3, 1024, 3}, {2, 3584, 2}, {2, 1024, 3}, {1, 7680, 2}, {1, 2560, 2},
                                 {1, 1024, 3}};
constexpr int kNumShapes = sizeof(kShapes) / sizeof(kShapes[0]);

// Block hand-over: the loading wavefront arrives when the block that the next step reads has landed,
// a computing one when its LDS accesses have (the ones for its next step included: what they read may be
// overwritten behind the barrier); its stores stay in flight until the end of the pass.
// Asm, because the compiler puts a wait for all vector memory in front of every barrier it
// knows of once a kernel has LDS-direct loads.
__device__ __forceinline__ void step_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
// Waits until at most n of the wavefront's loads are in flight (n is one of the counts the shapes give).
__device__ __forceinline__ void wait_loads(int n)
{
    switch (n) {
    case 4: asm volatile("s_waitcnt vmcnt(4)" ::: "memory"); break;
    case 6: asm volatile("s_waitcnt vmcnt(6)" ::: "memory"); break;
    case 8: asm volatile("s_waitcnt vmcnt(8)" ::: "memory"); break;
    case 10: asm volatile("s_waitcnt vmcnt(10)" ::: "memory"); break;
    case 14: asm volatile("s_waitcnt vmcnt(14)" ::: "memory"); break;
    case 30: asm volatile("s_waitcnt vmcnt(30)" ::: "memory"); break;
    default: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
    }
}

// acc = 2 acc + (sh < own): compare into vcc, add-with-carry.
__device__ __forceinline__ uint32_t shift_in_less(uint32_t acc, int sh, int own)
{
    uint32_t out;
    asm("v_cmp_lt_i32 vcc, %2, %3\n\tv_addc_co_u32 %0, vcc, %1, %1, vcc" : "=v"(out) : "v"(acc), "v"(sh), "v"(own) : "vcc");
    return out;
}

__device__ __forceinline__ StreamItem load_item(const StreamItem *e)
{
    // written earlier in the launch by another wavefront of the workgroup (same compute unit, same L1)
    StreamItem it;
    const unsigned long long *u = reinterpret_cast<const unsigned long long *>(e);
    const unsigned long long a = __hip_atomic_load(u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    it.upto = (int64_t)__hip_atomic_load(u + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    const unsigned long long c = __hip_atomic_load(u + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    it.w = (int)(uint32_t)a;
    it.v = (int)(uint32_t)(a >> 32);
    it.index = (int)(uint32_t)c;
    it.pad = 0;
    return it;
}

// The keep bit of (item q of the list, cell c): byte (c / 512) * 64 + c % 64 of the item's row, bit
// 7 - (c / 64) % 8.
__device__ __forceinline__ size_t keep_byte(int c) { return ((size_t)(c >> 9) << 6) + (c & 63); }

// What a computing wavefront does in one pass: one task of one level per step.
struct StreamTask {
    int w, v;          // the level's item
    int len, len_out;  // lengths of the ring read and of the ring written
    int32_t *rg;       // the ring read
    int32_t *rg_out;   // the ring written (not the last level)
    int32_t *row;      // the row (last level)
    uint8_t *keep;     // the item's keep row, this lane's byte
    int low, top;      // cells of the level's row outside these do not matter
    int c, at;         // the task's first cell at the level's first step, and its place in the rings
    int first;         // the level's first step
};
// AHEAD: the item weighs at least a block, so that the next step's shifted operand is complete when this
// step begins and is read then; it has arrived by the step's barrier.  (Read behind the stores instead: 2.39 ms
// on the GPT-2 shape, 2.30 so.)  LAST: the level stores to the row.
// Why a ring is long enough: while block b is computed from it, cells from b R - w (AHEAD: (b + 1) R - w,
// at most b R) are read, and block b + 1 is written, up to cell (b + 2) R (level 0: up to
// (b + 1 + ahead) R).  That is w + 2 R cells and, AHEAD, w + R (level 0: ahead - 1 blocks more).
// (AHEAD reads the operand of a level's first block beside that of its second; it lies below the band.)
template <bool AHEAD, bool LAST>
__device__ __forceinline__ void stream_task(const StreamTask &k, int R, int steps, int lane)
{
    int p = k.at, po = k.at, c0 = k.c;
    int shd[kTaskSlots], nxt[kTaskSlots];
    auto read_shifted = [&](int at, int (&to)[kTaskSlots]) {
        int from = at - k.w;
        if (from < 0) from += k.len;
        if (from + kTaskCells <= k.len) {
            const int32_t *s = k.rg + from + lane;
#pragma unroll
            for (int x = 0; x < kTaskSlots; ++x) to[x] = s[x * 64];
        } else {
#pragma unroll
            for (int x = 0; x < kTaskSlots; ++x) {
                const unsigned o = (unsigned)(from + lane + x * 64);
                to[x] = k.rg[min(o, o - (unsigned)k.len)];  // wraps past the ring's end
            }
        }
    };
    step_barrier();
    for (int t = 0; t < k.first; ++t) step_barrier();
    if (AHEAD) read_shifted(p, shd);
    for (int t = k.first; t < steps; ++t) {
        const bool here = c0 <= k.top && c0 + kTaskCells > k.low;
        int own[kTaskSlots];
        if (here) {
            const int32_t *s = k.rg + p + lane;
#pragma unroll
            for (int x = 0; x < kTaskSlots; ++x) own[x] = s[x * 64];
            if (!AHEAD) read_shifted(p, shd);
        }
        p += R;
        if (p >= k.len) p -= k.len;
        if (AHEAD) read_shifted(p, nxt);
        if (here) {
            if (c0 < k.w) {
#pragma unroll
                for (int x = 0; x < kTaskSlots; ++x)
                    if (c0 + x * 64 + lane < k.w) shd[x] = INT_MAX;
            }
            uint32_t bits = 0;
            int32_t *o = (LAST ? k.row + c0 : k.rg_out + po) + lane;
#pragma unroll
            for (int x = 0; x < kTaskSlots; ++x) {
                const int passed = (int)((uint32_t)own[x] + (uint32_t)k.v);
                bits = shift_in_less(bits, shd[x], passed);
                o[x * 64] = min(passed, shd[x]);
            }
            k.keep[(size_t)(c0 >> 9) << 6] = (uint8_t)bits;
        }
        c0 += R;
        po += R;
        if (po >= k.len_out) po -= k.len_out;
        step_barrier();
        if (AHEAD) {
#pragma unroll
            for (int x = 0; x < kTaskSlots; ++x) shd[x] = nxt[x];
        }
    }
}

// ---- teams ----
template <class T>
__device__ __forceinline__ T team_load(const T *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <class T>
__device__ __forceinline__ void team_store(T *p, T x) { __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// One item's cells of the task at c0, both operands from global memory: `src` holds the row before
// the item up to cell top_in, all cells above it are 0.
template <bool SHARED = false>
__device__ __forceinline__ void row_task(const int32_t *src, int32_t *dst, uint8_t *keep, int c0, int w, int v, int top_in, int lane)
{
    int own[kTaskSlots], shd[kTaskSlots];
#pragma unroll
    for (int k = 0; k < kTaskSlots; ++k) {
        const int c = c0 + k * 64 + lane;
        own[k] = c <= top_in ? src[c] : 0;
        shd[k] = c < w ? INT_MAX : c - w <= top_in ? src[c - w] : 0;
    }
    uint32_t bits = 0;
#pragma unroll
    for (int k = 0; k < kTaskSlots; ++k) {
        const int passed = (int)((uint32_t)own[k] + (uint32_t)v);
        bits = shift_in_less(bits, shd[k], passed);
        if (SHARED) team_store(&dst[c0 + k * 64 + lane], min(passed, shd[k]));
        else dst[c0 + k * 64 + lane] = min(passed, shd[k]);
    }
    keep[keep_byte(c0) + lane] = (uint8_t)bits;
}

__device__ __forceinline__ uint32_t team_count(uint32_t *p)
{
    return __hip_atomic_fetch_add(p, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long team_ask(TeamStripe *s)
{
    return __hip_atomic_fetch_add(&s->ticket, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// (of helpers + 1 workgroups, the owner being number 0)
__device__ __forceinline__ int team_stripes(int helpers) { return helpers >= 4 * kTeamStripes ? kTeamStripes : 1; }
// How many of 0 .. n - 1 are stripe s's.
__device__ __forceinline__ int striped(int n, int s, int stripes) { return (n - s + stripes - 1) / stripes; }
__device__ __forceinline__ uint32_t ticket_tiles(unsigned long long t) { return (uint32_t)(t >> 32); }
__device__ __forceinline__ uint32_t ticket_number(unsigned long long t) { return (uint32_t)t; }

// Tile `tile` of a job, by the whole workgroup; returns when its stores have been made.
__device__ __forceinline__ void team_tile(int32_t *buffers, int row_len, uint8_t *kp, size_t keep_row, const int32_t *job, int tile,
                                          int wave, int lane)
{
    int j[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) j[i] = __builtin_amdgcn_readfirstlane(job[i]);
    const int low = j[2], top = j[3], span = j[7];
    const int32_t *src = buffers + (size_t)j[6] * row_len;
    int32_t *dst = buffers + (size_t)(j[6] ^ 1) * row_len;
    int c0 = low / kTeamCells * kTeamCells + __builtin_amdgcn_readfirstlane(tile) * span * kTeamCells + wave * kTaskCells;
#pragma unroll 1
    for (int x = 0; x < span; ++x, c0 += kTeamCells)
        if (c0 <= top && c0 + kTaskCells > low) row_task<true>(src, dst, kp + (size_t)j[5] * keep_row, c0, j[0], j[1], j[4], lane);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
}

// Workgroup `number` will not look at the team's words again.
__device__ __forceinline__ void team_leave(TeamJob *job, int number, int helpers)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (what it has said itself)
    const int stripes = team_stripes(helpers), s = number % stripes;
    if (team_count(&job->stripe[s].gone) + 1 != (uint32_t)striped(helpers + 1, s, stripes)) return;
    if (team_count(&job->gone) + 1 != (uint32_t)stripes) return;
    for (int i = 0; i < stripes; ++i) {
        team_store(&job->stripe[i].ticket, 0ull);
        team_store(&job->stripe[i].done, 0u);
        team_store(&job->stripe[i].gone, 0u);
    }
    team_store(&job->gone, 0u);
}

// A helper: takes tiles of the instance's jobs until there are no more, or leaves if the instance's owner
// does not begin.
__device__ __forceinline__ void team_help(StreamShared *sh, TeamJob *job, int number, int helpers, int32_t *buffers, int row_len,
                                          uint8_t *kp, size_t keep_row, int wave, int lane)
{
    const int stripes = team_stripes(helpers), s = number % stripes;
    TeamStripe *mine = &job->stripe[s];
    while (true) {
        if (wave == 0) {
            unsigned long long t = kTeamOver;
            if (lane == 0) {
                for (int polls = 0; polls < kTeamStartPolls;) {
                    t = team_load(&mine->ticket);
                    if (t == 0) ++polls;
                    if (t >> 63) break;
                    // (the first of a stripe for its first tile, and so on; the others would only stand in the way)
                    if (ticket_number(t) < ticket_tiles(t) && (uint32_t)(number / stripes) < ticket_tiles(t)) {
                        t = team_ask(mine);
                        if (t >> 63 || ticket_number(t) < ticket_tiles(t)) break;
                    }
                    __builtin_amdgcn_s_sleep(2);
                    t = kTeamOver;
                }
                sh->ticket = t;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            if (lane < 8) sh->job[lane] = (int)team_load(&job->word[lane]);
        }
        __syncthreads();
        const unsigned long long t = sh->ticket;
        if (t >> 63) {
            if (threadIdx.x == 0) team_leave(job, number, helpers);
            return;
        }
        team_tile(buffers, row_len, kp, keep_row, sh->job, (int)ticket_number(t) * stripes + s, wave, lane);
        if (threadIdx.x == 0) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            team_count(&mine->done);
        }
    }
}

// The owner says the same to every stripe.
__device__ __forceinline__ void team_tell(TeamJob *job, int helpers, unsigned long long ticket)
{
    if ((int)threadIdx.x < team_stripes(helpers)) team_store(&job->stripe[threadIdx.x].ticket, ticket);
}

// The owner: one item as a job of `tiles` tiles.  `done`, lane x of the first wavefront: the tiles of
// stripe x that helpers took, all jobs.
__device__ __forceinline__ void team_lead(StreamShared *sh, TeamJob *job, int helpers, const int (&words)[8], int tiles, uint32_t &done,
                                          int32_t *buffers, int row_len, uint8_t *kp, size_t keep_row, int wave, int lane)
{
    const int stripes = team_stripes(helpers);
    const bool counts = wave == 0 && lane < stripes;
    if (wave == 0) {
        if (lane == 0) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                sh->job[i] = words[i];
                team_store(&job->word[i], (uint32_t)words[i]);
            }
        }
        // (the row as the workgroup has left it, too: a barrier lies behind the stores)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        if (counts) {
            const int part = striped(tiles, lane, stripes);
            team_store(&job->stripe[lane].ticket, (unsigned long long)part << 32 | (part > 0 ? 0u : 1u));
            done += part;
        }
    }
    // The first tile, then whatever no helper has asked for.
    int s = 0;
    while (s >= 0) {
        if (threadIdx.x == 0) sh->ticket = team_ask(&job->stripe[s]);
        __syncthreads();
        const unsigned long long t = sh->ticket;
        if (ticket_number(t) < ticket_tiles(t)) {
            if (wave == 0 && lane == s) --done;
            team_tile(buffers, row_len, kp, keep_row, sh->job, (int)ticket_number(t) * stripes + s, wave, lane);
        }
        if (wave == 0) {
            const unsigned long long left = counts ? team_load(&job->stripe[lane].ticket) : 0ull;
            const unsigned long long open = __ballot(counts && ticket_number(left) < ticket_tiles(left));
            if (lane == 0) sh->stripe = open ? __builtin_ctzll(open) : -1;
        }
        __syncthreads();
        s = sh->stripe;
    }
    if (wave == 0) {
        while (__ballot(counts && team_load(&job->stripe[lane].done) != done) != 0ull) __builtin_amdgcn_s_sleep(1);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    __syncthreads();
}

// All stages of one instance (see the head of this file), with the `helpers` workgroups of each instance behind the batch's own.
template <bool TEAMS>
__global__ void __launch_bounds__(kStreamThreads)
sg_stream(BatchArgs a, StreamItem *lists, int32_t *rows, uint8_t *keep, TeamJob *jobs, int helpers, int row_len, int max_items,
          int ring_cells, unsigned long long *streamed_cells)
{
    extern __shared__ __align__(16) char lds_stream[];
    StreamShared *sh = reinterpret_cast<StreamShared *>(lds_stream);
    int32_t *ring = reinterpret_cast<int32_t *>(lds_stream + kMiscBytes);
    const int inst = TEAMS ? blockIdx.x % a.batch : blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int32_t *buffers = rows + (size_t)inst * 2 * row_len;
    uint8_t *kp = keep + (size_t)inst * max_items * (row_len / 8);
    const size_t keep_row = row_len / 8;
    TeamJob *job = jobs + inst;
    if (TEAMS && (int)blockIdx.x >= a.batch) {
        team_help(sh, job, blockIdx.x / a.batch, helpers, buffers, row_len, kp, keep_row, wave, lane);
        return;
    }
    const bool answered = a.left && a.left[inst] == 0;  // (by the enumeration)
    const int status = answered ? -1 : check_instance(a, inst, false);
    if (!answered) clear_outputs(a, inst, status);
    // (may be said twice; the owner leaves at the very end)
    auto dismiss = [&]() {
        if (TEAMS) team_tell(job, helpers, kTeamOver);
    };
    if (status != DEFT_OK) {
        dismiss();
        if (TEAMS && tid == 0) team_leave(job, 0, helpers);
        return;
    }

    const int n = a.n_items[inst], m = a.n_knapsacks[inst];
    const int32_t *W = a.weights + (size_t)inst * a.item_stride;
    const int32_t *V = a.values + (size_t)inst * a.item_stride;
    const int32_t *cap = a.capacities + (size_t)inst * a.knap_stride;
    int32_t *out_asg = a.assignment + (size_t)inst * a.item_stride;
    int32_t *out_kv = a.knap_value + (size_t)inst * a.knap_stride;
    int32_t *out_kl = a.knap_load + (size_t)inst * a.knap_stride;
    StreamItem *list = lists + (size_t)inst * max_items;
    int cur = 0;  // the buffer that holds the row
    uint32_t done = 0;
    const bool caps_sweep = a.mode == DEFT_MODE_CAPACITY_SWEEP;
    for (int i = tid; i < kMaxItemsPlaced / 32; i += kStreamThreads) sh->placed[i] = 0;
    __syncthreads();

    long long total = 0;
    unsigned long long streamed = 0;
    const int stages = caps_sweep ? min(m, 1) : m;
    if (TEAMS) {
        if (tid == 0) sh->team = 1;
        team_tell(job, helpers, 1ull);  // (begun)
    }
    for (int s = 0; s < stages; ++s) {
        // ---- the stage's list, built by the first wavefront ------------------------------
        if (wave == 0) {
            const int j = caps_sweep ? 0 : a.fill_order ? a.fill_order[(size_t)inst * a.knap_stride + s] : s;
            int C = cap[j], C_min = C;
            if (caps_sweep)
                for (int x = 1; x < m; ++x) C = max(C, cap[x]), C_min = min(C_min, cap[x]);
            // offered: not placed, able to fit at all, worth something (an item of no value never
            // strictly improves a cell)
            int cnt = 0;
            long long weight = 0;
            int value = 0;
            for (int i0 = 0; i0 < n; i0 += 64) {
                const int i = i0 + lane;
                const int w = i < n ? W[i] : 0, v = i < n ? V[i] : 0;
                const bool f = i < n && !((sh->placed[i >> 5] >> (i & 31)) & 1u) && w <= C && v > 0;
                const unsigned long long mask = __ballot(f);
                long long upto = f ? w : 0;
                int vsum = f ? v : 0;
#pragma unroll
                for (int off = 1; off < 64; off <<= 1) {
                    const long long y = __shfl_up(upto, off);
                    if (lane >= off) upto += y;
                    vsum += __shfl_xor(vsum, off);
                }
                if (f) {
                    StreamItem e;
                    e.w = w; e.v = v; e.index = i; e.pad = 0;
                    e.upto = weight + upto;
                    list[cnt + __popcll(mask & ((1ull << lane) - 1ull))] = e;
                }
                cnt += __popcll(mask);
                weight += __shfl(upto, 63);
                value += vsum;
            }
            const bool settled = !caps_sweep && weight <= C;
            if (TEAMS && sh->team != 0) {
                // no band worth a job, now (at most weight - C_min wide) or later
                int widest = weight <= C_min ? 0 : (int)min((long long)C, weight - C_min);
                for (int x = s + 1; x < stages; ++x)
                    widest = max(widest, cap[a.fill_order ? a.fill_order[(size_t)inst * a.knap_stride + x] : x]);
                if (widest < (weight > (long long)cnt * kTeamHeavy ? kTeamMinBandHeavy : kTeamMinBand)) {
                    dismiss();
                    if (lane == 0) sh->team = 0;
                }
            }
            if (settled && cnt > 0) {
                // everything offered fits together: the DP takes it all
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                for (int p = lane; p < cnt; p += 64) {
                    const int i = load_item(list + p).index;
                    out_asg[i] = j;
                    atomicOr(&sh->placed[i >> 5], 1u << (i & 31));
                }
                if (lane == 0) {
                    out_kv[j] = value;
                    out_kl[j] = (int)weight;
                }
            }
            if (lane == 0) {
                sh->cnt = cnt; sh->knap = j; sh->cap = C; sh->cap_min = C_min;
                sh->weight = weight; sh->value = value; sh->settled = settled;
            }
        }
        __threadfence_block();
        __syncthreads();
        const int cnt = sh->cnt, j = sh->knap, C = sh->cap, C_min = sh->cap_min, value_all = sh->value;
        const long long weight_all = sh->weight;
        const bool team = TEAMS && __builtin_amdgcn_readfirstlane(sh->team) != 0;
        if (sh->settled || cnt == 0) {
            total += value_all;
            __syncthreads();
            continue;
        }

        // ---- the sweep -----------------------------------------------------------------
        // the cells of the row after the list's first p items that matter: upto = their weight
        auto top = [&](long long upto) { return (int)min((long long)C, upto); };
        auto bottom = [&](long long upto) { return (int)max(0ll, C_min - (weight_all - upto)); };
        long long before = 0;  // weight of the items gone through
        // (a capacity sweep whose every capacity holds the whole list has no band: the walks below never
        // meet a cell that is not known)
        for (int q = weight_all <= C_min ? cnt : 0; q < cnt;) {
            StreamItem it{};
            if (lane < kMaxLevels && q + lane < cnt) it = load_item(list + q + lane);
            const int room = (it.w + kTaskCells - 1) / kTaskCells * kTaskCells;
            const int left = cnt - q;
            int g = 0, R = 0, ahead = 0;
#pragma unroll
            for (int x = kNumShapes - 1; x >= 0; --x) {  // the first shape that fits
                // a ring: w cells back from the block being written, and one more block where the
                // shifted operand is not read a step ahead (see stream_task)
                int need = (kShapes[x].ahead - 1) * kShapes[x].block;
                for (int l = 0; l < kShapes[x].levels; ++l)
                    need += __builtin_amdgcn_readlane(room, l) + (__builtin_amdgcn_readlane(it.w, l) >= kShapes[x].block ? 1 : 2) * kShapes[x].block;
                if (kShapes[x].levels <= left && need <= ring_cells) g = kShapes[x].levels, R = kShapes[x].block, ahead = kShapes[x].ahead;
            }
            const int U_in = top(before), L_in = bottom(before);
            int32_t *row = buffers + (size_t)cur * row_len;
            // ---- one item by the team, where that is expected to be quicker than the owner alone.  Most passes are
            // too narrow for it by far, and what they pay for the question counts: no divisions, nothing in 64 bits.
            const int w_next = __builtin_amdgcn_readlane(it.w, 0);
            if (__builtin_expect(team && U_in - L_in + w_next > (g == 0 ? 4 * kStreamWaves * 2 * kTaskCells : 8 * g * R), 0)) {
                const int w = w_next, v = __builtin_amdgcn_readlane(it.v, 0);
                const int U = top(before + w), L = bottom(before + w);
                // as many tiles as the team has workgroups, or fewer
                const int span = (U / kTeamCells - L / kTeamCells + 1 + helpers) / (helpers + 1);
                const int tiles = (U / kTeamCells - L / kTeamCells) / span + 1;
                const int together = kTeamJobNs + span * kTeamTileNs;
                const int alone = g == 0 ? ((U - L) / (kStreamWaves * 2 * kTaskCells) + 1) * kHeavyStepNs
                                         : ((U - L) / R + g) * kStepNs / g;
                if (together < alone) {
                    const int words[8] = {w, v, L, U, q > 0 ? U_in : -1, q, cur, span};
                    team_lead(sh, job, helpers, words, tiles, done, buffers, row_len, kp, keep_row, wave, lane);
                    cur ^= 1;
                    streamed += (unsigned)(U_in - L_in + U - L + 2);
                    before += w;
                    q += 1;
                    continue;
                }
            }
            if (g == 0) {
                // ---- one item too heavy for the rings: in place, both operands from global memory,
                // from the top down in steps of at most its weight (a step's shifted operands lie
                // below everything it writes)
                const int w = __builtin_amdgcn_readlane(it.w, 0), v = __builtin_amdgcn_readlane(it.v, 0);
                const int U = top(before + w), L = bottom(before + w);
                constexpr int kStep = kStreamWaves * 2 * kTaskCells;
                for (int hi = U / kStep * kStep; hi >= 0 && hi + kStep > L; hi -= kStep) {
#pragma unroll
                    for (int x = 0; x < 2; ++x) {
                        const int c0 = hi + (wave * 2 + x) * kTaskCells;
                        if (c0 > U || c0 + kTaskCells <= L) continue;
                        row_task(row, row, kp + (size_t)q * keep_row, c0, w, v, q > 0 ? U_in : -1, lane);
                    }
                    __threadfence_block();
                    __syncthreads();
                }
                streamed += (unsigned)(U_in - L_in + U - L + 2);
                before += w;
                q += 1;
                continue;
            }

            // ---- g items per pass ----------------------------------------------------------
            // lane l < g: level l's ring (length, first cell)
            const int rlen = lane < g ? room + (it.w >= R ? 1 : 2) * R + (lane == 0 ? (ahead - 1) * R : 0) : 0;
            int rbase = rlen;
#pragma unroll
            for (int off = 1; off < 8; off <<= 1) {
                const int y = __shfl_up(rbase, off);
                if (lane >= off) rbase += y;
            }
            rbase -= rlen;
            auto upto_of = [&](int l) {  // weight of the list up to and with item q + l
                return ((long long)__builtin_amdgcn_readlane((int)(it.upto >> 32), l) << 32) |
                       (long long)(unsigned)__builtin_amdgcn_readlane((int)it.upto, l);
            };
            const long long after = upto_of(g - 1);
            const int U_out = top(after), L_out = bottom(after);
            const int b0 = L_in / R, nb = U_out / R - b0 + 1;
            const int real = q > 0 ? U_in / R - b0 + 1 : 0;  // blocks of the old row that hold anything
            const int tpl = R / kTaskCells;
            const int steps = nb + g - 1;
            if (wave == kStreamWaves - 1) {
                // the loading wavefront
                const int per_block = R / 256;
                const int ring0 = __builtin_amdgcn_readlane(rlen, 0);
                int at = 0;  // ring position of block `next`
                int next = 0;
                auto issue = [&]() {
                    if (next < real) {
                        const int32_t *src = row + (size_t)(b0 + next) * R + lane * 4;
                        int p = at;
                        for (int x = 0; x < per_block; ++x) {
                            __builtin_amdgcn_global_load_lds((global_ci32 *)(src + x * 256), (lds_i32 *)(ring + p), 16, 0, 0);
                            p += 256;
                            if (p >= ring0) p -= ring0;
                        }
                    }
                    ++next;
                    at += R;
                    if (at >= ring0) at -= ring0;
                };
                int ready = 0;  // ring position of the block to hand over
                // block x is complete in the ring: loaded, zero above the old row's top
                auto finish = [&](int x) {
                    if (x < real) wait_loads(min(next - 1 - x, real - 1 - x) * per_block);
                    if (x >= real) {
                        int p = ready;
                        for (int i = 0; i < per_block; ++i) {
                            *reinterpret_cast<int4 *>(ring + p + lane * 4) = make_int4(0, 0, 0, 0);
                            p += 256;
                            if (p >= ring0) p -= ring0;
                        }
                    } else if (x == real - 1) {
                        for (int i = U_in - (b0 + x) * R + 1 + lane; i < R; i += 64) {
                            int p = ready + i;
                            if (p >= ring0) p -= ring0;
                            ring[p] = 0;
                        }
                    }
                    ready += R;
                    if (ready >= ring0) ready -= ring0;
                };
                for (int x = 0; x < ahead; ++x) issue();
                finish(0);
                step_barrier();
                for (int t = 0; t < steps; ++t) {
                    issue();  // block t + ahead
                    if (t + 1 < nb) finish(t + 1);
                    step_barrier();
                }
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            } else {
                // A computing wavefront: one task of one level per step, the same all through the pass.
                const bool busy = wave < g * tpl;
                const int l = min(wave / tpl, g - 1), sub = wave - wave / tpl * tpl;
                StreamTask k;
                k.w = __builtin_amdgcn_readlane(it.w, l);
                k.v = __builtin_amdgcn_readlane(it.v, l);
                k.len = __builtin_amdgcn_readlane(rlen, l);
                k.rg = ring + __builtin_amdgcn_readlane(rbase, l);
                k.low = bottom(upto_of(l));
                k.top = U_out;
                k.len_out = l + 1 == g ? 0 : __builtin_amdgcn_readlane(rlen, l + 1);
                k.rg_out = ring + (l + 1 == g ? 0 : __builtin_amdgcn_readlane(rbase, l + 1));
                k.row = row;
                k.keep = kp + (size_t)(q + l) * keep_row + lane;
                k.c = b0 * R + sub * kTaskCells;
                k.at = sub * kTaskCells;
                k.first = l;
                if (!busy) {
                    for (int t = 0; t <= steps; ++t) step_barrier();
                } else if (l + 1 < g) {
                    if (k.w >= R) stream_task<true, false>(k, R, steps, lane); else stream_task<false, false>(k, R, steps, lane);
                } else {
                    if (k.w >= R) stream_task<true, true>(k, R, steps, lane); else stream_task<false, true>(k, R, steps, lane);
                }
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (the stores of the pass)
            }
            streamed += (unsigned)(U_in - L_in + U_out - L_out + 2);
            before = after;
            q += g;
            // the next pass reads what this one wrote (other wavefronts' cells included)
            __threadfence_block();
            __syncthreads();
        }

        if (TEAMS && s + 1 == stages) team_tell(job, helpers, kTeamOver);

        // ---- the value and the walk ------------------------------------------------------
        const int32_t *row = buffers + (size_t)cur * row_len;
        // From (last item, c) down the list: item q is taken where its keep bit is set at the capacity left,
        // and without a look once everything up to it fits.  A chain of dependent loads, so six
        // steps are taken per memory round trip: lane L in [2^d, 2^(d+1)) assumes the decisions
        // spelled by the bits of L below its leading one for items q .. q-d+1 and fetches the bit of
        // item q-d at the capacity those leave; a ballot gives all 63 answers.
        auto walk = [&](int c, auto &&take) {
            const int d = 31 - __clz(lane | 1), path = lane - (1 << d);
            int q = cnt - 1;
            while (q >= 0) {
                StreamItem e{};
                if (lane < 6 && q - lane >= 0) e = load_item(list + q - lane);
                const long long upto_q = ((long long)__builtin_amdgcn_readlane((int)(e.upto >> 32), 0) << 32) |
                                         (long long)(unsigned)__builtin_amdgcn_readlane((int)e.upto, 0);
                if (upto_q <= c) {  // everything left fits
                    for (int p = lane; p <= q; p += 64) take(load_item(list + p).index);
                    return c - (int)upto_q;
                }
                int wv[6], iv[6];
#pragma unroll
                for (int i = 0; i < 6; ++i) {
                    wv[i] = __builtin_amdgcn_readlane(e.w, i);
                    iv[i] = __builtin_amdgcn_readlane(e.index, i);
                }
                int cl = c, wd = wv[0];
                long long upto = upto_q;  // of the items up to and with q - d
#pragma unroll
                for (int i = 0; i < 5; ++i) {
                    if (i < d && ((path >> (d - 1 - i)) & 1)) cl -= wv[i];
                    if (i < d) upto -= wv[i];
                    if (d == i + 1) wd = wv[i + 1];
                }
                uint32_t bit = 0;
                if (lane >= 1 && q - d >= 0 && cl >= wd) {
                    if (cl >= upto) {
                        bit = 1;
                    } else {
                        const uint8_t byte = __hip_atomic_load(&kp[(size_t)(q - d) * keep_row + keep_byte(cl)], __ATOMIC_RELAXED,
                                                               __HIP_MEMORY_SCOPE_WORKGROUP);
                        bit = (byte >> (7 - ((cl >> 6) & 7))) & 1u;
                    }
                }
                const unsigned long long takes = __ballot(bit != 0);
                int node = 1;
#pragma unroll
                for (int i = 0; i < 6; ++i) {
                    const int b = (int)((takes >> node) & 1ull);
                    if (b) {
                        if (lane == 0) take(iv[i]);
                        c -= wv[i];
                    }
                    node = 2 * node + b;
                }
                q -= 6;
            }
            return c;
        };
        auto value_at = [&](int c) {
            return c >= weight_all ? value_all
                                   : value_all - __hip_atomic_load(&row[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        };
        if (!caps_sweep) {
            const int value = value_at(C);
            if (wave == 0) {
                const int left = walk(C, [&](int i) {
                    out_asg[i] = j;
                    atomicOr(&sh->placed[i >> 5], 1u << (i & 31));
                });
                if (lane == 0) {
                    out_kv[j] = value;
                    out_kl[j] = C - left;
                }
            }
            total += value;
        } else {
            for (int x = wave; x < m; x += kStreamWaves) {
                const int c = cap[x];
                const int left = walk(c, [&](int i) { atomicOr(reinterpret_cast<unsigned int *>(&out_asg[i]), 1u << x); });
                if (lane == 0) {
                    out_kv[x] = value_at(c);
                    out_kl[x] = c - left;
                }
            }
            total = value_at(C);
        }
        __syncthreads();
    }
    dismiss();
    if (tid == 0) {
        a.total_value[inst] = total;
        if (streamed_cells) atomicAdd(streamed_cells, streamed);
        if (TEAMS) team_leave(job, 0, helpers);
    }
}

}  // namespace

void seq_global_plan(int32_t max_capacity, int32_t max_items, int32_t max_batch, int32_t lds_per_wg_bytes,
                     int32_t compute_units, SeqGlobalPlan *p)
{
    p->compute_units = compute_units;
    p->threads = kThreads;
    p->cells_per_thread = kIter;
    // (check_instance keeps a few words of its own in LDS)
    p->ring_cells = (lds_per_wg_bytes - 256 - kMiscBytes) / 4 / kTaskCells * kTaskCells;
    p->lds_bytes = kMiscBytes + p->ring_cells * 4;
    const int64_t cells = (int64_t)max_capacity + 1;
    p->row_len = (int32_t)((cells + kWaveCells - 1) / kWaveCells * kWaveCells);
    p->keep_words = p->row_len / 64;
    p->max_items = max_items;
    p->max_batch = max_batch;
    p->scratch_bytes = (int64_t)(align256((size_t)max_batch * 2 * p->row_len * 4) +
                                 align256((size_t)max_batch * max_items * p->keep_words * 8) +
                                 2 * align256((size_t)max_batch * max_items * 4) +
                                 align256((size_t)max_batch * sizeof(InstState)) +
                                 align256((size_t)max_batch * max_items * sizeof(StreamItem)) +
                                 align256((size_t)max_batch * sizeof(TeamJob)));
}

hipError_t seq_global_prepare(const SeqGlobalPlan &p, void *scratch)
{
    const Scratch s = carve(p, scratch, p.max_batch);
    hipError_t e = hipMemset(s.jobs, 0, (size_t)p.max_batch * sizeof(TeamJob));  // (every call leaves them so)
    if (e == hipSuccess) e = hipStreamSynchronize(nullptr);
    if (e != hipSuccess) return e;
    // (the attribute belongs to the kernel, not to the handle, and the plan's LDS is the device's)
    for (const void *kernel : {reinterpret_cast<const void *>(&sg_stream<false>), reinterpret_cast<const void *>(&sg_stream<true>)}) {
        e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, p.lds_bytes);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t seq_global_launch(const SeqGlobalPlan &p, const BatchArgs &a, void *scratch, hipStream_t st,
                             Profiler *prof, unsigned long long *streamed_cells)
{
    const Scratch s = carve(p, scratch, p.max_batch);
    if (a.mode != DEFT_MODE_RECURSIVE) {
        int helpers = 0;
        if (p.row_len >= kTeamRows || (p.row_len > kTeamRowsHeavy && p.row_len >= (int64_t)kTeamCellsPerItem * a.item_stride)) {
            helpers = p.compute_units / a.batch - 1;
            const int tiles = p.row_len / kTeamCells;
            if (helpers > tiles) helpers = tiles;
        }
        if (prof) prof->sweep_begin(st);
        hipLaunchKernelGGL(helpers > 0 ? &sg_stream<true> : &sg_stream<false>, dim3((unsigned)a.batch * (unsigned)(helpers + 1)), dim3(kStreamThreads), (size_t)p.lds_bytes, st,
                           a, s.items, s.rows, reinterpret_cast<uint8_t *>(s.keep), s.jobs, helpers, p.row_len, p.max_items,
                           p.ring_cells, prof ? streamed_cells : nullptr);
        if (prof) prof->sweep_end(st);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(sg_init, dim3(a.batch), dim3(kThreads), 0, st, a, s.state);
    hipLaunchKernelGGL(sg_levels_setup, dim3(a.batch), dim3(64), 0, st, a, s.state, s.act, s.probe, p.max_items);
    const int tiles = p.row_len / kTileCells + (p.row_len % kTileCells ? 1 : 0);
    // (the host cannot know how many items an instance has: a workgroup whose instance has fewer exits)
    for (int q = 0; q < a.item_stride; ++q) {
        if (prof) prof->sweep_begin(st);
        hipLaunchKernelGGL(sg_sweep, dim3((unsigned)tiles * (unsigned)a.batch), dim3(kThreads), 0, st, a, q, s.state, s.act,
                           s.probe, s.rows, s.keep, p.row_len, p.keep_words, p.max_items, tiles);
        if (prof) prof->sweep_end(st);
    }
    hipLaunchKernelGGL(sg_traceback, dim3((a.batch + 63) / 64), dim3(64), 0, st, a, s.state, s.act, s.rows, s.keep,
                       p.row_len, p.keep_words, p.max_items);
    return hipGetLastError();
}

}  // namespace deft
