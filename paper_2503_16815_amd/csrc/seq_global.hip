// Sequential multiple-knapsack solve for capacities whose row does not fit LDS
// (Sec. III.B, Problem 1 per window): the row lives in global memory.
//
// The streamed sweep (sg_stream; the sequential mode and the capacity sweep): one launch, one
// workgroup per instance for all stages, lists and walks included.
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
// Measured on the GPT-2 shape (256 instances, C = 381000, one window swept): 2.36 ms, with nine
// instances 2.19 ms; one persistent workgroup per instance over all cells up to C, three items per pass,
// and launches of their own for lists and walks took 11.5 ms, one launch per item 3.55 ms.  What bounds
// it: a step is read, compute, write, barrier for all wavefronts at once (about 1850 cycles for fourteen
// tasks, of which the vector units are busy 740 and LDS 680).
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

struct Scratch {
    int32_t *rows;      // [batch][2][row_len]
    uint64_t *keep;     // [batch][max_items][keep_words]
    int32_t *act;       // [batch][max_items]
    int32_t *probe;     // [batch][max_items]  Algorithm 1: remaining time of the level that ends before entry q
    InstState *state;   // [batch]
    StreamItem *items;  // [batch][max_items]  the streamed sweep's lists
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
constexpr int kMiscBytes = 1024;      // LDS in front of the rings: StreamShared and the placed-item bits

typedef __attribute__((address_space(3))) int32_t lds_i32;
typedef const __attribute__((address_space(1))) int32_t global_ci32;

struct StreamShared {
    int32_t cnt, knap, cap, cap_min;
    int64_t weight;            // of the whole list
    int32_t value;             // of the whole list
    int32_t settled;
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

// All stages of one instance (see the head of this file).
__global__ void __launch_bounds__(kStreamThreads)
sg_stream(BatchArgs a, StreamItem *lists, int32_t *rows, uint8_t *keep, int row_len, int max_items, int ring_cells,
          unsigned long long *streamed_cells)
{
    extern __shared__ __align__(16) char lds_stream[];
    StreamShared *sh = reinterpret_cast<StreamShared *>(lds_stream);
    int32_t *ring = reinterpret_cast<int32_t *>(lds_stream + kMiscBytes);
    const int inst = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int status = check_instance(a, inst, false);
    clear_outputs(a, inst, status);
    if (status != DEFT_OK) return;

    const int n = a.n_items[inst], m = a.n_knapsacks[inst];
    const int32_t *W = a.weights + (size_t)inst * a.item_stride;
    const int32_t *V = a.values + (size_t)inst * a.item_stride;
    const int32_t *cap = a.capacities + (size_t)inst * a.knap_stride;
    int32_t *out_asg = a.assignment + (size_t)inst * a.item_stride;
    int32_t *out_kv = a.knap_value + (size_t)inst * a.knap_stride;
    int32_t *out_kl = a.knap_load + (size_t)inst * a.knap_stride;
    StreamItem *list = lists + (size_t)inst * max_items;
    int32_t *row = rows + (size_t)inst * 2 * row_len;
    uint8_t *kp = keep + (size_t)inst * max_items * (row_len / 8);
    const size_t keep_row = row_len / 8;
    const bool caps_sweep = a.mode == DEFT_MODE_CAPACITY_SWEEP;
    for (int i = tid; i < kMaxItemsPlaced / 32; i += kStreamThreads) sh->placed[i] = 0;
    __syncthreads();

    long long total = 0;
    unsigned long long streamed = 0;
    const int stages = caps_sweep ? min(m, 1) : m;
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
                        int own[kTaskSlots], shd[kTaskSlots];
#pragma unroll
                        for (int k = 0; k < kTaskSlots; ++k) {
                            const int c = c0 + k * 64 + lane;
                            own[k] = q > 0 && c <= U_in ? row[c] : 0;
                            shd[k] = c < w ? INT_MAX : q > 0 && c - w <= U_in ? row[c - w] : 0;
                        }
                        uint32_t bits = 0;
#pragma unroll
                        for (int k = 0; k < kTaskSlots; ++k) {
                            const int passed = (int)((uint32_t)own[k] + (uint32_t)v);
                            bits = shift_in_less(bits, shd[k], passed);
                            row[c0 + k * 64 + lane] = min(passed, shd[k]);
                        }
                        kp[(size_t)q * keep_row + keep_byte(c0) + lane] = (uint8_t)bits;
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

        // ---- the value and the walk ------------------------------------------------------
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
    if (tid == 0) {
        a.total_value[inst] = total;
        if (streamed_cells) atomicAdd(streamed_cells, streamed);
    }
}

}  // namespace

void seq_global_plan(int32_t max_capacity, int32_t max_items, int32_t max_batch, int32_t lds_per_wg_bytes,
                     SeqGlobalPlan *p)
{
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
                                 align256((size_t)max_batch * max_items * sizeof(StreamItem)));
}

hipError_t seq_global_prepare(const SeqGlobalPlan &p)
{
    // (the attribute belongs to the kernel, not to the handle, and the plan's LDS is the device's)
    return hipFuncSetAttribute(reinterpret_cast<const void *>(&sg_stream), hipFuncAttributeMaxDynamicSharedMemorySize,
                               p.lds_bytes);
}

hipError_t seq_global_launch(const SeqGlobalPlan &p, const BatchArgs &a, void *scratch, hipStream_t st,
                             Profiler *prof, unsigned long long *streamed_cells)
{
    const Scratch s = carve(p, scratch, p.max_batch);
    if (a.mode != DEFT_MODE_RECURSIVE) {
        if (prof) prof->sweep_begin(st);
        hipLaunchKernelGGL(sg_stream, dim3((unsigned)a.batch), dim3(kStreamThreads), (size_t)p.lds_bytes, st, a, s.items,
                           s.rows, reinterpret_cast<uint8_t *>(s.keep), p.row_len, p.max_items, p.ring_cells,
                           prof ? streamed_cells : nullptr);
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
