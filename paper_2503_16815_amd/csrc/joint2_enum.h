// Joint two-link solve by enumeration of the selections that can be optimal.
//
// For any prices l0, l1 >= 0 of the two links' capacity, an item's choices (skip, link 0, link 1) are worth
// 0, v - l0 w0 and v - l1 w1; let `best` be the greatest.  With  U = l0 C1 + l1 C2 + sum of best,  every
// selection that keeps to the capacities has
//     value = U - (sum over items of best - worth of the choice made) - l0 (room left on link 0) - l1 (on link 1).
// So a selection of value V departs from the best choices by a total loss of at most U - V, and an item whose
// departures all cost more than U - V has its best choice in every selection at least as good.  Once some
// selection of value V is known, what is left is to look through the departures of total loss up to U - V: on the
// two-link batch (64 items of 1 to 64, C1 = C2 = 512, U within 1 % of the optimum at the best prices)
// a few hundred to a hundred thousand of them, where the table has 17 million cell-updates.
//
// The prices come from a search on grids (U is convex in them; any prices give a valid bound).  A round
// opens the choices of loss up to G (the 16th least loss of all, the 24th, ..., never more than the best selection
// known leaves), splits the items that have any into three groups and lists every group's combinations of
// loss up to G in LDS: the combinations of group Q sorted by roughly what they take of link 1, then of link 0, those of
// P1 and P2 taken in pairs, each looking up the partners that leave little enough room on either link.  If
// the best selection met loses no more than G, all better or equal ones have been met: it is the answer, and
// among equals the one with the smallest choice number is the one that the DP's walk returns.  Where a list runs over,
// smaller steps and other groups are tried, then Q is made in parts, one after the other: the choices of its items of
// least loss (up to four, three choices each) are a part's own, and P1 and P2 stay as they are.  (The part of the best choices is the
// largest: of an item it keeps half of the list at least where one departure is open, a third where both are.)  If lists or time
// run over (a share of what the sweep is expected to take), or the table sweep, which begins beside it when a compute unit is free, ends
// first, the instance is left to that; so are instances in which the prices are zero (everything fits one link or the other:
// all choices cost nothing).
//
// All quantities that decide are whole numbers: prices and losses in units of 2^-F, values as they are.
//
// What bounds it: latency.  One workgroup owns an instance; a round is a chain of barriers (one for an item of each group
// once the lists are long), its pairs are lookups in LDS at places of the lanes' own, and a launch lasts as long as its hardest
// instance.  Of the two-link batch half of the instances are solved after 85 us, the last one after 0.6 to 1.3 ms, 1.1 to 2.4 where lists run
// over (2.8 to 4.4 without parts); by the input one of some 1200 is left to the table sweep, and the call takes 3.9 to 4.4 ms then (all
// by the sweep: 6.36).  40 instances of 20 to 62
// items 0.41 of the sweep, 256 0.53 (geometric means over 30 kinds each).
// Tried and not kept: every lane noting ties as it meets them (two passes instead, the second only where several selections
// are as good: 72 -> 5 ms), Q sorted by link 0 alone, or by link 1 in steps of 128 (cells of both: pairs / 3), no table of
// least losses (it turns nine of ten pairs away before they are looked up).
#pragma once

#include "instance_check.h"

namespace deft {

namespace {

constexpr int kEnumerated = 1, kSwept = 2;  // which side has come to its end (both may)
constexpr int kEnumThreads = 1024;
constexpr int kEnumWaves = kEnumThreads / 64;
constexpr int kEnumItems = kEnumThreads;  // a thread per item
constexpr int kEnumCapacity = 768;        // what P1 and P2 together (42 items) change on a link stays within 16 bits
constexpr int kEnumOpen = 64;             // items that may have open choices (the listed ones), and choices open in the last round
constexpr int kEnumRounds = 7;            // 16, 24, ..., 64 open choices
// Shorter lists are swept at once: 248 instances of 8 items (C1 = 75, C2 = 253) 92 us, by enumeration 155; four of 19
// items (138 and 407) 412 and 57.
constexpr int kEnumFewest = 16;
constexpr int kLeapChoices = 64, kReach = 2;
constexpr int kBranches = 4;              // items whose choices Q is split up by, at most, where it runs over
constexpr int kListQ = 5120, kListP1 = 2048, kListP2 = 1536;
constexpr int kCells0 = 128, kCells1 = 64;  // that group Q is sorted by
constexpr int kCells = kCells0 * kCells1;
constexpr int kFilterPairs = 1 << 13;     // the fewest pairs that make the table of least losses worth its 3 us
constexpr int kNever = 1 << 30;           // the loss of a choice that is out of the question
constexpr int kEnumComputeUnits = 256, kEnumAlike = 20;
constexpr int kLookTicks = 2000;          // of 10 ns, between looks at whether the sweep has come to its end
constexpr int kPriceGrid = 16, kPriceRounds = 4;

struct EnumResult {
    int q;                      // -1: no result
    uint32_t q_mask, pair;      // what it takes of Q, its places in P1 and P2 (11 bits each)
    unsigned long long lo, hi;  // the choices of the open items, two bits each by item index
};

struct EnumShared {
    union {
        struct {
            float4 item[kEnumItems];         // w0, value there (-1: does not fit), w1, value there
            int32_t loss[2][kEnumItems];     // of the two departures, the lesser first
            int32_t place[3][kEnumItems];
            float partial[4][kPriceGrid * kPriceGrid];
        } all;
        struct {
            int32_t q_loss[kListQ], q_use[kListQ];  // (after sorting: link 0 << 16 | link 1)
            uint32_t q_mask[kListQ];
            int32_t p1_loss[kListP1], p1_use[kListP1];
            uint32_t p1_mask[kListP1];
            int32_t p2_loss[kListP2], p2_use[kListP2];
            uint32_t p2_mask[kListP2];
            uint32_t begin[kCells / 2 + 1];         // 16 bits each: how many of Q are in a cell, then where they begin
            uint16_t least[kCells0][kCells1];
            uint32_t queue[kEnumWaves][192];
        } list;
    };
    // open items by their lesser loss
    int32_t loss[2][kEnumOpen], use[2][kEnumOpen], taken[kEnumOpen], item[kEnumOpen];
    uint8_t option[2][kEnumOpen], dflt[kEnumOpen], by_index[kEnumOpen], choice[kEnumOpen];
    uint8_t order[3][kEnumOpen];              // a group's items
    unsigned long long members[3];            // the same as bits
    // the round's
    int32_t size[3], places[3], bits[3];               // of the lists as their first wavefronts leave them, and the items to go
    uint16_t meaning[3][32];                  // of a mask bit: item << 2 | choice
    int32_t appended[kEnumOpen][3];
    int32_t q_default[2];                     // what the default choices of group Q's items take
    int32_t sum[4];
    int32_t threshold[kEnumRounds];
    int32_t unlisted;                         // the least loss of a departure of an item that is not listed
    int32_t most[2];
    int32_t bound[4], bound_at[4];            // of a grid of prices, by quarters
    int32_t wave_sum[kEnumWaves];
    union {
        int32_t edge[kEnumWaves][kCells1];
        ulonglong2 flips[3][8][16];           // of every four mask bits together
    };
    EnumResult result[kEnumWaves];
    unsigned long long default_lo, default_hi;
    unsigned long long flip_lo[3][32], flip_hi[3][32];  // what a mask bit changes of them
    int32_t over, late, least;                // least: what the best selection met so far loses
    uint32_t q_mask, pair;
};

static_assert(sizeof(EnumShared) + 64 <= 160 * 1024, "a compute unit's LDS");  // (check_instance has some words of its own)

// Over the 64 lanes of a wavefront whose lanes are all active, the result in every lane.
template <class Op>
__device__ __forceinline__ int enum_wave_reduce(int x, Op op)
{
    x = op(x, __builtin_amdgcn_update_dpp(x, x, 0xB1, 0xf, 0xf, false));   // quad_perm [1,0,3,2]
    x = op(x, __builtin_amdgcn_update_dpp(x, x, 0x4E, 0xf, 0xf, false));   // quad_perm [2,3,0,1]
    x = op(x, __builtin_amdgcn_update_dpp(x, x, 0x124, 0xf, 0xf, false));  // row_ror:4
    x = op(x, __builtin_amdgcn_update_dpp(x, x, 0x128, 0xf, 0xf, false));  // row_ror:8
    return op(op(__builtin_amdgcn_readlane(x, 0), __builtin_amdgcn_readlane(x, 16)),
              op(__builtin_amdgcn_readlane(x, 32), __builtin_amdgcn_readlane(x, 48)));
}
__device__ __forceinline__ int enum_wave_sum(int x) { return enum_wave_reduce(x, [](int a, int b) { return a + b; }); }
__device__ __forceinline__ int enum_wave_max(int x) { return enum_wave_reduce(x, [](int a, int b) { return max(a, b); }); }
__device__ __forceinline__ int enum_wave_min(int x) { return enum_wave_reduce(x, [](int a, int b) { return min(a, b); }); }
__device__ __forceinline__ int enum_below(unsigned long long mask, int lane) { return __popcll(mask & ((1ull << lane) - 1ull)); }
// a packed pair of changes: a on link 0, b on link 1
__device__ __forceinline__ int use_b(int ab) { return (int)(int16_t)(ab & 0xffff); }
__device__ __forceinline__ int use_a(int ab) { return (ab - use_b(ab)) >> 16; }

__device__ __forceinline__ bool enum_before(const EnumResult &x, const EnumResult &y)
{
    if (x.q < 0 || y.q < 0) return x.q >= 0;
    return x.hi != y.hi ? x.hi < y.hi : x.lo < y.lo;
}
// The departures of a combination that group l makes.
__device__ __forceinline__ uint32_t enum_mask(const EnumShared &s, int l, uint32_t pair, uint32_t q_mask)
{
    return l == 0 ? q_mask : l == 1 ? s.list.p1_mask[pair >> 11] : s.list.p2_mask[pair & 2047];
}

__device__ __forceinline__ bool enum_takes(int n, int c0, int c1) { return n <= kEnumItems && c0 <= kEnumCapacity && c1 <= kEnumCapacity; }

// The whole workgroup's.  What it answers gets kEnumerated in `solved`; anything else is left to the table sweep with its outputs
// cleared.  It gives up when the sweep has put kSwept there.
template <class State>
__device__ __forceinline__ void jt_enumerate(const BatchArgs &a, int inst, State *state, int32_t *solved, char *lds)
{
    EnumShared &s = *reinterpret_cast<EnumShared *>(lds);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int status = check_instance(a, inst, true);
    clear_outputs(a, inst, status);
    const int n = status == DEFT_OK ? a.n_items[inst] : 0;
    const int c0 = status == DEFT_OK ? a.capacities[(size_t)inst * a.knap_stride] : -1;
    const int c1 = status == DEFT_OK ? a.capacities[(size_t)inst * a.knap_stride + 1] : -1;
    if (tid == 0) {
        State st;
        st.status = status;
        st.n = n;
        st.c1 = c0;
        st.c2 = c1;
        state[inst] = st;
    }
    if (n == 0 || !enum_takes(n, c0, c1)) return;

    const long long began = wall_clock64();

    // ---- the items, one per thread ---------------------------------------------------
    const int32_t *W = a.weights + (size_t)inst * 2 * a.item_stride;
    const bool here = tid < n;
    const int v = here ? a.values[(size_t)inst * a.item_stride + tid] : 0;
    const int w0 = here ? W[tid] : 1, w1 = here ? W[a.item_stride + tid] : 1;
    const bool fits0 = v > 0 && w0 <= c0, fits1 = v > 0 && w1 <= c1;  // (an item of no value is never taken)
    if (tid < 4) s.sum[tid] = 0;
    if (tid < 2) s.most[tid] = 0;
    if (tid < kEnumRounds) s.threshold[tid] = kNever;
    if (tid == 0) s.over = s.late = 0, s.least = s.unlisted = kNever;
    __syncthreads();
    const int waves_used = (n + 63) >> 6;
    if (wave < waves_used) {
        s.all.item[tid] = make_float4((float)w0, fits0 ? (float)v : -1.0f, (float)w1, fits1 ? (float)v : -1.0f);
        // (not negative: ordered like their bits)
        const int most0 = enum_wave_max(__float_as_int(fits0 ? (float)v / (float)w0 : 0.0f));
        const int most1 = enum_wave_max(__float_as_int(fits1 ? (float)v / (float)w1 : 0.0f));
        const int wave_v = enum_wave_max(v), all0 = enum_wave_sum(v > 0 ? min(w0, c0 + 1) : 0);
        const int all_w = enum_wave_sum(here ? min(w0, c0 + 1) : 0);
        if (lane == 0) {
            atomicMax(&s.most[0], most0);
            atomicMax(&s.most[1], most1);
            atomicMax(&s.sum[3], wave_v);
            atomicAdd(&s.sum[0], all0);
            atomicAdd(&s.sum[1], all_w);
        }
    }
    __syncthreads();
    const bool all_on_link0 = s.sum[0] <= c0;  // every item of value fits there: the smallest of the best selections
    const int most_v = s.sum[3], all_weight = s.sum[1];
    __syncthreads();
    if (tid < 4) s.sum[tid] = 0;

    auto finish = [&](auto &&choice_of) {  // of this thread's item: 0 none, 1 link 0, 2 link 1
        __syncthreads();
        const int choice = choice_of();
        if (wave < waves_used) {
            const int v0 = enum_wave_sum(choice == 1 ? v : 0), v1 = enum_wave_sum(choice == 2 ? v : 0);
            const int l0 = enum_wave_sum(choice == 1 ? w0 : 0), l1 = enum_wave_sum(choice == 2 ? w1 : 0);
            if (lane == 0) {
                atomicAdd(&s.sum[0], v0);
                atomicAdd(&s.sum[1], v1);
                atomicAdd(&s.sum[2], l0);
                atomicAdd(&s.sum[3], l1);
            }
            if (choice != 0) a.assignment[(size_t)inst * a.item_stride + tid] = choice - 1;
        }
        __syncthreads();
        if (tid < 2) {  // (the threads that cleared these)
            a.knap_value[(size_t)inst * a.knap_stride + tid] = s.sum[tid];
            a.knap_load[(size_t)inst * a.knap_stride + tid] = s.sum[2 + tid];
        }
        if (tid == 0) {
            a.total_value[inst] = (long long)s.sum[0] + s.sum[1];
            __hip_atomic_fetch_or(&solved[inst], kEnumerated, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    };
    if (all_on_link0) {
        finish([&]() { return v > 0 ? 1 : 0; });
        return;
    }

    if (n < kEnumFewest) return;

    // ---- prices ---------------------------------------------------------------------------
    // 16 x 16 candidates at a time around the best so far; the first grid spans 2^10.5, every further one is
    // 3.75 times as fine, unless the best lies on its border.  Four wavefronts hold the grid, four times, each with
    // a quarter of the items.  Floats: prices only make the bound tighter or looser.
    float x0 = 0.0f, x1 = 0.0f, best_bound = INFINITY;
    {
        static_assert(kPriceGrid == 16 && kEnumWaves == 16, "a candidate per lane of four wavefronts, four times");
        const float most0 = __int_as_float(s.most[0]), most1 = __int_as_float(s.most[1]);
        float half0 = 0.0f, half1 = 0.0f;
        auto spread = [](float most, int i) { return i == 0 ? 0.0f : most * exp2f(-0.75f * (float)(kPriceGrid - 1 - i)); };
        const int g = tid & 255, part = wave >> 2;
        const int i_begin = n * part >> 2, i_end = n * (part + 1) >> 2;
#pragma unroll 1
        for (int round = 0; round <= kPriceRounds; ++round) {
            const float step0 = 2.0f * half0 / (kPriceGrid - 1), step1 = 2.0f * half1 / (kPriceGrid - 1);
            auto at0 = [&](int i) { return round == 0 ? spread(most0, i) : fmaxf(0.0f, x0 - half0 + step0 * (float)i); };
            auto at1 = [&](int i) { return round == 0 ? spread(most1, i) : fmaxf(0.0f, x1 - half1 + step1 * (float)i); };
            const float p0 = at0(g & (kPriceGrid - 1)), p1 = at1(g / kPriceGrid);
            float bound = part == 0 ? p0 * (float)c0 + p1 * (float)c1 : 0.0f;
#pragma unroll 4
            for (int i = i_begin; i < i_end; ++i) {
                const float4 it = s.all.item[i];
                bound += fmaxf(fmaxf(it.y - p0 * it.x, it.w - p1 * it.z), 0.0f);
            }
            s.all.partial[part][g] = bound;
            __syncthreads();
            if (part == 0) {
                bound = (bound + s.all.partial[1][g]) + (s.all.partial[2][g] + s.all.partial[3][g]);
                const int bits = __float_as_int(bound), least = enum_wave_min(bits);  // (not negative)
                const int first = __builtin_ctzll(__ballot(bits == least));
                if (lane == 0) s.bound[wave] = least, s.bound_at[wave] = wave * 64 + first;
            }
            __syncthreads();
            int at = 0;
            for (int i = 1; i < 4; ++i) at = s.bound[i] < s.bound[at] ? i : at;
            const int best = s.bound_at[at], i0 = best & (kPriceGrid - 1), i1 = best / kPriceGrid;
            const float y0 = at0(i0), y1 = at1(i1);
            bound = __int_as_float(s.bound[at]);
            if (round == 0) {
                half0 = fmaxf(at0(min(i0 + 1, kPriceGrid - 1)) - y0, y0 - at0(max(i0 - 1, 0)));
                half1 = fmaxf(at1(min(i1 + 1, kPriceGrid - 1)) - y1, y1 - at1(max(i1 - 1, 0)));
            } else {
                if (i0 != 0 && i0 != kPriceGrid - 1) half0 = 2.0f * step0;
                if (i1 != 0 && i1 != kPriceGrid - 1) half1 = 2.0f * step1;
            }
            if (bound < best_bound) best_bound = bound, x0 = y0, x1 = y1;
        }
    }
    if (x0 == 0.0f && x1 == 0.0f) return;
    // units of 2^-F: values below 2^29
    const int F = min(max(__builtin_clz(most_v) - 3, 0), 16);
    const int l0 = (int)rintf(ldexpf(x0, F)), l1 = (int)rintf(ldexpf(x1, F));

    // ---- losses ----------------------------------------------------------------------------
    int dflt = 0, option_a = 1, option_b = 2, loss_a = kNever, loss_b = kNever;
    {
        constexpr long long kOut = -(1ll << 60);
        const long long r0 = fits0 ? ((long long)v << F) - (long long)l0 * w0 : kOut;
        const long long r1 = fits1 ? ((long long)v << F) - (long long)l1 * w1 : kOut;
        const long long best = max(0ll, max(r0, r1));
        dflt = best == 0 ? 0 : r0 == best ? 1 : 2;
        auto loss = [&](int choice) {
            const long long x = best - (choice == 0 ? 0ll : choice == 1 ? r0 : r1);
            return x < kNever ? (int)x : kNever;
        };
        option_a = dflt == 0 ? 1 : 0;
        option_b = dflt == 2 ? 1 : 2;
        loss_a = v > 0 ? loss(option_a) : kNever;
        loss_b = v > 0 ? loss(option_b) : kNever;
        if (loss_b < loss_a) {
            const int x = loss_a, y = option_a;
            loss_a = loss_b, option_a = option_b;
            loss_b = x, option_b = y;
        }
    }
    if (wave < waves_used) {
        s.all.loss[0][tid] = loss_a;
        s.all.loss[1][tid] = loss_b;
        s.all.place[0][tid] = s.all.place[1][tid] = s.all.place[2][tid] = 0;
        const int u0 = enum_wave_sum(dflt == 1 ? w0 : 0), u1 = enum_wave_sum(dflt == 2 ? w1 : 0);
        const int near = __popcll(__ballot(loss_a < 1 << F)) + __popcll(__ballot(loss_b < 1 << F));
        if (lane == 0) {
            atomicAdd(&s.sum[0], u0);
            atomicAdd(&s.sum[1], u1);
            atomicAdd(&s.sum[2], near);
        }
    }
    if (tid < kEnumOpen) s.loss[0][tid] = s.loss[1][tid] = kNever;
    __syncthreads();
    const int used0 = s.sum[0], used1 = s.sum[1];  // by the default choices
    const int alike = s.sum[2];                    // departures within one unit of value
    int rank = kEnumItems;
    {
        // places among the lesser losses, and of both among all losses (ties in some order): every item's
        // against a share of the others
        const int parts = kEnumWaves / waves_used, part = wave / waves_used;
        if (part < parts) {
            const int i = tid - part * waves_used * 64, xa_i = s.all.loss[0][i], xb_i = s.all.loss[1][i];
            int place = 0, place_a = 0, place_b = 0;
#pragma unroll 2
            for (int j = n * part / parts; j < n * (part + 1) / parts; ++j) {
                const int xa = s.all.loss[0][j], xb = s.all.loss[1][j];
                place += xa < xa_i || (xa == xa_i && j < i) ? 1 : 0;
                place_a += xb < xa_i ? 1 : 0;
                place_b += (xa <= xb_i ? 1 : 0) + (xb < xb_i || (xb == xb_i && j < i) ? 1 : 0);
            }
            atomicAdd(&s.all.place[0][i], place);
            atomicAdd(&s.all.place[1][i], place + place_a);
            atomicAdd(&s.all.place[2][i], place_b);
        }
    }
    __syncthreads();
    if (wave < waves_used) {
        rank = s.all.place[0][tid];
        const int place_a = s.all.place[1][tid], place_b = s.all.place[2][tid];
        auto threshold = [&](int place, int loss) {
            if (loss < kNever && (place & 7) == 0 && place >= 16 && place <= kEnumOpen) s.threshold[(place >> 3) - 2] = loss;
        };
        threshold(place_a, loss_a);
        threshold(place_b, loss_b);
        if (rank == kEnumOpen) s.unlisted = loss_a;
        if (rank < kEnumOpen && loss_a < kNever) {
            auto takes = [&](int choice) { return choice == 1 ? w0 * 65536 : choice == 2 ? w1 : 0; };
            s.loss[0][rank] = loss_a;
            s.loss[1][rank] = loss_b;
            s.use[0][rank] = takes(option_a) - takes(dflt);
            s.use[1][rank] = loss_b < kNever ? takes(option_b) - takes(dflt) : 0;
            s.taken[rank] = takes(dflt);
            s.option[0][rank] = (uint8_t)option_a;
            s.option[1][rank] = (uint8_t)option_b;
            s.dflt[rank] = (uint8_t)dflt;
            s.item[rank] = tid;
        }
    }
    __syncthreads();
    // Three groups: of every ten items by loss, four to Q, three each to P1 and P2; where a list runs over so, about
    // a third each (split 1); where P1 or P2 still does, as at first again (2) and then half of them to Q (3), which is
    // made in parts then.
    auto make_groups = [&](int split) {
        const bool open = s.loss[0][lane] < kNever;
        const int five = lane % 5, ten = lane % 10, three = lane % 20 == 19 ? 0 : lane % 3, four = lane % 4;
        const int group = split == 3 ? (four & 1) * ((four + 1) >> 1) : split == 1 ? three : five == 0 || five == 3 ? 0 : five == 1 || ten == 4 ? 1 : 2;
#pragma unroll
        for (int l = 0; l < 3; ++l) {
            const unsigned long long mask = __ballot(open && group == l);
            if (open && group == l) s.order[l][enum_below(mask, lane)] = (uint8_t)lane;
            if (lane == 0) s.members[l] = mask;
        }
    };
    if (wave == 0) {
        make_groups(0);
        const bool open = s.loss[0][lane] < kNever;
        int by_index = 0;
        const int item = open ? s.item[lane] : kEnumItems;
#pragma unroll 4
        for (int j = 0; j < kEnumOpen; ++j) by_index += __builtin_amdgcn_readlane(item, j) < item ? 1 : 0;
        s.by_index[lane] = (uint8_t)by_index;
        unsigned long long lo = open && by_index < 32 ? (unsigned long long)s.dflt[lane] << (2 * by_index) : 0ull;
        unsigned long long hi = open && by_index >= 32 ? (unsigned long long)s.dflt[lane] << (2 * (by_index - 32)) : 0ull;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            lo |= __shfl_xor(lo, off);
            hi |= __shfl_xor(hi, off);
        }
        if (lane == 0) s.default_lo = lo, s.default_hi = hi;
    }
    __syncthreads();

    // ---- rounds -----------------------------------------------------------------------------
    int least = kNever;  // what the best selection met so far loses
    int last_G = -1;
    // What a sweep takes, in ticks of 10 ns: its rows times an item's, less those that hold everything or cannot be reached, a
    // row 300 cells more than it has (within 25 % of nine sweeps of ten).  While there are compute units for the sweeps as well,
    // an attempt may take as long as most of one; else the sweep begins only when some attempt ends.  Instances with more than
    // kEnumAlike departures within one unit of value are solved late if at all (of values that are the times on link 0 one in
    // ten, of unrelated values all have less).  Measured (calls against the sweep alone, the geometric mean over 150 kinds each of
    // 32 and 256 instances): shares of 0.6, 0.5 and 0.12 0.782 and 0.950; with sweeps that
    // looked at every block whether to end 0.6, 0.45 and 0.12 0.800 and 0.974; 1, 0.5 and 0.15 0.815 and 0.975; 1, 0.4 and 0.4 0.829
    // and 1.007; 0.25 for many leaves more of the calls to a sweep (256 of 20 to 64 items 0.62 of the sweep, 0.52 at 0.5).
    const float held = fminf(1.0f, (float)(c0 + 1) / (float)max(all_weight, 1));
    const long long sweep_ticks = n * 600 + (long long)((1.0f - held) * (float)((c0 + 1) * (c1 + 301)) * (float)n / 41.0f);
    const int share = 2 * a.batch <= kEnumComputeUnits ? 60 : alike > kEnumAlike ? 12 : 50;
    const long long deadline = began + sweep_ticks * share / 100;
    long long look = began + sweep_ticks / 2;                   // (it does not before)
    // Looked at wherever a list begins (a part, a round) and by every wavefront for 64 pairs looked up: a part whose pairs are
    // all passed over takes up to 60 us, and there are up to 81.  (Looked at for pairs alone, attempts of 392 of 600 kinds of calls ended
    // late, by up to 13.7 ms where they were allowed 0.23.)
    auto late = [&]() {
        const long long now = wall_clock64();
        if (now <= look) return now > deadline;
        look = now + kLookTicks;
        return now > deadline || __hip_atomic_load(&solved[inst], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
    };
    const int group = wave < 10 ? 0 : wave < 13 ? 1 : 2;        // the list that this wavefront makes
    const int first_wave = group == 0 ? 0 : group == 1 ? 10 : 13, list_waves = group == 0 ? 10 : 3;
    const int limit = group == 0 ? kListQ : group == 1 ? kListP1 : kListP2;
    int32_t *const l_loss = group == 0 ? s.list.q_loss : group == 1 ? s.list.p1_loss : s.list.p2_loss;
    int32_t *const l_use = group == 0 ? s.list.q_use : group == 1 ? s.list.p1_use : s.list.p2_use;
    uint32_t *const l_mask = group == 0 ? s.list.q_mask : group == 1 ? s.list.p1_mask : s.list.p2_mask;
    const float per0 = l0 > 0 ? 1.0f / (float)l0 : 0.0f, per1 = l1 > 0 ? 1.0f / (float)l1 : 0.0f;
    // cells of 2^cell0 by 2^cell1 (the last ones take what is left)
    int cell0 = 0, cell1 = 0;
    while ((c0 >> cell0) > kCells0) ++cell0;
    while ((c1 >> cell1) > kCells1) ++cell1;
    const uint16_t *const begin16 = reinterpret_cast<const uint16_t *>(s.list.begin);
    auto row_of = [&](int on0) { return min(on0 >> cell0, kCells0 - 1) * kCells1; };
    auto column_of = [&](int on1) { return min(on1 >> cell1, kCells1 - 1); };

    bool may_leap = true;
    int split = 0, branches = 0;
    for (int round = 0; round < kEnumRounds;) {
        int G = s.threshold[round] - 1;
        // What is left to look through is known: straight to it, unless the choices open then are so many that a better
        // selection, met by a round before, will be worth its time, or some of them are of items that are not listed.
        // (A round's own G leaves at most 64 choices open, and the items of those are listed.)
        const int choices = __popcll(__ballot(s.loss[0][lane] <= least)) + __popcll(__ballot(s.loss[1][lane] <= least));
        const bool leap = may_leap && least > G && least < s.unlisted && choices <= kLeapChoices;
        if (leap || least <= G) G = least;
        if (G <= last_G) {
            ++round;
            continue;
        }
        auto retry = [&](bool q_over) {  // a list has run over: in smaller steps, other groups, or Q in parts
            if (leap) {
                may_leap = false;
            } else if (split > 0 && alike > kEnumAlike) {
                // (solved late if at all; by parts none was, and 32 instances of 39 items at 103 x 316 took 0.92 ms, 0.71 so)
                if (tid == 0) s.over = 1;
            } else if (split == 0 || (!q_over && split < 3)) {
                ++split;
                branches = split == 1 ? 0 : max(branches, 1);
                if (wave == 0) make_groups(split);
            } else if (q_over && branches < kBranches) {
                ++branches;
            } else if (tid == 0) {
                s.over = 1;
            }
            __syncthreads();
        };
        const int open = __popcll(__ballot(s.loss[0][lane] <= G));
        const unsigned long long opened = open >= 64 ? ~0ull : (1ull << open) - 1ull;
        // The group's open items in the lanes of its wavefronts: the two departures, their mask bits (the first one's is
        // the item's place, the second one's behind all those).
        const int count = __popcll(s.members[group] & opened);
        const bool mine = lane < count;
        const int r = mine ? s.order[group][lane] : 0;
        const int first_l = mine ? s.loss[0][r] : kNever, second_l = mine ? s.loss[1][r] : kNever;
        const int first_u = s.use[0][r], second_u = s.use[1][r];
        const unsigned long long both = __ballot(second_l <= G);
        const int second_b = count + enum_below(both, lane);
        // Q in parts: the choices of its `branches` items of least loss are the part's, three to an item (one group's items are
        // any of them, so a part is its combinations with those choices).
        int turns = 1;
        for (int b = 0; b < branches; ++b) turns *= 3;
        const int q_count = __popcll(s.members[0] & opened), stop = group == 0 ? branches : 0;
        // (the first rounds look beyond G, for a selection that says how far the others have to)
        const int known = least < kNever ? least : (int)min(kReach * (long long)G, (long long)kNever - 1);
        int best = known + 1, copies = 0;  // what this lane's best selection loses, and whether it has met it twice
        EnumResult chosen{-1, 0, 0, 0, 0};
        bool several = false, again = false, filtered = false;
        int size[3] = {0, 0, 0};
        const int coarse = max(0, 18 - __builtin_clz(G | 1));  // G in 14 bits
#pragma unroll 1
        for (int pass = 0, part = 0;;) {
            int part_loss = 0, part_use = 0;
            uint32_t part_mask = 0;
            for (int b = 0, digits = part, second = q_count; b < branches; ++b, digits /= 3) {
                const int at = s.order[0][b], digit = b < q_count ? digits % 3 : digits % 3 == 0 ? 0 : 3;
                const bool twice = b < q_count && s.loss[1][at] <= G;
                if (digit == 1) part_loss = min(part_loss + s.loss[0][at], kNever), part_use += s.use[0][at], part_mask |= 1u << b;
                if (digit == 2 && twice) part_loss = min(part_loss + s.loss[1][at], kNever), part_use += s.use[1][at], part_mask |= 1u << second;
                if (digit == 3 || (digit == 2 && !twice)) part_loss = kNever;
                second += twice ? 1 : 0;
            }
            part_loss = __builtin_amdgcn_readfirstlane(part_loss);
            const bool first_turn = pass == 0 && part == 0;
            // No selection counts that loses more than the best one met so far, by this part or one before.
            const int cut = __builtin_amdgcn_readfirstlane(min(G, s.least));
            if (part_loss <= cut && (pass == 0 || turns > 1)) {
                int have = 1, place = count - 1;
                // One item into the list, by `waves` wavefronts of which this is number `w`: entries [0, have) are followed
                // by what they make with the item's departures.  to(more) is where this wavefront's go.
                auto grow = [&](int p, int w, int waves, auto &&to) {
                    const int loss1 = __builtin_amdgcn_readlane(first_l, p), loss2 = __builtin_amdgcn_readlane(second_l, p);
                    const int use1 = __builtin_amdgcn_readlane(first_u, p), use2 = __builtin_amdgcn_readlane(second_u, p);
                    const int bit2 = __builtin_amdgcn_readlane(second_b, p);
                    const bool twice = loss2 <= cut;
                    for (int base = w * 64; base < have; base += waves * 64) {
                        const int e = base + lane;
                        const int loss = e < have ? l_loss[e] : kNever, use = e < have ? l_use[e] : 0;
                        const uint32_t mask = e < have ? l_mask[e] : 0;
                        const bool one = loss <= cut - loss1, two = twice && loss <= cut - loss2;
                        const unsigned long long ones = __ballot(one), twos = __ballot(two);
                        const int at = to(__popcll(ones) + __popcll(twos));
                        const int at1 = at + enum_below(ones, lane), at2 = at + __popcll(ones) + enum_below(twos, lane);
                        if (one && at1 < limit) {
                            l_loss[at1] = loss + loss1;
                            l_use[at1] = use + use1;
                            l_mask[at1] = mask | 1u << p;
                        }
                        if (two && at2 < limit) {
                            l_loss[at2] = loss + loss2;
                            l_use[at2] = use + use2;
                            l_mask[at2] = mask | 1u << bit2;
                        }
                    }
                };
                // The greatest losses first (they combine with little, so the lists stay short for long).  A short list is
                // its first wavefront's alone.
                if (wave == first_wave && (first_turn || group == 0)) {
                    auto means = [&](int bit, int option) {
                        const int at = s.by_index[r];
                        const unsigned long long flip = (unsigned long long)(option ^ s.dflt[r]) << (2 * (at & 31));
                        s.meaning[group][bit] = (uint16_t)(r << 2 | option);
                        s.flip_lo[group][bit] = at < 32 ? flip : 0ull;
                        s.flip_hi[group][bit] = at < 32 ? 0ull : flip;
                    };
                    const int bits = count + __popcll(both);
                    if (bits > 32) {
                        if (lane == 0) s.over = 1;
                    } else {
                        if (mine) means(lane, s.option[0][r]);
                        if (second_l <= G) means(second_b, s.option[1][r]);
                        if (group == 0) {
                            const int u = mine ? s.taken[r] : 0, u0 = enum_wave_sum(u >> 16), u1 = enum_wave_sum(u & 0xffff);
                            if (lane == 0) s.q_default[0] = u0, s.q_default[1] = u1;
                        }
                        if (lane == 0) {
                            l_loss[0] = group == 0 ? part_loss : 0;
                            l_use[0] = group == 0 ? part_use : 0;
                            l_mask[0] = group == 0 ? part_mask : 0;
                        }
                        while (place >= stop && have <= 64 * list_waves) {
                            int next = have;
                            __builtin_amdgcn_wave_barrier();
                            grow(place, 0, 1, [&](int more) {
                                const int at = next;
                                next += more;
                                return at;
                            });
                            __builtin_amdgcn_wave_barrier();
                            have = next;
                            --place;
                            if (have > limit) break;
                        }
                        if (lane == 0) s.size[group] = have, s.places[group] = place, s.bits[group] = bits;
                    }
                }
                for (int i = tid; i < kEnumOpen * 3; i += kEnumThreads) s.appended[i / 3][i % 3] = 0;
                if (tid == kEnumThreads - 1) s.late = late() ? 1 : 0;  // (of a wavefront that makes no short list)
                __syncthreads();
                if (s.over | s.late) return;
                int steps = 0;
                bool over = false;
        #pragma unroll
                for (int l = 0; l < 3; ++l) {
                    if (l > 0 && !first_turn) continue;
                    size[l] = s.size[l];
                    over = over || size[l] > (l == 0 ? kListQ : l == 1 ? kListP1 : kListP2);
                    steps = max(steps, s.places[l] + 1 - (l == 0 ? branches : 0));
                }
                if (over) {
                    again = true;
                    break;
                }
                place = first_turn || group == 0 ? s.places[group] : -1;
                // A longer one is made by all of the group's wavefronts, a barrier per item.
                for (int step = 0; step < steps; ++step) {
                    have = group == 0 ? size[0] : group == 1 ? size[1] : size[2];
                    if (place - step >= stop) {
                        grow(place - step, wave - first_wave, list_waves, [&](int more) {
                            int at = 0;
                            if (more > 0) {
                                if (lane == 0) at = have + atomicAdd(&s.appended[step][group], more);
                                at = __builtin_amdgcn_readfirstlane(at);
                            }
                            return at;
                        });
                    }
                    __syncthreads();
        #pragma unroll
                    for (int l = 0; l < 3; ++l) {
                        size[l] += s.appended[step][l];
                        over = over || size[l] > (l == 0 ? kListQ : l == 1 ? kListP1 : kListP2);
                    }
                    if (over) break;
                }
                if (over) {
                    again = true;
                    break;
                }
                // Q: sorted by cells (a counting sort in place, by way of registers).
                for (int i = tid; i <= kCells / 2; i += kEnumThreads) s.list.begin[i] = 0;
                constexpr int kMine = (kListQ + kEnumThreads - 1) / kEnumThreads;
                int q_cell[kMine], q_loss[kMine], q_used[kMine];
                uint32_t q_mask[kMine];
                __syncthreads();
        #pragma unroll
                for (int x = 0; x < kMine; ++x) {
                    const int e = tid + x * kEnumThreads;
                    q_cell[x] = -1;
                    if (e < size[0]) {
                        const int use = s.list.q_use[e], ua = s.q_default[0] + use_a(use), ub = s.q_default[1] + use_b(use);
                        if (ua <= c0 && ub <= c1) {
                            const int cell = row_of(ua) + column_of(ub), half = (cell & 1) * 16;
                            q_cell[x] = (int)(atomicAdd(&s.list.begin[cell >> 1], 1u << half) >> half & 0xffffu) << 16 | cell;
                            q_loss[x] = s.list.q_loss[e];
                            q_used[x] = ua << 16 | ub;
                            q_mask[x] = s.list.q_mask[e];
                        }
                    }
                }
                __syncthreads();
                {
                    constexpr int kWords = kCells / 2 / kEnumThreads;
                    uint32_t word[kWords];
                    int sum = 0;
        #pragma unroll
                    for (int x = 0; x < kWords; ++x) {
                        word[x] = s.list.begin[tid * kWords + x];
                        sum += (int)(word[x] & 0xffffu) + (int)(word[x] >> 16);
                    }
                    int upto = sum;
        #pragma unroll
                    for (int off = 1; off < 64; off <<= 1) {
                        const int y = __shfl_up(upto, off);
                        if (lane >= off) upto += y;
                    }
                    if (lane == 63) s.wave_sum[wave] = upto;
                    __syncthreads();
                    int begin = upto - sum;
        #pragma unroll 1
                    for (int x = 0; x < wave; ++x) begin += s.wave_sum[x];
        #pragma unroll
                    for (int x = 0; x < kWords; ++x) {
                        const int lo = begin, hi = begin + (int)(word[x] & 0xffffu);
                        s.list.begin[tid * kWords + x] = (uint32_t)hi << 16 | (uint32_t)lo;
                        begin = hi + (int)(word[x] >> 16);
                    }
                    if (tid == kEnumThreads - 1) s.list.begin[kCells / 2] = (uint32_t)begin;
                }
                __syncthreads();
        #pragma unroll
                for (int x = 0; x < kMine; ++x) {
                    if (q_cell[x] >= 0) {
                        const int at = begin16[q_cell[x] & 0xffff] + (q_cell[x] >> 16);  // (its cell, and its place there)
                        s.list.q_loss[at] = q_loss[x];
                        s.list.q_use[at] = q_used[x];
                        s.list.q_mask[at] = q_mask[x];
                    }
                }
                __syncthreads();
                // What a partner loses at least, the room that it leaves included, where a pair leaves room in a cell: the least loss
                // in the cell, or in one below it plus the price of the room that is certainly left then.  16 bits, rounded
                // down.
                filtered = size[1] * size[2] >= kFilterPairs;
                if (filtered) {
                    constexpr int kRows = kCells0 / kEnumWaves, kFar = 0xffff;
                    const int one0 = min(l0 >> coarse, kFar), one1 = min(l1 >> coarse, kFar);
                    const int wide0 = (int)min(((long long)l0 << cell0) >> coarse, (long long)kFar);
                    const int wide1 = (int)min(((long long)l1 << cell1) >> coarse, (long long)kFar);
                    int row[kRows], last = kFar;
        #pragma unroll
                    for (int x = 0; x < kRows; ++x) {
                        const int cell = (wave * kRows + x) * kCells1 + lane, end = begin16[cell + 1];
                        int own = kNever;
                        for (int k = begin16[cell]; k < end; ++k) own = min(own, s.list.q_loss[k]);
                        own = min(own >> coarse, kFar);
                        int least_below = own - wide1 * lane;
        #pragma unroll
                        for (int off = 1; off < 64; off <<= 1) {
                            const int y = __shfl_up(least_below, off);
                            if (lane >= off) least_below = min(least_below, y);
                        }
                        const int below = __shfl_up(least_below + wide1 * lane, 1);
                        row[x] = lane > 0 ? min(own, below + one1) : own;
                        last = min(row[x], last + wide0);
                    }
                    s.edge[wave][lane] = last;
                    __syncthreads();
                    int below = kFar;
        #pragma unroll 1
                    for (int x = 0; x < wave; ++x) below = min(s.edge[x][lane], below + wide0 * kRows);
        #pragma unroll
                    for (int x = 0; x < kRows; ++x) {
                        s.list.least[wave * kRows + x][lane] = (uint16_t)min(row[x], min(below + one0, kFar));
                        below = min(row[x], below + wide0);
                    }
                    __syncthreads();
                }

            }

            // Pairs of P1 and P2 that some partner may suit: collected 64 at a time, then every lane looks its partners up.  If
            // this settles the matter but several selections are as good, once more, for the one whose choices, two
            // bits each with the last item's on top, make the smallest number.  (One loop for everything: the code is run
            // a few times, and fetching it is a good part of what that takes.)
            const int room0 = c0 - used0 + s.q_default[0], room1 = c1 - used1 + s.q_default[1];
            uint32_t *queue = s.list.queue[wave];
            const int chunks = (size[2] + 63) >> 6;
            if (pass == 1) {  // (in the place of what the table of least losses was made with)
                if (tid < 3 * 8 * 16) {
                    const int l = tid >> 7, at = tid >> 4 & 7, bits = tid & 15;
                    ulonglong2 flips = make_ulonglong2(0ull, 0ull);
        #pragma unroll
                    for (int b = 0; b < 4; ++b) {
                        if ((bits >> b & 1) != 0 && at * 4 + b < s.bits[l]) {
                            flips.x ^= s.flip_lo[l][at * 4 + b];
                            flips.y ^= s.flip_hi[l][at * 4 + b];
                        }
                    }
                    s.flips[l][at][bits] = flips;
                }
                __syncthreads();
            }
            if (part_loss <= cut) {
                int queued = 0;
                // a tile: sixteen of P1, one after the other, with 64 of P2
                int first1 = 0, chunk = wave, x = 16, i2 = 0, left0_2 = 0, left1_2 = 0, a1 = 0, b1 = 0, spare2 = 0, loss1 = 0;
                bool more = true;
                while (true) {
                    const int limit = min(min(known, best), *(volatile int32_t *)&s.least);  // no selection that loses more matters
                    if (more && queued < 64) {
                        if (x == 16) {
                            while (chunk >= chunks) chunk -= chunks, first1 += 16;
                            if (first1 >= size[1]) {
                                more = false;
                                continue;
                            }
                            i2 = chunk * 64 + lane;
                            chunk += kEnumWaves;
                            const int i1 = first1 + (lane & 15);
                            const int use2 = s.list.p2_use[i2], use1 = i1 < size[1] ? s.list.p1_use[i1] : 0;
                            left0_2 = room0 - use_a(use2), left1_2 = room1 - use_b(use2), a1 = use_a(use1), b1 = use_b(use1);
                            spare2 = i2 < size[2] ? __builtin_amdgcn_readfirstlane(limit) - s.list.p2_loss[i2] : -1;
                            loss1 = i1 < size[1] ? s.list.p1_loss[i1] : kNever;
                            // (first1 stays the tile's until chunk runs over)
                            x = 0;
                        }
                        bool valid[2];
                        int at_least[2], spare[2];
    #pragma unroll
                        for (int y = 0; y < 2; ++y) {
                            spare[y] = spare2 - __builtin_amdgcn_readlane(loss1, x + y);
                            const int left0 = left0_2 - __builtin_amdgcn_readlane(a1, x + y);
                            const int left1 = left1_2 - __builtin_amdgcn_readlane(b1, x + y);
                            valid[y] = (spare[y] | left0 | left1) >= 0;
                            at_least[y] = filtered ? (&s.list.least[0][0])[row_of(max(left0, 0)) + column_of(max(left1, 0))] : 0;
                        }
    #pragma unroll
                        for (int y = 0; y < 2; ++y) {
                            valid[y] = valid[y] && at_least[y] <= spare[y] >> coarse;
                            const unsigned long long mask = __ballot(valid[y]);
                            if (valid[y]) queue[queued + enum_below(mask, lane)] = (uint32_t)(first1 + x + y) << 11 | (uint32_t)i2;
                            queued += __popcll(mask);
                        }
                        __builtin_amdgcn_wave_barrier();
                        x += 2;
                        continue;
                    }
                    if (queued == 0) break;
                    const bool valid = lane < queued;
                    const uint32_t pair = queue[lane], rest = queue[64 + lane], rest2 = queue[128 + lane];
                    __builtin_amdgcn_wave_barrier();
                    queue[lane] = rest;
                    queue[64 + lane] = rest2;
                    queued = max(queued - 64, 0);
                    if (valid) {
                        const int p1 = pair >> 11, p2 = pair & 2047;
                        const int use = s.list.p1_use[p1] + s.list.p2_use[p2], loss = s.list.p1_loss[p1] + s.list.p2_loss[p2];
                        const int left0 = room0 - use_a(use), left1 = room1 - use_b(use), spare = limit - loss;
                        // room left on a link costs its price: no partner may leave more of it than what is spare pays for
                        const int slack0 = l0 > 0 ? (int)fminf((float)spare * per0, 65535.0f) + 1 : 65536;
                        const int slack1 = l1 > 0 ? (int)fminf((float)spare * per1, 65535.0f) + 1 : 65536;
                        const int to0 = row_of(left0), from1 = column_of(max(left1 - slack1, 0)), to1 = column_of(left1) + 1;
                        for (int row = spare >= 0 ? row_of(max(left0 - slack0, 0)) : kCells; row <= to0; row += kCells1) {
                            const int end = begin16[row + to1];
                            for (int k = begin16[row + from1]; k < end; ++k) {
                                const int its_loss = s.list.q_loss[k];
                                if (its_loss > spare) continue;
                                const int used = s.list.q_use[k], room_a = left0 - (used >> 16), room_b = left1 - (used & 0xffff);
                                if ((room_a | room_b | (slack0 - room_a) | (slack1 - room_b)) < 0) continue;
                                const long long more_lost = (long long)l0 * room_a + (long long)l1 * room_b + its_loss;
                                if (more_lost > spare) continue;
                                const int lost = loss + (int)more_lost;
                                if (pass == 0) {
                                    copies = lost < best ? 0 : lost == best ? 1 : copies;
                                    if (lost < best) chosen.q = 0, chosen.q_mask = s.list.q_mask[k], chosen.pair = pair, best = lost;
                                } else if (lost == least) {
                                    EnumResult other{0, s.list.q_mask[k], pair, s.default_lo, s.default_hi};
    #pragma unroll 1
                                    for (int l = 0; l < 3; ++l) {
                                        const uint32_t mask = enum_mask(s, l, pair, other.q_mask);
    #pragma unroll
                                        for (int at = 0; at < 8; ++at) {
                                            const ulonglong2 flips = s.flips[l][at][mask >> (at * 4) & 15];
                                            other.lo ^= flips.x;
                                            other.hi ^= flips.y;
                                        }
                                    }
                                    if (enum_before(other, chosen)) chosen = other;
                                }
                            }
                        }
                    }
                    if (late()) s.over = 1;
                    if (__builtin_amdgcn_readfirstlane(*(volatile int32_t *)&s.over)) break;
                }
                if (pass == 0 && best <= known) atomicMin(&s.least, best);
                __syncthreads();
                if (s.over) return;
            }
            if (++part < turns) continue;
            part = 0;
            if (pass == 1) break;
            least = s.least;
            if (least > G) break;
            // nothing is better, and nothing as good has not been met
            const int met = __popcll(__ballot(best == least)) + __popcll(__ballot(best == least && copies != 0));
            if (lane == 0) s.wave_sum[wave] = met;
            if (best == least) s.q_mask = chosen.q_mask, s.pair = chosen.pair;  // (whichever, where there are several)
            __syncthreads();
            int all = 0;
    #pragma unroll 4
            for (int w = 0; w < kEnumWaves; ++w) all += s.wave_sum[w];
            several = all > 1;
            if (!several) break;
            chosen.q = -1;
            best = least;
            pass = 1;
        }
        if (again) {
            retry(size[0] > kListQ);
            if (s.over) return;
            continue;
        }
        last_G = G;
        ++round;
        if (least <= G) {
            if (several) {
#pragma unroll 1
                for (int off = 1; off < 64; off <<= 1) {
                    EnumResult other;
                    other.q = __shfl_xor(chosen.q, off);
                    other.q_mask = __shfl_xor(chosen.q_mask, off);
                    other.pair = __shfl_xor(chosen.pair, off);
                    other.lo = __shfl_xor(chosen.lo, off);
                    other.hi = __shfl_xor(chosen.hi, off);
                    if (enum_before(other, chosen)) chosen = other;
                }
                if (lane == 0) s.result[wave] = chosen;
                __syncthreads();
                if (s.over) return;
                if (tid == 0) {
#pragma unroll 1
                    for (int w = 1; w < kEnumWaves; ++w)
                        if (enum_before(s.result[w], chosen)) chosen = s.result[w];
                    s.q_mask = chosen.q_mask;
                    s.pair = chosen.pair;
                }
                __syncthreads();
            }
            if (tid < kEnumOpen) s.choice[tid] = s.dflt[tid];
            if (tid < 4) s.sum[tid] = 0;
            __syncthreads();
            if (tid < 96) {
                const int l = tid >> 5, b = tid & 31;
                if (enum_mask(s, l, s.pair, s.q_mask) >> b & 1u) s.choice[s.meaning[l][b] >> 2] = (uint8_t)(s.meaning[l][b] & 3);
            }
            finish([&]() { return rank < kEnumOpen && loss_a < kNever ? (int)s.choice[rank] : dflt; });
            return;
        }
        __syncthreads();
    }
}

}  // namespace

}  // namespace deft
