// One stage (Problem 1 on one window) by enumeration of the selections that can be optimal, by one wavefront.
//
// For any price l >= 0 of capacity an item is worth v - l w taken and 0 left.  With  U = l C + sum of max(v - l w, 0),
// every selection of value V that fits has  U - V = (sum over the items it treats otherwise of |v - l w|) + l (room
// left).  So an item whose |v - l w| exceeds U - V is treated the same in every selection at least as good as one
// of value V, and those selections depart from that by a total loss of at most U - V.  At the price of the item at
// which the window runs over, U is usually so close to the optimum that a handful of items are open: of 148 GPT-2
// buckets with priorities 7 to 30, with 100 to 8000 selections to look at, where a row has 381000 cells for each item.
//
// The 64 items of least loss (the pool) are sorted by it.  A round opens those of loss up to G, deals them to two
// lists in turn and spells out, in LDS, every combination of either list of loss up to G; all pairs are looked at for
// the greatest value that fits.  If that loses no more than G, every selection as good or better has been met: it is
// the stage's value, and of several such the one with the smallest mask is the one that the DP's walk returns.
// Otherwise G grows, never beyond what the best selection met leaves.  Lists that run over end the attempt: the
// caller sweeps its row.
//
// All quantities that decide are whole numbers: losses in units of 2^-F, rounded down by `coarse` bits in the lists.
//
// Bound by latency: one wavefront works through a few thousand dependent steps.  GPT-2 windows in 1 us units (148
// items with priorities), us a stage, half of the stages and 97 of 100: price 2.2 and 2.3, losses and pool 4.5 and 4.9,
// lists 1 to 2 and 6 to 10, pairs 4 and 16; the sweep of the same stage takes 2000.  Six items of a list are spelled
// out at once, a subset for every lane (a step for each of them: 4 us instead of 1); the price and the pool are found
// by three candidates at a time from registers (by one from LDS: 4 and 5 us instead of 2 and 4).
#pragma once

#include <limits.h>

#include "kernels.h"

namespace deft {

namespace {

constexpr int kPool = 64;
constexpr int kPoolRounds = 7;   // 12, 20, ... 60 open items
constexpr int kPoolNever = 1 << 30;
constexpr int kPoolFirst = 1024; // the longest list before heavy items are gone through one by one
constexpr int kPoolBins = 256;
constexpr int kPoolSort = 6144;  // the fewest pairs that make it worth sorting one list by weight
// Where an attempt ends early, so that what it cannot settle costs little on top of the sweep.  Values unrelated to
// weights or priorities times them, 148 items on a long row: at most 2 items within one unit of value of the price, 4
// selections as good as the best a stage.  Values of a few kinds: up to 64 of the pool and 39000 selections, gone
// through one by one (128 instances of 60 items, C = 60000, the sweep 0.38 ms: 28.8 ms, now 0.39; values 1 to 3, 256 of 100, C = 100000,
// 0.88 ms: 7.9, now 0.89; values within 2 of the weights, 128 of 60 0.40 ms: 2.9, now 0.41).
constexpr int kPoolAlike = 16;   // REDUCE = false: with more items within one unit too many selections are as good
// REDUCE: a stage whose items are mostly within one unit is reduced to hardly fewer, at 12 to 25 us.  Given up with two thirds
// of them, in stages of fewer cells with half (values within 2 of the weights, 256 instances of 96 items, C = 7000: the sweep 112 us,
// tried 162, now 114; 16 of 148, C = 38000 511, 602, now 518; values 1 to 3, about half within one unit, 16 of 148, C = 38000
// 478, 174 without these limits, now 211).
constexpr long long kPoolHope = 2400000;
constexpr int kPoolTies = 16;    // more selections of the greatest value (0.4 us each)
constexpr int kPoolSteps = 2048; // more steps through the fullest bin (40 ns each)

// What a stage needs: the items' weights and values (64 at a time, padded), and space for their losses, the pool and lists.
constexpr int kPoolEntryBytes = 16;
__host__ __device__ constexpr int pool_items_bytes(int n) { return (n + 63) / 64 * 64 * 8; }
__host__ __device__ constexpr int pool_space_bytes(int n, int entries) { return (n + 63) / 64 * 64 * 4 + 8 * (kPoolBins + 4) + 3 * entries * kPoolEntryBytes; }

template <class Op>
__device__ __forceinline__ int pool_reduce(int x, Op op)
{
    x = op(x, __builtin_amdgcn_update_dpp(x, x, 0xB1, 0xf, 0xf, false));   // quad_perm [1,0,3,2]
    x = op(x, __builtin_amdgcn_update_dpp(x, x, 0x4E, 0xf, 0xf, false));   // quad_perm [2,3,0,1]
    x = op(x, __builtin_amdgcn_update_dpp(x, x, 0x124, 0xf, 0xf, false));  // row_ror:4
    x = op(x, __builtin_amdgcn_update_dpp(x, x, 0x128, 0xf, 0xf, false));  // row_ror:8
    return op(op(__builtin_amdgcn_readlane(x, 0), __builtin_amdgcn_readlane(x, 16)),
              op(__builtin_amdgcn_readlane(x, 32), __builtin_amdgcn_readlane(x, 48)));
}
__device__ __forceinline__ int pool_sum(int x) { return pool_reduce(x, [](int a, int b) { return a + b; }); }
__device__ __forceinline__ int pool_max(int x) { return pool_reduce(x, [](int a, int b) { return max(a, b); }); }
__device__ __forceinline__ float pool_sum(float x)
{
    return __int_as_float(pool_reduce(__float_as_int(x), [](int a, int b) { return __float_as_int(__int_as_float(a) + __int_as_float(b)); }));
}
// Three sums side by side: a chain of eight dependent steps once instead of three times.
__device__ __forceinline__ void pool_sums(float &x, float &y, float &z)
{
#define DEFT_POOL_STEP(CTRL)                                                                                              \
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, false));                        \
    y += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(y), CTRL, 0xf, 0xf, false));                        \
    z += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(z), CTRL, 0xf, 0xf, false));
    DEFT_POOL_STEP(0xB1)   // quad_perm [1,0,3,2]
    DEFT_POOL_STEP(0x4E)   // quad_perm [2,3,0,1]
    DEFT_POOL_STEP(0x124)  // row_ror:4
    DEFT_POOL_STEP(0x128)  // row_ror:8
#undef DEFT_POOL_STEP
    auto rows = [](float a) {
        const int i = __float_as_int(a);
        return (__int_as_float(__builtin_amdgcn_readlane(i, 0)) + __int_as_float(__builtin_amdgcn_readlane(i, 16))) +
               (__int_as_float(__builtin_amdgcn_readlane(i, 32)) + __int_as_float(__builtin_amdgcn_readlane(i, 48)));
    };
    x = rows(x), y = rows(y), z = rows(z);
}
__device__ __forceinline__ int pool_below(unsigned long long mask, int lane) { return __popcll(mask & ((1ull << lane) - 1ull)); }
__device__ __forceinline__ void pool_sync()
{
    // one wavefront: LDS executes its instructions in order; only the compiler has to be kept from reordering
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// The stage's answer: its value, its weight, and the items taken (bit c of lane l: item 64 c + l).
struct PoolAnswer {
    int value, load;
    unsigned long long chosen;
    unsigned long long open;  // kPoolReduced: the items that are still to be decided; the others are as in `chosen`
};

// `offered`, laid out like `chosen`: the items that are open, fit at all (w <= C) and are worth something (v > 0);
// together they weigh more than C.  `items`: weight and value of item i, whole chunks of 64.  `space`: `space_bytes`
// of LDS, 16-byte aligned.  `entries`: how long the lists may get.
// `least_value`: only selections of that value or more matter.
// `deadline`: no round begins after it (by the wall clock).
// REDUCE: where lists run over but a selection is known, the stage is reduced to the items that it leaves open.
// kPoolHopeless: nor will it be settled with some of the items given.
enum PoolOutcome { kPoolHopeless, kPoolFailed, kPoolNone, kPoolFound, kPoolReduced };
template <bool REDUCE>
__device__ __forceinline__ PoolOutcome pool_stage(const int2 *items, char *space, int space_bytes, int entries, int n, int C,
                                                  unsigned long long offered, int least_value, long long deadline, int lane, PoolAnswer &answer)
{
    const int chunks = (n + 63) >> 6;
    // losses as floats, negative where the item is worth taking; in front of the lists
    int *const loss_of = reinterpret_cast<int *>(space);
    int *const begin = loss_of + chunks * 64, *const top = begin + kPoolBins + 4;  // of the bins
    int4 *const list_a = reinterpret_cast<int4 *>(top + kPoolBins + 4);
    entries = min(entries, (space_bytes - pool_space_bytes(n, 0)) / (3 * kPoolEntryBytes));
    if (entries < kPool) return kPoolFailed;  // (the pool itself lies there first)
    int4 *const list_b = list_a + entries, *const spare = list_b + entries;
    auto is_offered = [&](int c) { return ((offered >> c) & 1ull) != 0; };

    // ---- the price: the least at which what is worth taking fits, to one part in 2^13 --------------------
    // (the first chunks stay in registers)
    constexpr int kHeld = 4;
    float w_held[kHeld], v_held[kHeld];
    float most = 0.0f, fewest = INFINITY;
#pragma unroll
    for (int c = 0; c < kHeld; ++c) {
        const bool in = c < chunks && is_offered(c);
        const int2 it = items[c < chunks ? c * 64 + lane : lane];
        w_held[c] = in ? (float)it.x : 0.0f;
        v_held[c] = in ? (float)it.y : 0.0f;
        const float ratio = (float)it.y / (float)it.x;
        if (in) most = fmaxf(most, ratio), fewest = fminf(fewest, ratio);
    }
    for (int c = kHeld; c < chunks; ++c) {
        const int2 it = items[c * 64 + lane];
        const float ratio = (float)it.y / (float)it.x;
        if (is_offered(c)) most = fmaxf(most, ratio), fewest = fminf(fewest, ratio);
    }
    // (floats above 0 are ordered like their bits)
    int hi = pool_max(__float_as_int(most)), lo = max(pool_reduce(__float_as_int(fewest), [](int a, int b) { return min(a, b); }) - 1, 0);
    while (hi - lo > 1 << 10) {
        const int step = (hi - lo) >> 2;
        const float p1 = __int_as_float(lo + step), p2 = __int_as_float(lo + 2 * step), p3 = __int_as_float(lo + 3 * step);
        float s1 = 0.0f, s2 = 0.0f, s3 = 0.0f;
        auto add = [&](float w, float v) {
            s1 += v > p1 * w ? w : 0.0f;
            s2 += v > p2 * w ? w : 0.0f;
            s3 += v > p3 * w ? w : 0.0f;
        };
#pragma unroll
        for (int c = 0; c < kHeld; ++c) add(w_held[c], v_held[c]);
        for (int c = kHeld; c < chunks; ++c) {
            const int2 it = items[c * 64 + lane];
            add(is_offered(c) ? (float)it.x : 0.0f, (float)it.y);
        }
        pool_sums(s1, s2, s3);
        const float room = (float)C;
        const int quarter = s1 <= room ? 1 : s2 <= room ? 2 : s3 <= room ? 3 : 4;
        if (quarter < 4) hi = lo + quarter * step;
        lo += (quarter - 1) * step;
    }
    const float rate = __int_as_float(hi);
    if (rate <= 0.0f) return kPoolFailed;
    const int F = min(max(20 - (((hi >> 23) & 255) - 127), 0), 30);
    const long long price = (long long)ceilf(ldexpf(rate, F));

    // ---- losses -----------------------------------------------------------------------------------
    int weight = 0, worth = 0, count = 0, alike = 0, greatest = 0;
    float weight_f = 0.0f;
    for (int c = 0; c < chunks; ++c) {
        const int2 it = items[c * 64 + lane];
        const long long x = ((long long)it.y << F) - price * it.x;
        const bool in = is_offered(c), take = in && x > 0;
        const float loss = (float)(x > 0 ? x : -x);
        weight += take ? it.x : 0;
        worth += take ? it.y : 0;
        weight_f += take ? (float)it.x : 0.0f;
        loss_of[c * 64 + lane] = __float_as_int(take ? -loss : loss);
        greatest = max(greatest, in ? __float_as_int(loss) : 0);
        count += __popcll(__ballot(in));
        alike += __popcll(__ballot(in && loss <= ldexpf(1.0f, F)));
    }
    if (REDUCE ? alike * ((long long)count * C < kPoolHope ? 4 : 3) > count * 2 : alike > kPoolAlike) return kPoolHopeless;
    if (pool_sum(weight_f) > 1.0e9f) return kPoolFailed;
    weight = pool_sum(weight);
    worth = pool_sum(worth);
    const int room = C - weight;
    const long long unused = price * room;  // what the selection of all that is worth taking loses

    // ---- the pool: the items of least loss, those of loss up to the float `limit` --------------------------
    int limit = 0x7f800000;
    if (count > kPool) {
        int held_loss[kHeld];
#pragma unroll
        for (int c = 0; c < kHeld; ++c) held_loss[c] = c < chunks && is_offered(c) ? loss_of[c * 64 + lane] & 0x7fffffff : INT_MAX;
        greatest = pool_max(greatest);
        // (first 1 / 2^12, 1 / 2^6 and 1 / 2^3 of the greatest loss)
        int below = -1, above = limit, m1 = max(greatest - (12 << 23), 0), m2 = max(greatest - (6 << 23), 0), m3 = max(greatest - (3 << 23), 0);
        while (above - below > 1) {
            int h1 = 0, h2 = 0, h3 = 0;
            auto add = [&](int f) {
                h1 += __popcll(__ballot(f <= m1));
                h2 += __popcll(__ballot(f <= m2));
                h3 += __popcll(__ballot(f <= m3));
            };
#pragma unroll
            for (int c = 0; c < kHeld; ++c) add(held_loss[c]);
            for (int c = kHeld; c < chunks; ++c) add(is_offered(c) ? loss_of[c * 64 + lane] & 0x7fffffff : INT_MAX);
            if (h1 > kPool) {
                above = m1;
            } else {
                below = h3 <= kPool ? m3 : h2 <= kPool ? m2 : m1;
                if (h3 > kPool) above = h2 > kPool ? m2 : m3;
                if ((h3 <= kPool ? h3 : h2 <= kPool ? h2 : h1) >= kPool * 7 / 8) break;
            }
            const int step = above - below < 4 ? 1 : (int)((unsigned)(above - below) >> 2);
            m1 = below + step, m2 = min(m1 + step, above - 1), m3 = min(m2 + step, above - 1);
        }
        if (below < 0) return kPoolFailed;
        limit = below;
    }
    int held = 0;
    for (int c = 0; c < chunks; ++c) {
        const int f = loss_of[c * 64 + lane];
        const bool in = is_offered(c) && (f & 0x7fffffff) <= limit;
        const unsigned long long mask = __ballot(in);
        const int at = held + pool_below(mask, lane);
        if (in) {
            const int2 it = items[c * 64 + lane];
            list_a[at] = make_int4(it.x, it.y, c * 64 + lane, f);
        }
        held += __popcll(mask);
    }
    pool_sync();
    const bool mine = lane < held;
    const int4 own = list_a[lane];
    const int longest = pool_max(mine ? own.w & 0x7fffffff : 0);
    const int coarse = max(((longest >> 23) & 255) - 127 + 1 - 29, 0);  // losses in 30 bits
    const bool taken = mine && own.w < 0;
    int loss = kPoolNever;
    if (mine) {
        const long long x = ((long long)own.y << F) - price * own.x;
        loss = (int)((x > 0 ? x : -x) >> coarse);
    }
    // an item outside loses more than `limit`
    const int G_pool = limit == 0x7f800000 ? kPoolNever - 1
                                           : (int)min((long long)kPoolNever - 1, ((long long)__int_as_float(limit) >> coarse) - 1);
    const unsigned long long taken_mask = __ballot(taken);
    int rank = 0;
    for (int j = 0; j < held; ++j) {
        const int other = __builtin_amdgcn_readlane(loss, j);
        rank += other < loss || (other == loss && j < lane) ? 1 : 0;
    }
    if (!mine) rank = lane;
    // sorted: change of weight and value when the item is treated otherwise; its place in the pool (by index)
    const int s_loss = __builtin_amdgcn_ds_permute(rank * 4, loss);
    const int s_weight = __builtin_amdgcn_ds_permute(rank * 4, taken ? -own.x : own.x);
    const int s_value = __builtin_amdgcn_ds_permute(rank * 4, taken ? -own.y : own.y);
    const int s_place = __builtin_amdgcn_ds_permute(rank * 4, lane);
    const int index = own.z;
    pool_sync();

    // ---- rounds --------------------------------------------------------------------------------
    // what the best selection met so far loses, or one of the least value that matters
    long long least = least_value < 0 ? 1ll << 62 : unused - ((long long)(least_value - worth) << F);
    if (least < 0) return kPoolNone;
    int last_G = -1;
    bool may_leap = true;
    for (int round = 0; round <= kPoolRounds && wall_clock64() < deadline;) {
        const int opened = 12 + 8 * round;
        int G = min(opened < held ? __builtin_amdgcn_readlane(s_loss, min(opened, 63)) - 1 : kPoolNever - 1, G_pool);
        const int left = (int)min(least >> coarse, (long long)kPoolNever);
        const bool leap = may_leap && left > G && left <= G_pool;
        if (leap || left <= G) G = left;
        if (G <= last_G) {
            if (G >= G_pool) break;
            ++round;
            continue;
        }
        const int open = __popcll(__ballot(s_loss <= G));
        // every other item to either list, the greatest losses first (they combine with little)
        // six items of either list at once, a subset for every lane
        const int count_a = (open + 1) >> 1, count_b = open >> 1;
        auto seed = [&](int4 *list, int l, int count_l) {
            const int used = min(6, count_l);
            int4 x = make_int4(0, 0, 0, 0);
            for (int t = 0; t < used; ++t) {
                const int p = count_l - 1 - t, at = 2 * p + l;
                const int x_loss = __builtin_amdgcn_readlane(s_loss, at), x_weight = __builtin_amdgcn_readlane(s_weight, at);
                const int x_value = __builtin_amdgcn_readlane(s_value, at);
                if ((lane >> t) & 1) x = make_int4(x.x + x_weight, x.y + x_value, min(x.z + x_loss, kPoolNever), x.w | (int)(1u << p));
            }
            const bool ok = lane < 1 << used && x.z <= G;
            const unsigned long long with = __ballot(ok);
            if (ok) list[pool_below(with, lane)] = x;
            return (int)__popcll(with);
        };
        pool_sync();
        int size_a = seed(list_a, 0, count_a), size_b = seed(list_b, 1, count_b);
        bool over = false;
        for (int p = count_a - 7; p >= 0 && !over; --p) {
            pool_sync();
            const bool both = p < count_b - 6;
            // (the first chunks of either list at once: most lists are no longer)
            const int4 first_a = list_a[min(lane, size_a - 1)], first_b = list_b[min(lane, size_b - 1)];
            auto grow = [&](int4 *list, int size, int at, int4 x) {
                const int x_loss = __builtin_amdgcn_readlane(s_loss, at), x_weight = __builtin_amdgcn_readlane(s_weight, at);
                const int x_value = __builtin_amdgcn_readlane(s_value, at);
                int next = size;
                for (int base = 0; base < size; base += 64) {
                    const int e = base + lane;
                    if (base > 0) x = list[min(e, size - 1)];
                    const bool ok = e < size && x.z <= G - x_loss;
                    const unsigned long long mask = __ballot(ok);
                    const int to = next + pool_below(mask, lane);
                    if (ok && to < entries) list[to] = make_int4(x.x + x_weight, x.y + x_value, x.z + x_loss, x.w | (int)(1u << p));
                    next += __popcll(mask);
                }
                over = over || next > entries;
                return next;
            };
            size_a = grow(list_a, size_a, 2 * p, first_a);
            if (both) size_b = grow(list_b, size_b, 2 * p + 1, first_b);
        }
        if (over) {
            if (!leap || REDUCE) break;
            may_leap = false;
            continue;
        }
        last_G = G;
        ++round;
        pool_sync();
        // The greatest value of a pair that fits; then, if that settles the stage, the pairs of that value: the one with
        // the smallest mask.  With long lists, the second one's partners of an item of the first are not gone through one by one:
        // they are sorted into bins by weight, with the greatest value of all bins below; what is left is the one bin at
        // the limit.
        const bool sorted = size_a * size_b >= kPoolSort;
        const int4 *partners = list_b;
        int lightest = 0;
        float scale = 0.0f;
        int fullest = 0;
        auto bin_of = [&](int w) { return (int)fminf((float)(w - lightest) * scale, (float)(kPoolBins - 1)); };
        if (sorted) {
            int least_w = INT_MAX, most_w = INT_MIN;
            for (int base = 0; base < size_b; base += 64) {
                const int w = list_b[min(base + lane, size_b - 1)].x;
                least_w = min(least_w, w);
                most_w = max(most_w, w);
            }
            lightest = pool_reduce(least_w, [](int a, int b) { return min(a, b); });
            scale = (float)kPoolBins / ((float)(pool_max(most_w) - lightest) + 1.0f);
            for (int b = lane; b <= kPoolBins; b += 64) begin[b] = 0, top[b] = INT_MIN;
            pool_sync();
            for (int base = 0; base < size_b; base += 64) {
                if (base + lane < size_b) {
                    const int2 x = *reinterpret_cast<const int2 *>(&list_b[base + lane]);
                    const int b = bin_of(x.x);
                    atomicAdd(&begin[b], 1);
                    atomicMax(&top[b], x.y);
                }
            }
            pool_sync();
            // bin b: where it begins, and the greatest value below it (four bins a lane)
            int4 counts = *reinterpret_cast<const int4 *>(&begin[lane * 4]), tops = *reinterpret_cast<const int4 *>(&top[lane * 4]);
            const int own_count = counts.x + counts.y + counts.z + counts.w, own_top = max(max(tops.x, tops.y), max(tops.z, tops.w));
            fullest = pool_max(max(max(counts.x, counts.y), max(counts.z, counts.w)));
            int upto = own_count, best_upto = own_top;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int x = __shfl_up(upto, off), y = __shfl_up(best_upto, off);
                if (lane >= off) upto += x, best_upto = max(best_upto, y);
            }
            const int before = __shfl_up(best_upto, 1), above = lane == 0 ? INT_MIN : before;
            const int4 begins = make_int4(upto - own_count, upto - own_count + counts.x, upto - counts.z - counts.w, upto - counts.w);
            *reinterpret_cast<int4 *>(&begin[lane * 4]) = begins;
            const int top1 = max(above, tops.x), top2 = max(top1, tops.y);
            *reinterpret_cast<int4 *>(&top[lane * 4]) = make_int4(above, top1, top2, max(top2, tops.z));
            if (lane == 63) begin[kPoolBins] = upto, top[kPoolBins] = best_upto;
            pool_sync();
            for (int base = 0; base < size_b; base += 64) {
                if (base + lane < size_b) {
                    const int4 x = list_b[base + lane];
                    spare[atomicAdd(&begin[bin_of(x.x)], 1)] = x;  // (a bin's beginning moves to its end, the next one's beginning)
                }
            }
            pool_sync();
            partners = spare;
        }
        if (fullest * ((size_a + 63) >> 6) > kPoolSteps) break;
        int best = INT_MIN, load = 0, ties = 0;
        bool met = false;
        unsigned long long mask = 0;
#pragma unroll 1
        for (int pass = 0; pass < 2; ++pass) {
            for (int base = 0; base < size_a; base += 64) {
                const int4 x = list_a[min(base + lane, size_a - 1)];
                const int x_room = room - x.x;
                int partner = INT_MIN;  // the greatest value of a partner
                if (sorted) {
                    if (x_room >= lightest) {
                        const int b = bin_of(x_room), end = begin[b];
                        partner = top[b];
                        for (int k = b > 0 ? begin[b - 1] : 0; k < end; ++k) {
                            const int2 y = *reinterpret_cast<const int2 *>(&partners[k]);
                            partner = max(partner, y.x <= x_room ? y.y : INT_MIN);
                        }
                    }
                } else {
                    for (int first = 0; first < size_b; first += 64) {
                        const int2 y = *reinterpret_cast<const int2 *>(&list_b[min(first + lane, size_b - 1)]);
                        const int end = min(64, size_b - first);
                        for (int j = 0; j < end; ++j)
                            partner = max(partner, __builtin_amdgcn_readlane(y.x, j) <= x_room ? __builtin_amdgcn_readlane(y.y, j) : INT_MIN);
                    }
                }
                const int both = partner == INT_MIN ? INT_MIN : x.y + partner;
                if (pass == 0) {
                    best = max(best, both);
                    continue;
                }
                for (unsigned long long hits = __ballot(both == best && base + lane < size_a); hits && ties <= kPoolTies; hits &= hits - 1) {
                    const int i = __builtin_ctzll(hits);
                    const int i_room = __builtin_amdgcn_readlane(x_room, i), i_value = best - __builtin_amdgcn_readlane(x.y, i);
                    unsigned long long one = taken_mask;
                    for (unsigned bits = (unsigned)__builtin_amdgcn_readlane(x.w, i); bits; bits &= bits - 1)
                        one ^= 1ull << __builtin_amdgcn_readlane(s_place, 2 * __builtin_ctz(bits));
                    for (int first = 0; first < size_b; first += 64) {
                        const int4 y = partners[min(first + lane, size_b - 1)];
                        for (unsigned long long with = __ballot(first + lane < size_b && y.x <= i_room && y.y == i_value); with && ties <= kPoolTies; with &= with - 1) {
                            const int j = __builtin_ctzll(with);
                            unsigned long long other = one;
                            for (unsigned bits = (unsigned)__builtin_amdgcn_readlane(y.w, j); bits; bits &= bits - 1)
                                other ^= 1ull << __builtin_amdgcn_readlane(s_place, 2 * __builtin_ctz(bits) + 1);
                            if (!met || other < mask) mask = other, load = C - i_room + __builtin_amdgcn_readlane(y.x, j);
                            met = true;
                            ++ties;
                        }
                    }
                }
            }
            if (pass == 0) {
                best = pool_max(best);
                if (best != INT_MIN) least = min(least, unused - ((long long)best << F));
                if ((least >> coarse) > G) break;
                if (best == INT_MIN || unused - ((long long)best << F) != least) return kPoolNone;  // none is worth that much
            }
        }
        if (!met) {
            if (G >= G_pool) break;
            continue;
        }
        if (ties > kPoolTies) break;
        answer.value = worth + best;
        answer.load = load;
        unsigned long long chosen = 0;
        for (int c = 0; c < chunks; ++c)
            if (is_offered(c) && loss_of[c * 64 + lane] < 0) chosen |= 1ull << c;
        for (unsigned long long other = mask ^ taken_mask; other; other &= other - 1) {
            const int i = __builtin_amdgcn_readlane(index, __builtin_ctzll(other));
            if (lane == (i & 63)) chosen ^= 1ull << (i >> 6);
        }
        answer.chosen = chosen;
        return kPoolFound;
    }
    if (!REDUCE || least >= 1ll << 62) return kPoolFailed;
    // What loses more than the selection known is treated the same in every one as good.
    const int open_limit = __float_as_int((float)least * (1.0f + 0x1p-22f));  // (rounding included)
    unsigned long long chosen = 0, open_items = 0;
    int load = 0, value = 0;
    for (int c = 0; c < chunks; ++c) {
        const int f = loss_of[c * 64 + lane];
        const int2 it = items[c * 64 + lane];
        if (!is_offered(c)) continue;
        if ((f & 0x7fffffff) <= open_limit) {
            open_items |= 1ull << c;
        } else if (f < 0) {
            chosen |= 1ull << c;
            load += it.x;
            value += it.y;
        }
    }
    answer = PoolAnswer{pool_sum(value), pool_sum(load), chosen, open_items};
    return kPoolReduced;
}

// A selection's items as numbers to compare: whether x comes before y (the last item that one of them alone takes is
// y's).
__device__ __forceinline__ bool pool_before(unsigned long long x, unsigned long long y, int lane)
{
    const unsigned long long differs = x ^ y;
    const int at = differs ? (63 - __builtin_clzll(differs)) * 64 + lane : -1, last = pool_max(at);
    return __ballot(at == last && at >= 0 && ((y >> (last >> 6)) & 1ull) != 0) != 0ull;
}

// The stage as a whole; `offered`: the items that are open and worth something.  Where a few heavy items leave the bound far from the optimum (three buckets that hold 85 % of
// the time: the window's last quarter is not one any of them fits), all combinations of the heaviest ones are gone through,
// each with a price of its own.
__device__ __forceinline__ bool pool_solve(const int2 *items, char *space, int space_bytes, int entries, int n, int C,
                                           unsigned long long offered, long long deadline, int lane, PoolAnswer &answer)
{
    constexpr int kHeavy = 3;
    unsigned long long rest = offered, pick[kHeavy] = {};
    int pick_w[kHeavy] = {}, pick_v[kHeavy] = {};
    answer = PoolAnswer{-1, 0, 0, 0};
#pragma unroll 1
    for (int sub = -1; sub < 1 << kHeavy; ++sub) {
        unsigned long long taken = 0;
        int weight = 0, value = 0;
        if (sub == 0) {
            for (int t = 0; t < kHeavy; ++t) {
                int heaviest = 0, chunk = 0;
                for (int c = 0; c < (n + 63) >> 6; ++c) {
                    const int w = ((rest >> c) & 1ull) != 0 ? items[c * 64 + lane].x : 0;
                    if (w > heaviest) heaviest = w, chunk = c;
                }
                const int w = pool_max(heaviest);
                if (w == 0) return false;
                const int l = __builtin_ctzll(__ballot(heaviest == w)), i = __builtin_amdgcn_readlane(chunk, l) * 64 + l;
                const unsigned long long bit = lane == l ? 1ull << (i >> 6) : 0ull;
                rest &= ~bit;
#pragma unroll
                for (int u = 0; u < kHeavy; ++u)
                    if (u == t) pick[u] = bit, pick_w[u] = w, pick_v[u] = __builtin_amdgcn_readfirstlane(items[i].y);
            }
        }
        if (sub >= 0) {
            long long sum = 0;
#pragma unroll
            for (int t = 0; t < kHeavy; ++t)
                if ((sub >> t) & 1) taken |= pick[t], sum += pick_w[t], value += pick_v[t];
            if (sum > C) continue;
            weight = (int)sum;
        }
        // what is left of the window, and of the list
        const int room = C - weight;
        unsigned long long fits = 0;
        int its_weight = 0, its_value = 0;
        constexpr int kOver = (1 << 24) + 1;  // (above every capacity; a lane has at most 64 items)
        for (int c = 0; c < (n + 63) >> 6; ++c) {
            const int2 it = items[c * 64 + lane];
            if (((rest >> c) & 1ull) != 0 && it.x <= room) fits |= 1ull << c, its_weight += it.x, its_value += it.y;
        }
        if (sub < 0) rest = fits;
        PoolAnswer part{0, pool_sum(min(its_weight, kOver)), fits, 0};
        if (part.load <= room) {
            part.value = pool_sum(its_value);
        } else {
            const PoolOutcome outcome = pool_stage<false>(items, space, space_bytes, sub < 0 ? min(entries, kPoolFirst) : entries, n, room, fits,
                                                   answer.value < 0 ? -1 : answer.value - value, deadline, lane, part);
            if (outcome == kPoolHopeless || (outcome == kPoolFailed && sub >= 0)) return false;
            if (outcome == kPoolFailed) continue;
            if (outcome == kPoolNone) continue;
        }
        part.value += value;
        part.load += weight;
        part.chosen |= taken;
        if (part.value > answer.value || (part.value == answer.value && pool_before(part.chosen, answer.chosen, lane))) answer = part;
        if (sub < 0) return true;
    }
    return true;
}

}  // namespace

}  // namespace deft
