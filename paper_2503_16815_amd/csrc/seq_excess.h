// One stage of a subset-sum problem by what it leaves out.  Included by seq_bits_kernel.h.
//
// The row's sweep and walk (seq_bits_kernel.h) return, where the capacity C itself can be reached, the items of the
// shortest prefix of the list that reaches it, less what can be spared of them from the end of the list on:
//   C is reachable with items 0 .. p exactly when their weight less C, the excess E, is the weight of some items
//   among them; for the least such p item p itself stays (else the items before it reached C already);
//   going down from p, the walk leaves item i out exactly when what then remains of the excess can be left out of the
//   items before i (of two selections of one value the one without the later item has the smaller mask).
// So the sums 0 .. E answer the stage, and E is less than the weight of the item that takes the list's weight
// past C: some hundreds where the row has ten thousand cells.  An item heavier than every sum still missing adds none,
// so that a stage is through after some light items, most others passed over by a ballot (4096
// ResNet-101-shaped schedules: 15 items a stage, where the row's sweep goes through 150 of up to seven words a lane each).
//
// What bounds it: one wavefront's chain of scalar instructions, 17 an item, and of the ballots and DPP sums over the
// list, 64 items each; it moves nothing but the list in LDS.
//
// The list is handed over as a function: list(first item, a multiple of 64) is the weight of the lane's item among
// those 64, kGone where it is not in the list any more (or beyond its end).
#pragma once

namespace deft {

namespace {

constexpr int kGone = 0x7fffffff;    // the weight of an item that is not in the list any more
constexpr int kExcessCells = 2048;   // sums the wide set holds: a word a lane
// Fewer items up to C than this have few light ones, and the row's sweep is as quick.  Where C is not reachable with items
// 0 .. p the next p is tried, six in all (that costs little where the 64 lowest sums say so).
constexpr int kExcessFewest = 48, kExcessTries = 6;
// Windows from which on what the 64 lowest sums and the run in the items' order do not show is looked for further (the runs
// lightest first, the wide set): below, the row's own sweep is as quick.
constexpr int kExcessThorough = 2048;
// And not where the excess is more than three quarters of the window and fewer items than this come before it: there it is mostly a list of
// heavy items, what is looked for further is not found, and takes as long as the row's sweep.  Forty inputs each, looked for always,
// up to half of the window or from 160 items on, and so, us in the geometric mean: 4096 ResNet-101-shaped schedules 46.0, 45.9, 43.5; task queues 125.9,
// 127.7, 122.4; 1500 lists of 140 items (Algorithm 1) with windows of 8000 cells 26.7, 28.3, 26.1, of 11700 cells 37.0, 34.0, 34.0; of 240
// items in two windows 35.0, 34.8, 33.0.  A capacity sweep looks in any case, for it would sweep at the largest capacity for all of them
// (454 lists of 348 items, two capacities from 3748 on: 22 us, 43 otherwise).
constexpr int kExcessMany = 140;

enum ExcessResult { kExcessEmpty, kExcessDone, kExcessNot };
enum ExcessAnswer { kExcessYes, kExcessNo, kExcessUnsure };

// Which items are spared: lane c holds the mask of items 64 c .. 64 c + 63.
struct ExcessSpared {
    uint32_t lo, hi;
};

__device__ __forceinline__ void excess_spare(ExcessSpared &x, int lane, int chunk, unsigned long long mask)
{
    x.lo |= lane == chunk ? (uint32_t)mask : 0u;
    x.hi |= lane == chunk ? (uint32_t)(mask >> 32) : 0u;
}

// The 64 sums 0 .. 63 in a scalar register pair, first[] a lane each: an item is a scalar shift and or, one select
// and the search for the greatest sum that is missing.  Beyond 63 a run shows what is reachable: once 32 .. 63 all are, an
// item of weight up to 32 makes it 32 .. 63 + w, and so on, as many items at a time as the run is long.  Where the run by the
// items in their order is too short for a question of the walk, the runs of up to 64 parts of the list are grown by
// weight, lightest items first, which makes them as long as they get.  What that does not show either is left open
// (kExcessUnsure), with the walk as far as it came: E is what is left, `limit` the item to go on below.
template <class List>
__device__ __forceinline__ ExcessAnswer excess_narrow(List &&list, int lane, int C, bool thorough, int &limit, int &E, ExcessSpared &spared)
{
    const unsigned long long mask = E >= 63 ? ~0ull : (2ull << E) - 1ull;
    unsigned long long set = 1ull;
    int first = lane == 0 ? -1 : kGone;  // the item that made the sum `lane` reachable (-1: the empty sum)
    int missing = min(min(63, E), C);    // no item above this adds one of the 64 sums
    for (int i0 = 0; i0 < limit && missing > 0; i0 += 64) {
        const int w_ = list(i0), w = i0 + lane < limit ? w_ : kGone;
        unsigned long long in = __builtin_amdgcn_ballot_w64(w <= missing);
        if (in == 0ull) continue;
        do {
            const int b = __builtin_ctzll(in);
            const int wt = __builtin_amdgcn_readlane(w, b);
            const unsigned long long fresh = (set << wt) & ~set;
            set |= fresh;
            first = __builtin_amdgcn_inverse_ballot_w64(fresh) ? i0 + b : first;
            const unsigned long long holes = mask & ~set;
            missing = holes != 0ull ? min(C, 63 - (int)__builtin_clzll(holes)) : 0;
            in = __builtin_amdgcn_ballot_w64(w <= missing) & (~1ull << b);
        } while (in != 0ull);
    }
    if (E <= 63 && ((set >> E) & 1ull) == 0ull) return kExcessNo;
    if (E > 63 && (set >> 32) != 0xffffffffull) return kExcessUnsure;
    // the last item that one of the sums 32 .. 63 needs: the run begins behind it
    const int begin = E > 63 ? bits_wave_max(lane >= 32 ? first : 0) : -1;
    int shown = begin;  // from behind this item on all sums 64 .. E are reachable, by the items in their order
    for (int length = 32, lacking = E - 63; lacking > 0;) {
        const int i0 = (shown + 1) & ~63, i = i0 + lane;
        if (i0 >= limit) {
            shown = kGone;
            break;
        }
        const int w_ = list(i0), w = i > shown && i < limit ? w_ : kGone;
        const int upto = bits_wave_prefix_sum(w <= min(length, C) ? w : 0, lane);
        const unsigned long long enough = __builtin_amdgcn_ballot_w64(upto >= min(length, lacking));
        const int b = enough != 0ull ? __builtin_ctzll(enough) : 63;
        const int more = __builtin_amdgcn_readlane(upto, b);
        shown = i0 + b;
        length += more;
        lacking -= more;
    }
    bool closely = shown == kGone;
    if (closely && !thorough) return kExcessUnsure;
    int shift = 0, length = 32;  // closely: lane x: the run of the items up to begin + (x + 1 << shift)
    for (;;) {
        if (closely) {
            while ((64 << shift) < limit - 1 - begin) ++shift;
            const int cut = begin + ((lane + 1) << shift);
            for (int lighter = 0, upper = 32;; lighter = upper, upper *= 2) {
                for (int i0 = (begin + 1) & ~63; i0 < limit; i0 += 64) {
                    const int i = i0 + lane, w = list(i0);
                    unsigned long long in = __builtin_amdgcn_ballot_w64(i > begin && i < limit && w > lighter && w <= min(upper, C));
                    for (; in != 0ull; in &= in - 1ull) {
                        const int b = __builtin_ctzll(in), wt = __builtin_amdgcn_readlane(w, b);
                        length += i0 + b <= cut && wt <= length ? wt : 0;
                    }
                }
                if (upper >= E || __builtin_amdgcn_ballot_w64(length > upper) == 0ull) break;
            }
        }
        // The walk, until E is used up or it comes to an item whose answer the run does not show.
        bool on = true;
        for (int i0 = (limit - 1) & ~63; E > 0 && on; i0 -= 64) {
            if (i0 < 0) return kExcessUnsure;  // (never: a sum that is reachable can be left out)
            const int i = i0 + lane, w_ = list(i0), w = i < limit && w_ <= C ? w_ : kGone;
            unsigned long long out = 0ull, below = ~0ull;
            int sure = i > shown ? kGone : 63;  // all sums from 64 on up to this are those of items before i
            if (closely) {
                const int part = ((i - 1 - begin) >> shift) - 1;
                const int x = __builtin_amdgcn_ds_bpermute(part << 2, length);
                sure = part >= 0 ? 31 + x : 63;
            }
            if (E > 127) {
                // All items from the end of the list on that leave 64 or more of E are spared together, up to the first one
                // that would leave less than that but not nothing, or that the run does not show.
                const int most = E - 64, x = w <= most && E <= sure ? w : 0;
                const int upto = bits_wave_suffix_sum(x, lane);
                const unsigned long long end = __builtin_amdgcn_ballot_w64(w <= E && (x == 0 || upto > most));
                const int b = end != 0ull ? 63 - (int)__builtin_clzll(end) : -1;
                if (b < 63) E -= __builtin_amdgcn_readlane(upto, b + 1);
                below = b < 0 ? 0ull : (2ull << b) - 1ull;
                out = __builtin_amdgcn_ballot_w64(x > 0) & ~below;
                if (b >= 0) limit = min(limit, i0 + b + 1);
            }
            auto spare = [&]() {
                const int d = E - w;
                const int f = __builtin_amdgcn_ds_bpermute(d << 2, first);  // (lane d mod 64)
                return __builtin_amdgcn_ballot_w64((d > 63) | ((d >= 0) & (f < i)));
            };
            unsigned long long m = spare() & below;
            while (m != 0ull && on) {
                const int b = 63 - (int)__builtin_clzll(m), wt = __builtin_amdgcn_readlane(w, b);
                const unsigned long long bit = 1ull << b;
                on = E - wt <= 63 || E - wt <= __builtin_amdgcn_readlane(sure, b);
                E -= on ? wt : 0;
                out |= on ? bit : 0ull;
                limit = i0 + b + (on ? 0 : 1);
                m = spare() & (bit - 1ull);
            }
            excess_spare(spared, lane, i0 >> 6, out);
        }
        if (E == 0) return kExcessYes;
        if (closely || !thorough) return kExcessUnsure;
        closely = true;
    }
}

// Lane i gets lane i - 1's word, lane 0 zero.
__device__ __forceinline__ uint32_t excess_below(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x138, 0xf, 0xf, true);  // wave_shr:1
}

// The sums 0 .. E < 2048, a word a lane, for what the 64 lowest sums do not show.  first[] is kept as bit planes, the
// item's number in binary, set where the item's sums are new; the walk asks it only about items at or below the last
// one that added a sum (above it the set decides).
template <int NP, class List>
__device__ __forceinline__ ExcessAnswer excess_wide(List &&list, int lane, int p, int C, int E, ExcessSpared &spared)
{
    const uint32_t mask = E >= lane * 32 + 31 ? 0xffffffffu : E < lane * 32 ? 0u : (2u << (E - lane * 32)) - 1u;
    uint32_t own = lane == 0 ? 1u : 0u, first[NP];
#pragma unroll
    for (int j = 0; j < NP; ++j) first[j] = 0;
    int last = -1;            // the last item that added a sum
    int missing = min(E, C);  // no item above this adds one
    for (int i0 = 0; i0 < p && missing > 0; i0 += 64) {
        const int w_ = list(i0), w = i0 + lane < p ? w_ : kGone;
        unsigned long long in = __builtin_amdgcn_ballot_w64(w <= missing);
        while (in != 0ull) {
            const int b = __builtin_ctzll(in);
            const int wt = __builtin_amdgcn_readlane(w, b), ws = (wt - 1) >> 5;
            // new word i = old cells 32 i - wt .. 32 i - wt + 31, as in the row's sweep
            const uint32_t from = (uint32_t)__builtin_amdgcn_ds_bpermute((lane - ws) << 2, (int)own);
            const uint32_t hi = lane >= ws ? from : 0u;
            const uint32_t fresh = __builtin_amdgcn_alignbit(hi, excess_below(hi), (uint32_t)-wt) & mask & ~own;
            own |= fresh;
            last = __builtin_amdgcn_ballot_w64(fresh != 0u) != 0ull ? i0 + b : last;
#pragma unroll
            for (int j = 0; j < NP; ++j) first[j] |= fresh & (uint32_t)-(((i0 + b) >> j) & 1);
            const uint32_t holes = mask & ~own;
            const unsigned long long any = __builtin_amdgcn_ballot_w64(holes != 0u);
            const int top = 63 - (int)__builtin_clzll(any | 1ull);
            const uint32_t word = (uint32_t)__builtin_amdgcn_readlane((int)holes, top);
            missing = word != 0u ? min(C, top * 32 + 31 - (int)__builtin_clz(word)) : 0;
            in = __builtin_amdgcn_ballot_w64(w <= missing) & (~1ull << b);
        }
    }
    if ((((uint32_t)__builtin_amdgcn_readlane((int)own, E >> 5) >> (E & 31)) & 1u) == 0u) return kExcessNo;
    for (int i0 = (p - 1) & ~63; E > 0; i0 -= 64) {
        if (i0 < 0) return kExcessUnsure;  // (never: a sum that is reachable can be left out)
        const int i = i0 + lane, w_ = list(i0), w = i < p && w_ <= C ? w_ : kGone;
        unsigned long long out = 0ull;
        auto spare = [&]() {
            const int d = E - w, at = max(d, 0);
            const uint32_t word = (uint32_t)__builtin_amdgcn_ds_bpermute((at >> 5) << 2, (int)own);
            return __builtin_amdgcn_ballot_w64((d >= 0) & (((word >> (at & 31)) & 1u) != 0u));
        };
        unsigned long long m = spare();
        while (m != 0ull) {
            const int b = 63 - (int)__builtin_clzll(m), wt = __builtin_amdgcn_readlane(w, b), d = E - wt;
            const unsigned long long bit = 1ull << b;
            bool is = true;
            if (i0 + b <= last && d > 0) {
                int f = 0;
#pragma unroll
                for (int j = 0; j < NP; ++j) f |= (int)(((uint32_t)__builtin_amdgcn_readlane((int)first[j], d >> 5) >> (d & 31)) & 1u) << j;
                is = f < i0 + b;
            }
            E -= is ? wt : 0;
            out |= is ? bit : 0ull;
            m = spare() & (bit - 1ull);
        }
        excess_spare(spared, lane, i0 >> 6, out);
    }
    return kExcessYes;
}

// One stage: the items of the list, n at most, of weight at most C.  kExcessEmpty: no item is in the list any more.
// kExcessDone: answered; take(first item, mask) was called for every 64 items of the selection, `value` is its weight,
// `last` its last item (-1: none).  kExcessNot: not answered, nothing taken.  `persistent`: the row's sweep costs more than
// this stage's.
template <int NP, class List, class Take>
__device__ __forceinline__ ExcessResult excess_stage(List &&list, int lane, int n, int C, bool persistent, int &value, int &last, Take &&take)
{
    int sum = 0, items = 0, p = -1, E = 0;
    value = 0;
    last = -1;
    unsigned long long open = 0ull;
    for (int i0 = 0; i0 < n; i0 += 64) {
        const int w = list(i0);
        const unsigned long long in = __builtin_amdgcn_ballot_w64(w <= C);
        open |= __builtin_amdgcn_ballot_w64(w != kGone);
        const int upto = sum + bits_wave_prefix_sum(w <= C ? w : 0, lane);
        const unsigned long long past = __builtin_amdgcn_ballot_w64(upto >= C) & in;
        if (past != 0ull) {
            const int b = __builtin_ctzll(past);
            p = i0 + b;
            E = __builtin_amdgcn_readlane(upto, b) - C;
            items += (int)__popcll(in & ((2ull << b) - 1ull));
            break;
        }
        if (in != 0ull) last = i0 + 63 - (int)__builtin_clzll(in);
        items += (int)__popcll(in);
        sum = __builtin_amdgcn_readlane(upto, 63);
    }
    ExcessSpared spared{0u, 0u};
    if (p < 0) {
        // all that is offered fits together and is taken (every value is positive)
        value = sum;
        if (open == 0ull) return kExcessEmpty;
    } else {
        last = -1;
        if (E > 0 && items < kExcessFewest) return kExcessNot;
        ExcessAnswer answer = kExcessYes;
        for (int attempt = 0; E > 0; ++attempt) {
            const bool thorough = persistent || (C >= kExcessThorough && (4 * E <= 3 * C || items >= kExcessMany));
            // Where all that is lighter than the excess weighs less than that, the items that follow do not help for long: each adds
            // to both.
            if (E > 63) {
                int light = 0;
                for (int i0 = 0; i0 < p && light < E; i0 += 64) {
                    const int w = list(i0);
                    light += bits_wave_sum(i0 + lane < p && w <= min(E, C) ? w : 0);
                }
                if (light < E) return kExcessNot;
            }
            int limit = p, left = E;
            answer = excess_narrow(list, lane, C, thorough, limit, left, spared);
            if (answer == kExcessUnsure && left < kExcessCells && thorough) {
                answer = excess_wide<NP>(list, lane, limit, C, left, spared);
                if (answer == kExcessNo && !persistent) return kExcessNot;
            }
            if (answer != kExcessNo || attempt + 1 >= kExcessTries) break;
            int next = -1;
            for (int i0 = (p + 1) & ~63; i0 < n; i0 += 64) {
                const int w_ = list(i0), w = i0 + lane > p ? w_ : kGone;
                const unsigned long long in = __builtin_amdgcn_ballot_w64(w <= C);
                if (in == 0ull) continue;
                const int b = __builtin_ctzll(in);
                next = i0 + b;
                E += __builtin_amdgcn_readlane(w, b);
                break;
            }
            if (next < 0) break;
            p = next;
        }
        if (answer != kExcessYes) return kExcessNot;
        value = C;
        last = p;
    }
    for (int i0 = 0; i0 <= last; i0 += 64) {
        const int w = list(i0);
        const unsigned long long in = __builtin_amdgcn_ballot_w64(i0 + lane <= last && w <= C);
        const unsigned long long out = (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)spared.lo, i0 >> 6) |
                                       (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)spared.hi, i0 >> 6) << 32;
        take(i0, in & ~out);
    }
    return kExcessDone;
}

}  // namespace

}  // namespace deft
