// Sequential multiple-knapsack solve for instances whose values equal their weights (the
// paper's Problem 1: a bucket's profit is its communication time), one bit per capacity cell.
//
// With v == w the DP value row[c] is the largest reachable sum not above c, so the row is
// described by the set of reachable sums: one bit per cell, and an item is a shift-and-or of
// the whole set, reach |= reach << w, 32 cells per instruction.  The selection the exact DP
// walks back (take an item at a cell only when it strictly improves the value, walk from
// the last item: among optimal subsets the one with the smallest mask) comes out of one
// more table, first[t] = the first offered item that made the sum t reachable:
//   the DP keeps item q at cell c exactly when the best sum up to c rises with item q, i.e.
//   when the target t = row_q[c] was not reachable before q; if q is not kept the target
//   stays, if it is the target becomes t - w_q.  So the walk is t = row[C]; while t > 0:
//   q = first[t], take q, t -= w_q.
//
// One wavefront owns an instance.  Word i of the set (cells 32 i .. 32 i + 31) lives in lane
// i % 64, register slot i / 64, with a copy in LDS that the shifted operand is read from
// (below it a zone of zero words as long as the set, so that no shift needs clamping).
//
// first[] is kept bit-sliced, in registers, as NP planes of one bit per cell, and costs one
// exclusive-or per word and item.  Number the items by a Gray code g: from one item to the next
// exactly one bit j of it toggles, and the item's step is plane[j] ^= set (as it stands after
// the item).  A sum t first reached by item q is in the set from step q on, so plane j has
// toggled once for every change of bit j from q to the last step L: the planes of t spell
// g(q) ^ g(L).  Which bit toggles follows from the item's number alone (the trailing zeros of
// q + 1), so four items are unrolled with planes 0, 1, 0 fixed and the fourth item's plane
// picked by a uniform branch.  (An array of first[] cells in LDS, written where an
// item reached a fresh sum, took half of the kernel - the fresh words are few and found by
// ballots, bit by bit - and its LDS held a compute unit to eight instances.  The ResNet-101-shaped
// sweep of 4096 schedules took 0.469 ms with it and one lookup per taken item in the walk, and
// 0.096 ms so; stages of such lists are now mostly answered without a sweep, seq_excess.h: 0.033 to 0.046 ms.)
//
// What bounds the sweep: a chain of one LDS write and one LDS read per item (1024 instances, a wavefront per SIMD:
// vector units busy 27 % of the cycles, LDS 16 %, the wavefront waiting 43 %) and, with the compute unit full
// of instances, the vector units (4096 ResNet-101-shaped schedules: busy 79 %, LDS 45 %).
//
// Items only ever reach as far as the sum of the weights so far, so a block of four items works
// on the register slots below that, a compile-time count moved up as the sum grows: on average
// a little more than half of the slots.
//
// The walk reads its planes from LDS, where they are put once the sweep is over.  It does not
// follow the chain item by item: 64 lanes suppose that the next 64 items down the list are
// all taken, each looks first[] up at the target this leaves it, and a ballot finds the first
// lane whose item was not the one; the lanes before it take theirs.  A sweep that fills the
// window from the front takes long runs (all but a handful of the items in front of the
// last one), so a walk is a few rounds where it was a chain of a hundred dependent lookups.
// The planes are the largest part of the LDS an instance needs, and only during its walk: the
// wavefronts of a workgroup share one copy under a lock (held for one walk at a time; the
// holder waits for nobody).
#pragma once

#include "instance_check.h"

#include <type_traits>

namespace deft {

namespace {

// Shorter lists are swept at once (81 items, 1735 of them: by what their stages leave out 27.4 -> 36 us; 93 items 13.9 -> 16.7).
// Calls of shorter lists run on kernels without it, whose sweep has the registers (66 items: 17.7 against 20.8 us).
constexpr int kBitsExcessItems = 97;
// In a capacity sweep one sweep answers all capacities, and one capacity that is not answered by itself sends the others
// along, which takes both.  What pays goes by how many items of mean weight fill the smallest window, and by the capacities that a wavefront has
// in turn.  Time by the row alone = 1, 2100 calls (129 to 420 items, 1 to 2500 lists, one to eleven capacities), every list tried: one
// capacity in turn 1.27 where 40 to 48 items fill it, 0.97 to 54, 0.93 to 60, 0.74 to 66; two 1.33, 1.13, 1.03, 0.80; three 1.49,
// 1.28, 1.19, 0.89; four to six 1.5 up to 66, 1.24 to 75, 0.85 from there on; more 1.9 up to 75, 1.58 to 85, 0.97.  Lists that are
// not tried take some 2 us longer on these kernels (14 -> 16), so from four in turn on shorter ones get kernels without them, and rows of 7
// words and more ask for 36 items of up to 32 besides, which the lowest sums are made of, or lists of 300 (200 items without, 1500 lists, eleven
// capacities: 98 us by the row, 184 tried).
struct BitsTried {
    int fewest, fill;  // items of a list whose stages are tried by what they leave out, and of its mean weight in the window
    int sure, light;   // fewer items than `sure`: if so many are light
};
constexpr BitsTried bits_tried_caps(int capacities, int words)
{
    const int fill = 48 + 6 * (capacities - 1);
    return capacities <= 3 ? BitsTried{129, fill, 129, 0} : words < 7 ? BitsTried{225, fill, 225, 0} : BitsTried{160, fill, 300, 36};
}
constexpr int kBitsEnumItems = 6;  // stages offered at most this many items are settled by enumeration

// words-per-lane counts are compiled for; a block of items works on a multiple of bits_grain(K) slots
constexpr int bits_grain(int k) { return k <= 7 ? 1 : k <= 14 ? 2 : 4; }
constexpr int bits_plane_stride(int np) { return np | 1; }  // odd: a lane's planes are spread over the LDS banks
// Wavefronts per SIMD the register budget is held to: planes, set, and about fifty others.  That leaves out the
// two shifted words per slot of the item in progress, so most builds beyond five words or six planes
// spill, some of it in the item loop (7 words, 9 planes: 62 registers; 20 and 9: 350; 32 and 9: 727; with stages by what
// they leave out the sweep has a frame of its own, bits_row_function).  Against the array of cells in LDS these builds were
// quicker all the same, 2048 instances of 300 items in two windows: 20000 cells 0.58 -> 0.087 ms, 40000 cells
// 2.07 -> 0.32, 65535 cells 5.95 -> 0.66.
constexpr int bits_waves_per_simd(int k, int np)
{
    const int regs = k * (np + 1) + 50;
    return regs <= 64 ? 8 : regs <= 80 ? 6 : regs <= 96 ? 5 : regs <= 128 ? 4 : regs <= 168 ? 3 : regs <= 256 ? 2 : 1;
}

__device__ __forceinline__ void wave_lds_sync()
{
    // one wavefront: LDS executes its instructions in order; only the compiler has to be
    // kept from reordering
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// The lane index as a value the compiler knows nothing about: what follows from the index alone (a
// slot's address, its mask, for every slot) is cheap to compute where it is used; left visible it is
// all computed once at kernel entry and parked in scratch memory.
__device__ __forceinline__ int bits_local(int lane)
{
    asm volatile("" : "+v"(lane));
    return lane;
}

template <class Op>
__device__ __forceinline__ int bits_wave_reduce(int x, Op op)
{
    x = op(x, __builtin_amdgcn_update_dpp(x, x, 0xB1, 0xf, 0xf, false));   // quad_perm [1,0,3,2]
    x = op(x, __builtin_amdgcn_update_dpp(x, x, 0x4E, 0xf, 0xf, false));   // quad_perm [2,3,0,1]
    x = op(x, __builtin_amdgcn_update_dpp(x, x, 0x124, 0xf, 0xf, false));  // row_ror:4
    x = op(x, __builtin_amdgcn_update_dpp(x, x, 0x128, 0xf, 0xf, false));  // row_ror:8
    return op(op(__builtin_amdgcn_readlane(x, 0), __builtin_amdgcn_readlane(x, 16)),
              op(__builtin_amdgcn_readlane(x, 32), __builtin_amdgcn_readlane(x, 48)));
}
// Sum over the lanes at and above `lane`: shifts inside each row of sixteen lanes (zeros come
// in from beyond the row), then the totals of the rows above are added in.
__device__ __forceinline__ int bits_wave_suffix_sum(int x, int lane)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x101, 0xf, 0xf, true);  // row_shl:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x102, 0xf, 0xf, true);  // row_shl:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x104, 0xf, 0xf, true);  // row_shl:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x108, 0xf, 0xf, true);  // row_shl:8
    const int t1 = __builtin_amdgcn_readlane(x, 16), t2 = __builtin_amdgcn_readlane(x, 32),
              t3 = __builtin_amdgcn_readlane(x, 48);
    return x + (lane < 16 ? t1 : 0) + (lane < 32 ? t2 : 0) + (lane < 48 ? t3 : 0);
}
// Sum over the lanes at and below `lane`, the same way from the other side.
__device__ __forceinline__ int bits_wave_prefix_sum(int x, int lane)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);  // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);  // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true);  // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true);  // row_shr:8
    const int t0 = __builtin_amdgcn_readlane(x, 15), t1 = __builtin_amdgcn_readlane(x, 31),
              t2 = __builtin_amdgcn_readlane(x, 47);
    return x + (lane >= 16 ? t0 : 0) + (lane >= 32 ? t1 : 0) + (lane >= 48 ? t2 : 0);
}
__device__ __forceinline__ int bits_wave_sum(int x) { return bits_wave_reduce(x, [](int a, int b) { return a + b; }); }
__device__ __forceinline__ int bits_wave_max(int x) { return bits_wave_reduce(x, [](int a, int b) { return max(a, b); }); }

}  // namespace

}  // namespace deft

#include "seq_excess.h"

namespace deft {

namespace {

// LDS of a workgroup, in 32-bit words: [lock: 4][planes: plane_words] and per wavefront
// [zeros: row_words][set: row_words][pad: 4][prefix: n_pad + 8][index: n_pad / 2][marks: mark_words].
struct BitsLayout {
    int32_t row_words, n_pad, mark_words, plane_words, wave_words;
    int16_t share;  // wavefronts of an instance (capacity sweep; else 1): they share its part, and deal its capacities out
    int16_t turns;  // capacities that a wavefront has in turn then
};
// One instance's share of it.
struct BitsLds {
    uint32_t *set;      // reachable sums, zeros below
    int32_t *prefix;    // prefix[p]: weight of the stage's first p offered items.  Outside a sweep and its walk: the
                        // weight of every item that is still in the list, kGone for the others
    uint16_t *index;    // the item at position p of the stage's list
    uint32_t *marks;    // sequential modes: a byte per item, its knapsack (255: none); capacity sweep: a word per item
    uint32_t *planes;   // first[] of the walk in progress (shared by the workgroup)
    int32_t *lock;
};

// The state of a stage's sweep.
template <int K, int NP>
struct BitsRows {
    uint32_t own[K];
    uint32_t plane[NP][K];
};

// A sweep in progress: the stage's list, where it may end, and how far it has come.
struct BitsSweep {
    int cnt, cap;             // items listed; the capacity
    int stop_slot, stop_lane; // where cell `cap` lives; slot -1: the sweep does not end there
    uint32_t stop_bit;
    int check_mask;           // looked at after the items whose number has these bits set: every eighth, or every
                              // second one of a list of at most 64
    bool caps_sweep;          // the sweep ends once every lane's capacity `goal` is reachable
    int goal;
    int q;                    // items gone through so far (Gray steps taken)
    int items;                // the same without the empty steps that fill up the last block
    int wchunk, upto;         // lane x: weight of item (q & ~63) + x, and the list's weight up to and with it
    bool reached;
};

// plane[k] ^= set[k] for M slots, if h == J (uniform).  The branch is inside the asm: as a branch of the
// program every plane is merged behind it, and the merges of a chain of them cost the compiler
// half of the registers again in copies.
template <int J, int M>
__device__ __forceinline__ void bits_toggle_if(int h, uint32_t *plane, const uint32_t *set)
{
    static_assert(M >= 1 && M <= 7, "slots per branch");
    if constexpr (M == 1)
        asm volatile("s_cmp_lg_u32 %2, %3\n\ts_cbranch_scc1 .Lkeep%=\n\t"
                     "v_xor_b32 %0, %0, %1\n.Lkeep%=:"
                     : "+v"(plane[0]) : "v"(set[0]), "s"(h), "n"(J) : "scc");
    else if constexpr (M == 2)
        asm volatile("s_cmp_lg_u32 %4, %5\n\ts_cbranch_scc1 .Lkeep%=\n\t"
                     "v_xor_b32 %0, %0, %2\n\tv_xor_b32 %1, %1, %3\n.Lkeep%=:"
                     : "+v"(plane[0]), "+v"(plane[1]) : "v"(set[0]), "v"(set[1]), "s"(h), "n"(J) : "scc");
    else if constexpr (M == 3)
        asm volatile("s_cmp_lg_u32 %6, %7\n\ts_cbranch_scc1 .Lkeep%=\n\t"
                     "v_xor_b32 %0, %0, %3\n\tv_xor_b32 %1, %1, %4\n\tv_xor_b32 %2, %2, %5\n.Lkeep%=:"
                     : "+v"(plane[0]), "+v"(plane[1]), "+v"(plane[2]) : "v"(set[0]), "v"(set[1]), "v"(set[2]), "s"(h), "n"(J) : "scc");
    else if constexpr (M == 4)
        asm volatile("s_cmp_lg_u32 %8, %9\n\ts_cbranch_scc1 .Lkeep%=\n\t"
                     "v_xor_b32 %0, %0, %4\n\tv_xor_b32 %1, %1, %5\n\tv_xor_b32 %2, %2, %6\n\tv_xor_b32 %3, %3, %7\n.Lkeep%=:"
                     : "+v"(plane[0]), "+v"(plane[1]), "+v"(plane[2]), "+v"(plane[3]) : "v"(set[0]), "v"(set[1]), "v"(set[2]), "v"(set[3]), "s"(h), "n"(J) : "scc");
    else if constexpr (M == 5)
        asm volatile("s_cmp_lg_u32 %10, %11\n\ts_cbranch_scc1 .Lkeep%=\n\t"
                     "v_xor_b32 %0, %0, %5\n\tv_xor_b32 %1, %1, %6\n\tv_xor_b32 %2, %2, %7\n\tv_xor_b32 %3, %3, %8\n\tv_xor_b32 %4, %4, %9\n.Lkeep%=:"
                     : "+v"(plane[0]), "+v"(plane[1]), "+v"(plane[2]), "+v"(plane[3]), "+v"(plane[4]) : "v"(set[0]), "v"(set[1]), "v"(set[2]), "v"(set[3]), "v"(set[4]), "s"(h), "n"(J) : "scc");
    else if constexpr (M == 6)
        asm volatile("s_cmp_lg_u32 %12, %13\n\ts_cbranch_scc1 .Lkeep%=\n\t"
                     "v_xor_b32 %0, %0, %6\n\tv_xor_b32 %1, %1, %7\n\tv_xor_b32 %2, %2, %8\n\tv_xor_b32 %3, %3, %9\n\tv_xor_b32 %4, %4, %10\n\tv_xor_b32 %5, %5, %11\n.Lkeep%=:"
                     : "+v"(plane[0]), "+v"(plane[1]), "+v"(plane[2]), "+v"(plane[3]), "+v"(plane[4]), "+v"(plane[5]) : "v"(set[0]), "v"(set[1]), "v"(set[2]), "v"(set[3]), "v"(set[4]), "v"(set[5]), "s"(h), "n"(J) : "scc");
    else if constexpr (M == 7)
        asm volatile("s_cmp_lg_u32 %14, %15\n\ts_cbranch_scc1 .Lkeep%=\n\t"
                     "v_xor_b32 %0, %0, %7\n\tv_xor_b32 %1, %1, %8\n\tv_xor_b32 %2, %2, %9\n\tv_xor_b32 %3, %3, %10\n\tv_xor_b32 %4, %4, %11\n\tv_xor_b32 %5, %5, %12\n\tv_xor_b32 %6, %6, %13\n.Lkeep%=:"
                     : "+v"(plane[0]), "+v"(plane[1]), "+v"(plane[2]), "+v"(plane[3]), "+v"(plane[4]), "+v"(plane[5]), "+v"(plane[6]) : "v"(set[0]), "v"(set[1]), "v"(set[2]), "v"(set[3]), "v"(set[4]), "v"(set[5]), "v"(set[6]), "s"(h), "n"(J) : "scc");
}
template <int J, int KK>
__device__ __forceinline__ void bits_toggle_slots(int h, uint32_t *plane, const uint32_t *set)
{
    if constexpr (KK <= 7) {
        bits_toggle_if<J, KK>(h, plane, set);
    } else {
        bits_toggle_if<J, 4>(h, plane, set);
        bits_toggle_slots<J, KK - 4>(h, plane + 4, set + 4);
    }
}
// The same for planes J .. NP - 1.
template <int J, int NP, int KK, int K>
__device__ __forceinline__ void bits_toggle_from(int h, uint32_t (&plane)[NP][K], const uint32_t (&set)[K])
{
    if constexpr (J < NP) {
        bits_toggle_slots<J, KK>(h, plane[J], set);
        bits_toggle_from<J + 1, NP, KK, K>(h, plane, set);
    }
}

// Items until the list ends, the sweep may end, or slots beyond the first KK are needed; then on to
// the next slot count.
template <int KK, int K, int NP>
__device__ __forceinline__ void bits_run(const BitsLds &l, BitsRows<K, NP> &r, int lane, BitsSweep &w)
{
    constexpr int GS = bits_grain(K);
    uint32_t *set = l.set;
    auto look = [&]() {
        uint32_t word = 0;
#pragma unroll
        for (int k = KK - GS; k < KK; ++k)
            if (k == w.stop_slot) word = (uint32_t)__builtin_amdgcn_readlane((int)r.own[k], w.stop_lane);
        return (word & w.stop_bit) != 0;
    };
    while (w.q < w.cnt) {
        if ((w.q & 63) == 0) {
            const int p = w.q + lane;
            w.upto = l.prefix[min(p + 1, w.cnt)];
            w.wchunk = p < w.cnt ? w.upto - l.prefix[p] : 0;
        }
        if (KK < K && min(__builtin_amdgcn_readlane(w.upto, (w.q & 63) + 3), w.cap) >= KK * 2048) break;
        bool early = false;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            int wt = __builtin_amdgcn_readlane(w.wchunk, (w.q & 63) + i);
            if (i >= 2) wt = early ? 0 : wt;  // (an item of no weight changes nothing)
            // new word i = old cells 32 i - wt .. 32 i - wt + 31, of the old words i - ws and i - ws - 1
            // with ws = (wt - 1) / 32: a funnel shift by -wt mod 32 (the instruction takes the low five bits)
            const uint32_t *src = set + (lane - ((wt - 1) >> 5));
            uint32_t lo[KK], hi[KK];
#pragma unroll
            for (int k = 0; k < KK; ++k) {
                lo[k] = src[k * 64 - 1];
                hi[k] = src[k * 64];
            }
            wave_lds_sync();
#pragma unroll
            for (int k = 0; k < KK; ++k) {
                r.own[k] |= __builtin_amdgcn_alignbit(hi[k], lo[k], (uint32_t)-wt);
                set[k * 64 + lane] = r.own[k];
                if (i < 3) {
                    r.plane[i & 1][k] ^= r.own[k];
                    asm volatile("" : "+v"(r.plane[i & 1][k]));  // (here: sunk to the end of the block it keeps three sets alive)
                }
            }
            wave_lds_sync();
            if (i == 1 && w.check_mask == 1) early = look();
        }
        const int hp = __builtin_amdgcn_readfirstlane(__builtin_ctz((w.q >> 2) + 1) + 2);  // the plane of the fourth item
        bits_toggle_slots<2, KK>(hp, r.plane[2], r.own);  // (half of the time)
        if (hp > 2) bits_toggle_from<3, NP, KK, K>(hp, r.plane, r.own);
        w.items = w.q + (early ? 2 : 4);
        w.q += 4;
        if (((w.q - 1) & w.check_mask) == w.check_mask) {
            w.reached = early || look();
            if (w.caps_sweep) w.reached = __builtin_amdgcn_ballot_w64((set[w.goal >> 5] >> (w.goal & 31) & 1u) == 0) == 0ull;
            if (w.reached) return;
        }
    }
    if constexpr (KK < K) {
        if (w.q < w.cnt) bits_run<KK + GS, K, NP>(l, r, lane, w);
    }
}

// Sweeps the stage's list (`cnt` items, prefix sums in l.prefix) at capacity C.  Ends early once C
// itself is reachable: the value is final, and the walk from C only follows sums that earlier
// items reached.  (caps_sweep: once every lane's capacity `goal` is.)
template <int K, int NP>
__device__ __forceinline__ BitsSweep bits_sweep(const BitsLds &l, BitsRows<K, NP> &r, int lane, int cnt, int C,
                                                bool caps_sweep, int goal)
{
    constexpr int GS = bits_grain(K);
    lane = bits_local(lane);
    const int slots_all = ((C >> 11) + GS) / GS * GS;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        r.own[k] = (k == 0 && lane == 0) ? 1u : 0u;  // the empty sum
        if (k < slots_all) l.set[k * 64 + lane] = r.own[k];
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            r.plane[j][k] = 0;
        }
    }
    wave_lds_sync();
    BitsSweep w{cnt, C, caps_sweep ? -1 : C >> 11, (C >> 5) & 63, 1u << (C & 31), !caps_sweep && cnt <= 64 ? 1 : 7,
                caps_sweep, goal, 0, 0, 0, 0, false};
    bits_run<GS, K, NP>(l, r, lane, w);
    w.items = min(w.items, cnt);
    return w;
}

// Largest reachable sum <= C.
template <int K, int NP>
__device__ __forceinline__ int bits_top(const BitsRows<K, NP> &r, int lane, int C)
{
    int top = 0;
    lane = bits_local(lane);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int cell0 = (k * 64 + lane) * 32;
        const uint32_t need = cell0 + 31 <= C ? 0xffffffffu : cell0 > C ? 0u : (1u << (C - cell0 + 1)) - 1u;
        const uint32_t x = r.own[k] & need;
        if (x) top = max(top, cell0 + 31 - __builtin_clz(x));
    }
    return bits_wave_max(top);
}

// The planes to LDS (taking the workgroup's lock), word by word: the NP planes of a word side by side.
template <int K, int NP>
__device__ __forceinline__ void bits_publish(const BitsLds &l, const BitsRows<K, NP> &r, int lane, int C)
{
    constexpr int PS = bits_plane_stride(NP);
    lane = bits_local(lane);
    if (blockDim.x > 64) {
        if (lane == 0) {
            while (atomicCAS(l.lock, 0, 1) != 0) __builtin_amdgcn_s_sleep(2);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        __builtin_amdgcn_wave_barrier();
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if (k * 2048 <= C) {
#pragma unroll
            for (int j = 0; j < NP; ++j) l.planes[(k * 64 + lane) * PS + j] = r.plane[j][k];
        }
    }
    wave_lds_sync();
}
__device__ __forceinline__ void bits_release(const BitsLds &l, int lane)
{
    wave_lds_sync();
    if (blockDim.x > 64) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        if (lane == 0) atomicExch(l.lock, 0);
    }
}

// first[t] after `steps` Gray steps, read off the published planes.
template <int NP>
__device__ __forceinline__ int bits_first(const uint32_t *planes, int t, int steps)
{
    const uint32_t *at = planes + (t >> 5) * bits_plane_stride(NP);
    const int b = t & 31;
    uint32_t code = 0;
#pragma unroll
    for (int j = 0; j < NP; ++j) code |= ((at[j] >> b) & 1u) << j;
    code ^= (uint32_t)(steps ^ (steps >> 1)) & ((1u << NP) - 1u);
    code ^= code >> 1;  // Gray code to number
    code ^= code >> 2;
    code ^= code >> 4;
    if constexpr (NP > 8) code ^= code >> 8;
    return (int)code;
}

// The walk from the sum `t`, by groups of G lanes (a power of two), each with a target of its
// own.  Lane x of a group supposes that the x items before position `from` + 1 down the list are
// taken.  take(p) is called by the lanes whose item (position p) is taken.  Returns what is
// left of t (0, unless something is broken).
template <int NP, class Take>
__device__ __forceinline__ int bits_walk(const BitsLds &l, int lane, int G, int t, int cnt, int steps, Take &&take)
{
    const int x = lane & (G - 1), group = lane & ~(G - 1);
    const unsigned long long group_mask = (G == 64 ? ~0ull : (1ull << G) - 1ull) << group;
    int q = t > 0 ? min(bits_first<NP>(l.planes, t, steps), cnt - 1) : 0;
    int guard = 2 * cnt + 2;  // (every round takes an item or moves down the list)
    while (__builtin_amdgcn_ballot_w64(t > 0) != 0ull && guard-- > 0) {
        const int p = q - x;
        const bool in_list = t > 0 && p >= 0;
        const int left = in_list ? t - (l.prefix[q + 1] - l.prefix[p + 1]) : 0;
        const int first = left > 0 ? min(bits_first<NP>(l.planes, left, steps), cnt - 1) : 0;
        const bool fits = left > 0 && first == p;
        const unsigned long long miss = __builtin_amdgcn_ballot_w64(!fits) & group_mask;
        const int stop = miss != 0ull ? __builtin_ctzll(miss) : group + G;  // lanes of the group before it take
        if (lane < stop && fits) take(p);
        // the next target: what the stopping lane was left with (nothing, once t is used up or
        // the list is), or what follows the group's last item
        const int src = min(stop, group + G - 1);
        int t_next = __shfl(left, src), q_next = __shfl(first, src);
        if (stop == group + G) {
            const int p_last = q - (G - 1);
            t_next = t - (l.prefix[q + 1] - l.prefix[p_last]);
            q_next = p_last - 1;
            if (q_next < 0) q_next = 0;
        }
        t = t > 0 ? max(t_next, 0) : t;
        q = q_next;
    }
    return t;
}

// One stage by the row's sweep and its walk, or walks, over the list in LDS.
struct BitsStage {
    int cnt, C, j;  // items listed; the capacity (of a capacity sweep: the largest); the knapsack
    int m, goal;    // capacity sweep: capacities, and the lane's
    int levels, caps_sweep;
};
struct BitsAnswer {
    int value;   // of a capacity sweep: the lane's
    int last;    // Algorithm 1: the item that completed the value (-1: none)
    int failed;  // (never expected)
};
template <int K, int NP>
__device__ __forceinline__ BitsAnswer bits_row(const BitsLds &l, int lane, const BitsStage &g, unsigned long long *swept_cells)
{
    BitsRows<K, NP> rows;
    BitsAnswer r{0, -1, 0};
    const BitsSweep sw = bits_sweep<K, NP>(l, rows, lane, g.cnt, g.C, g.caps_sweep != 0, g.goal);
    const int steps = sw.q;
    if (swept_cells && lane == 0) {
        // measurement only: C - w + 1 per item the sweep went through
        atomicAdd(swept_cells,
                  (unsigned long long)sw.items * (unsigned)(g.C + 1) - (unsigned long long)(unsigned)l.prefix[sw.items]);
    }
    bits_publish<K, NP>(l, rows, lane, g.C);
    if (!g.caps_sweep) {
        uint8_t *mark8 = reinterpret_cast<uint8_t *>(l.marks);
        r.value = sw.reached ? g.C : bits_top<K, NP>(rows, lane, g.C);
        if (g.levels && r.value > 0) r.last = l.index[min(bits_first<NP>(l.planes, r.value, steps), g.cnt - 1)];
        r.failed = bits_walk<NP>(l, lane, 64, r.value, g.cnt, steps, [&](int p) { mark8[l.index[p]] = (uint8_t)g.j; }) != 0;
    } else {
        // One sweep at the largest capacity answers every capacity: the largest reachable
        // sum not above it, and the chain from that sum is the selection the DP would walk
        // back there.  The lanes are dealt out to the capacities in groups, all walks run side
        // by side, and an item's word collects the capacities at which it is taken.
        if (lane < g.m) {
            int wi = g.goal >> 5;
            uint32_t bits = l.set[wi] & (0xffffffffu >> (31 - (g.goal & 31)));
            while (bits == 0) bits = l.set[--wi];  // (word 0 holds the empty sum)
            r.value = wi * 32 + 31 - __builtin_clz(bits);
        }
        int G = 64;
        while (G > 1 && 64 / G < g.m) G >>= 1;
        const int x = lane / G;  // this group's capacity
        int t_group = __shfl(r.value, x);
        if (x >= g.m) t_group = 0;
        const int left = bits_walk<NP>(l, lane, G, t_group, g.cnt, steps,
                                       [&](int p) { atomicOr(&l.marks[l.index[p]], 1u << x); });
        r.failed = __builtin_amdgcn_ballot_w64(left != 0) != 0ull;
    }
    bits_release(l, lane);
    return r;
}

// The same as a function of its own, for kernels with stages by what they leave out: what the compiler keeps in
// registers for those it took from the row's sweep, whose item loop spilled twice as much (7 words and 9 planes: 131
// registers in place of 64).  900 lists of 334 items of which three hold 85 % of the time, windows of 11700 and 5900 cells: 117 us in kernels
// without those stages, 149 inlined, 94 so; 24000 and 12000: 155, 194 (230 before), 154.  A call saves and restores up
// to a hundred registers, a microsecond or so: where the sweep fits the registers anyhow it stays inlined (up to 60 words of set and planes:
// 2013 lists of 150 items in windows of 9000 cells 44 us, 46 by calls; and the task queues, 114 and 127).
// LDS pointers go as offsets: as generic ones they would be loaded from by flat instructions.
template <class T>
__device__ __forceinline__ int bits_lds_offset(T *p)
{
    return (int)(uint32_t)(uintptr_t)(__attribute__((address_space(3))) T *)p;
}
template <class T>
__device__ __forceinline__ T *bits_lds_pointer(int offset)
{
    return (T *)(__attribute__((address_space(3))) T *)(uintptr_t)(uint32_t)__builtin_amdgcn_readfirstlane(offset);
}
template <int K, int NP>
__device__ __noinline__ BitsAnswer bits_row_function(int set, int prefix, int index, int marks, int planes, int lock, int cnt, int C, int j,
                                                     int m, int goal, int levels, int caps_sweep, unsigned long long *swept_cells)
{
    const auto uniform = [](int x) { return __builtin_amdgcn_readfirstlane(x); };
    const BitsLds l{bits_lds_pointer<uint32_t>(set), bits_lds_pointer<int32_t>(prefix), bits_lds_pointer<uint16_t>(index),
                    bits_lds_pointer<uint32_t>(marks), bits_lds_pointer<uint32_t>(planes), bits_lds_pointer<int32_t>(lock)};
    const BitsStage g{uniform(cnt), uniform(C), uniform(j), uniform(m), goal, uniform(levels), uniform(caps_sweep)};
    return bits_row<K, NP>(l, threadIdx.x & 63, g, swept_cells);
}
template <int K, int NP>
__device__ __forceinline__ BitsAnswer bits_row_call(const BitsLds &l, const BitsStage &g, unsigned long long *swept_cells)
{
    return bits_row_function<K, NP>(bits_lds_offset(l.set), bits_lds_offset(l.prefix), bits_lds_offset(l.index), bits_lds_offset(l.marks),
                                    bits_lds_offset(l.planes), bits_lds_offset(l.lock), g.cnt, g.C, g.j, g.m, g.goal, g.levels,
                                    g.caps_sweep, swept_cells);
}

// The task queues' arguments, of the kernels that solve those.
struct BitsNoArgs {
    int32_t n_buckets, iterations;
};
template <bool QUEUES>
using BitsQueueArgs = std::conditional_t<QUEUES, ScheduleArgs, BitsNoArgs>;
// The arguments and the workgroup's size behind them (12 bytes on) end within three cache lines: a fourth is fetched by itself, 0.2 us
// of a call's 8 to 12.
static_assert(sizeof(BatchArgs) + sizeof(BitsNoArgs) + sizeof(BitsLayout) + sizeof(void *) + 14 <= 192, "kernel arguments");

// K: words per lane (capacities up to 2048 K - 1).  NP: planes (lists of up to 2^NP items).
// a.mode: DEFT_MODE_SEQUENTIAL, DEFT_MODE_RECURSIVE or DEFT_MODE_CAPACITY_SWEEP.  QUEUES: the two task queues (q; the
// candidates' times as a's weights and values), all stages of a candidate by its wavefront; its current queue is the
// list as it stands after the stage before.
template <int K, int NP, bool QUEUES, bool EXCESS>
__global__ void __launch_bounds__(256, bits_waves_per_simd(K, NP))
seq_bits_kernel(BatchArgs a, BitsQueueArgs<QUEUES> q, BitsLayout lay, unsigned long long *swept_cells)
{
    extern __shared__ __align__(16) int32_t lds_bits[];
    const int lane_ = threadIdx.x & 63, lane = lane_;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    constexpr bool by_excess = EXCESS;  // stages by what they leave out (seq_excess.h)
    const int share = QUEUES || !by_excess ? 1 : lay.share;
    const int inst = share > 1 ? (int)blockIdx.x : (int)blockIdx.x * (int)(blockDim.x >> 6) + wave;
    BitsLds l;
    l.lock = lds_bits;
    l.planes = reinterpret_cast<uint32_t *>(lds_bits) + 4;
    uint32_t *zeros = l.planes + lay.plane_words + (size_t)(share > 1 ? 0 : wave) * lay.wave_words;
    l.set = zeros + lay.row_words;
    l.prefix = reinterpret_cast<int32_t *>(l.set + lay.row_words + 4);
    l.index = reinterpret_cast<uint16_t *>(l.prefix + lay.n_pad + 8);
    l.marks = reinterpret_cast<uint32_t *>(l.prefix + lay.n_pad + 8 + lay.n_pad / 2);
    if (blockDim.x > 64) {
        if (threadIdx.x == 0) *l.lock = 0;
        __syncthreads();
    }
    if (inst >= a.batch) return;  // (the whole wavefront; no barrier follows)

    constexpr bool queues = QUEUES;
    const bool levels = !queues && a.mode == DEFT_MODE_RECURSIVE, caps_sweep = !queues && a.mode == DEFT_MODE_CAPACITY_SWEEP;
    const bool drops = levels || queues;
    // Everything whose address follows from the instance number alone is fetched at once: the
    // kernel's entry is one memory round trip.  The weights stay in registers (lists of up to
    // 512 items; longer ones are read again per stage).
    constexpr int NCH = NP <= 6 ? 1 : NP <= 9 ? 8 : 1;
    const int32_t *__restrict__ W = a.weights + (size_t)inst * a.item_stride;
    const int32_t *__restrict__ V = a.values + (size_t)inst * a.item_stride;
    const int32_t *drop = drops ? a.drop_time + (size_t)inst * a.item_stride : nullptr;
    const int32_t *cap = queues ? nullptr : a.capacities + (size_t)inst * a.knap_stride;
    const int32_t *ord = a.fill_order ? a.fill_order + (size_t)inst * a.knap_stride : nullptr;
    int wreg[NCH], vreg[NCH], dreg[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        const bool have = c * 64 + lane < a.item_stride;
        wreg[c] = have ? W[c * 64 + lane] : 0;
        vreg[c] = have ? V[c * 64 + lane] : 0;
        dreg[c] = 0;
    }
    if (drops && NP <= 9) {
#pragma unroll
        for (int c = 0; c < NCH; ++c)
            if (c * 64 + lane < a.item_stride) dreg[c] = drop[c * 64 + lane];
    }
    int cap_raw;
    if constexpr (queues) cap_raw = lane == 0 ? q.forward_time[inst] : lane == 1 ? q.backward_time[inst] : 0;
    else cap_raw = lane < a.knap_stride ? cap[lane] : 0;
    const int ord_raw = ord && lane < a.knap_stride ? ord[lane] : lane;
    const int n = queues ? q.n_buckets : a.n_items[inst], m = queues ? 2 : a.n_knapsacks[inst];
    for (int i = lane; i < lay.row_words; i += 64) zeros[i] = 0;
    // f(first item of the chunk, this lane's weight, this lane's value) for every 64 items
    auto chunks = [&](auto &&f) {
#pragma unroll
        for (int c = 0; c < NCH; ++c)
            if (c * 64 < n) f(c * 64, wreg[c], vreg[c]);
        if constexpr (NP > 9) {
            for (int i0 = 64; i0 < n; i0 += 64) f(i0, i0 + lane < n ? W[i0 + lane] : 0, i0 + lane < n ? V[i0 + lane] : 0);
        }
    };

    // Input checks, in the order every kernel of the library reports them: invalid data, the
    // handle's limits, overflow of the value sum; then the handle's promise that every value
    // equals its weight.
    int status = DEFT_OK;
    {
        uint32_t flags = 0;
        unsigned long long vs = 0;
        bool differs = false;
        if (n < 0 || n > a.item_stride || m < 0 || m > a.knap_stride || (levels && m != 1) || (caps_sweep && m > 31)) {
            flags = 1;
        } else {
            chunks([&](int i0, int w, int v) {
                if (i0 + lane < n) {
                    bool bad = w < 1 || v < 0;
                    if (drops) bad = bad || (NP <= 9 ? dreg[i0 >> 6 & (NCH - 1)] : drop[i0 + lane]) < 0;
                    if (bad) flags |= 1; else vs += (unsigned)v;
                    differs = differs || v != w;
                }
            });
            unsigned long long seen = 0;
            if (lane < m) {
                if (cap_raw < 0) flags |= 1; else if (cap_raw > a.max_capacity) flags |= 2;
                if (ord_raw < 0 || ord_raw >= m) flags |= 1; else seen = 1ull << ord_raw;
            }
            if (ord) {
                // a fill order names every knapsack once: m entries in range with m distinct values
                auto bit_or = [](int x, int y) { return x | y; };
                const int seen_lo = bits_wave_reduce((int)(uint32_t)seen, bit_or);
                const int seen_hi = bits_wave_reduce((int)(uint32_t)(seen >> 32), bit_or);
                if ((int)(__popc((uint32_t)seen_lo) + __popc((uint32_t)seen_hi)) != m) flags |= 1;
            }
        }
        // (a lane adds at most 64 values below 2^31: two pieces, of 24 and 13 bits, keep the sums in range)
        const unsigned long long total_v = (unsigned long long)(unsigned)bits_wave_sum((int)(vs & 0xffffffu)) +
                                           ((unsigned long long)(unsigned)bits_wave_sum((int)(vs >> 24)) << 24);
        if (__builtin_amdgcn_ballot_w64((flags & 1) != 0) != 0ull) status = DEFT_ERR_INVALID_ARG;
        else if (__builtin_amdgcn_ballot_w64((flags & 2) != 0) != 0ull) status = DEFT_ERR_LIMIT;
        else if (total_v >= (1ull << 31)) status = DEFT_ERR_OVERFLOW;
        else if (__builtin_amdgcn_ballot_w64(differs) != 0ull) status = DEFT_ERR_INVALID_ARG;
        if (a.left) {
            // no promise was made: an instance in order that is not a subset-sum problem is the next kernel's
            const bool not_mine = status == DEFT_ERR_INVALID_ARG && __builtin_amdgcn_ballot_w64((flags & 1) != 0) == 0ull;
            if (lane == 0) a.left[inst] = not_mine ? 1 : 0;
            if (not_mine) return;
        }
    }
    int32_t *out_asg = queues ? nullptr : a.assignment + (size_t)inst * a.item_stride;
    const size_t record0 = queues ? (size_t)inst * 2 * q.iterations : 0;
    if constexpr (queues) {
        if (status != DEFT_OK) {
            for (int x = lane; x < 2 * q.iterations; x += 64) q.stage_case[record0 + x] = q.stage_count[record0 + x] = q.stage_time[record0 + x] = 0;
            for (int x = lane; x < q.iterations; x += 64) q.update_k[record0 / 2 + x] = 0;
            if (lane < 2) q.tail[(size_t)inst * 2 + lane] = 0;
            if (lane == 0) q.status[inst] = status;
            return;
        }
    }
    if (status != DEFT_OK) {
        for (int i = lane; i < a.item_stride; i += 64) out_asg[i] = caps_sweep ? 0 : -1;
        if (lane < a.knap_stride) {
            a.knap_value[(size_t)inst * a.knap_stride + lane] = 0;
            a.knap_load[(size_t)inst * a.knap_stride + lane] = 0;
        }
        if (lane == 0) {
            a.total_value[inst] = 0;
            a.status[inst] = status;
        }
        return;
    }
    for (int i = lane; i < lay.mark_words; i += 64) l.marks[i] = caps_sweep ? 0u : queues ? 0x7f7f7f7fu : 0xffffffffu;
    uint8_t *mark8 = reinterpret_cast<uint8_t *>(l.marks);
    const int cap_l = lane < m ? cap_raw : 0;
    const int ord_l = lane < m ? ord_raw : lane;
    int kv_l = 0, kl_l = 0;  // lane j: knapsack j's value and load
    long long total = 0;
    wave_lds_sync();
    // the list as it stands
    auto list_weights = [&]() {
        if constexpr (by_excess) {
            chunks([&](int i0, int w, int) {
                const int i = i0 + lane;
                if (i < n) l.prefix[i] = caps_sweep || mark8[i] == 0xff ? w : kGone;
            });
            wave_lds_sync();
        }
    };
    auto list = [&](int i0) { return i0 + lane < n ? l.prefix[i0 + lane] : kGone; };
    // (Where items heavier than a quarter of the window hold more than half of the time, the excess is mostly out of reach, and where
    // too few items of the list's mean weight fill the window, a capacity sweep's smallest one, it is not tried.)
    const BitsTried tried = caps_sweep ? bits_tried_caps(lay.turns, K) : BitsTried{kBitsExcessItems, kExcessFewest, kBitsExcessItems, 0};
    bool long_list = EXCESS && n >= tried.fewest;
    if (long_list) {
        const int most = bits_wave_max(cap_l), quarter = most >> 2;
        const int window = caps_sweep ? min(most, -bits_wave_max(cap_l > 0 ? -cap_l : -0x7fffffff)) : most;
        int light = 0, heavy = 0, items = 0, tiny = 0;
        chunks([&](int i0, int w, int) {
            const bool in = i0 + lane < n && w <= most;
            items += (int)__popcll(__builtin_amdgcn_ballot_w64(in));
            tiny += (int)__popcll(__builtin_amdgcn_ballot_w64(in && w <= 32));
            light += in && w <= quarter ? w : 0;
            heavy += in && w > quarter ? w : 0;
        });
        light = bits_wave_sum(light);
        heavy = bits_wave_sum(heavy);
        long_list = light > heavy && items * window / tried.fill >= light + heavy && (n >= tried.sure || tiny >= tried.light);  // (4096 items of 65535)
    }
    if (long_list) list_weights();
    // Where wavefronts share an instance: [0 .. 30] the values, then whether a capacity is left over (in the place of the
    // walk's planes).
    uint32_t *shared = l.planes;
    if (share > 1) {
        if (threadIdx.x == 31) shared[31] = 0;
        __syncthreads();
    }
    const int cap_max = caps_sweep ? bits_wave_max(cap_l) : 0;
    const int stages = queues ? 2 * q.iterations : m;
    // Task queues: items and time of the current queue, the iterations that it, the future queue and what is
    // complete carry, and the time of all buckets.
    int cur_items = 0, cur_time = 0, cur_k = 0, fut_k = 0, done_k = 0, all_time = 0;
    if (queues) {
        chunks([&](int i0, int w, int) { all_time += i0 + lane < n ? w : 0; });
        all_time = bits_wave_sum(all_time);
    }
    bool to_row = false;
    for (int s = share > 1 ? wave : 0;; s += share) {
        if (s >= stages) {
            if (share == 1) break;
            __syncthreads();  // (the instance's other wavefronts have answered theirs)
            if (wave != 0) return;
            if (shared[31] == 0u) {
                kv_l = kl_l = lane < m ? (int)shared[lane] : 0;
                break;
            }
            to_row = true;
        }
        const int j = __builtin_amdgcn_readlane(ord_l, queues ? s & 1 : min(s, 63));
        int C = __builtin_amdgcn_readlane(cap_l, j);
        const int lane = bits_local(lane_);
        int case_now = 0, first_items = 0, first_time = 0;
        if (queues) {
            if (cur_items > 0 && (j == 0 || cur_time > C)) {
                case_now = j + 1;  // Case 1 / Case 2: Problem 1 over the current queue
            } else if (j == 1) {
                // Case 3 (the current queue fits and goes first) / Case 4 (it is empty): Algorithm 1 over this iteration's
                // buckets merged with the future queue, with what is left.  (Of its levels the whole list has
                // the greatest value, and the level that is returned selects the same.)
                case_now = cur_items > 0 ? 3 : 4;
                first_items = cur_items;
                first_time = cur_time;
                C -= cur_time;
                done_k += cur_k;
                cur_k = fut_k + 1;
                fut_k = 0;
                cur_items = n;
                cur_time = all_time;
                for (int i = lane; i < lay.mark_words; i += 64) l.marks[i] = 0xffffffffu;
                wave_lds_sync();
                if (long_list) list_weights();
            }
        }
        int value = 0, last = -1, got = 0;  // last: the item that completed the value
        // (a capacity sweep: every capacity is a stage of its own over the whole list)
        ExcessResult r = queues && case_now == 0 ? kExcessEmpty : kExcessNot;
        if constexpr (by_excess) {
            if (r == kExcessNot && !to_row && long_list) {
                r = excess_stage<NP>(list, lane, n, C, caps_sweep, value, last, [&](int i0, unsigned long long in) {
                    got += (int)__popcll(in);
                    if ((in >> lane) & 1ull) {
                        if (caps_sweep) {
                            atomicOr(&l.marks[i0 + lane], 1u << s);
                        } else {
                            mark8[i0 + lane] = (uint8_t)j;
                            l.prefix[i0 + lane] = kGone;
                        }
                    }
                });
                if (r == kExcessEmpty && !levels && !caps_sweep && !queues) break;  // every item is placed: the remaining stages stay empty
            }
            if (share > 1 && !to_row) {
                if (lane == 0) shared[r == kExcessNot ? 31 : s] = r == kExcessNot ? 1u : (uint32_t)value;
                if (r == kExcessNot) s = stages;
                continue;
            }
        }
        if (r == kExcessNot) {
            // the row's own sweep, over a list in LDS (in the place of the weights); for all capacities of a capacity sweep at once
            if (caps_sweep) C = cap_max;
            int cnt = 0, sum = 0;
            bool all_placed = true;
            if (lane == 0) l.prefix[0] = 0;
            chunks([&](int i0, int w, int) {
                const int i = i0 + lane;
                const bool open = i < n && (caps_sweep || mark8[i] == 0xff), offered = open && w <= C;
                all_placed = all_placed && __builtin_amdgcn_ballot_w64(open) == 0ull;
                const unsigned long long mask = __builtin_amdgcn_ballot_w64(offered);
                const int upto = sum + bits_wave_prefix_sum(offered ? w : 0, lane);  // (4096 weights of at most 65535)
                if (offered) {
                    const int pos = cnt + __popcll(mask & ((1ull << lane) - 1ull));
                    l.prefix[pos + 1] = upto;
                    l.index[pos] = (uint16_t)i;
                }
                cnt += __popcll(mask);
                sum = __builtin_amdgcn_readlane(upto, 63);
            });
            if (all_placed && !levels && !queues && !caps_sweep) break;  // every item is placed: the remaining stages stay empty
            wave_lds_sync();
            if (cnt == 0) {
                // nothing is offered
            } else if (sum <= C && !caps_sweep) {
                // everything offered fits together: the DP takes it all (every value is positive)
                for (int p = lane; p < cnt; p += 64) mark8[l.index[p]] = (uint8_t)j;
                value = sum;
                if (levels) last = l.index[cnt - 1];
            } else if (cnt <= kBitsEnumItems && !caps_sweep) {
                // A handful of items: lane x weighs the subset whose members are the set bits of x.  The
                // DP with its walk returns the feasible subset of greatest value and, among
                // equals, the one with the smallest such number.
                int ws = 0;
                for (int p = 0; p < cnt; ++p)
                    if ((lane >> p) & 1) ws += l.prefix[p + 1] - l.prefix[p];
                const bool feasible = lane < (1 << cnt) && ws <= C;
                value = bits_wave_max(feasible ? ws : -1);
                const int pick = __builtin_ctzll(__builtin_amdgcn_ballot_w64(feasible && ws == value));  // (the empty set is feasible)
                if (lane < cnt && ((pick >> lane) & 1)) mark8[l.index[lane]] = (uint8_t)j;
                if (levels) last = l.index[31 - __builtin_clz(pick | 1)];
            } else {
                const BitsStage g{cnt, C, j, m, cap_l, levels, caps_sweep};
                unsigned long long *counter = swept_cells ? swept_cells + (inst & (kBitsCounters - 1)) * kBitsCounterStride : nullptr;
                BitsAnswer r;
                if constexpr (EXCESS && !QUEUES && K * (NP + 1) > 60) r = bits_row_call<K, NP>(l, g, counter);
                else r = bits_row<K, NP>(l, lane, g, counter);
                if (caps_sweep) kv_l = kl_l = r.value;
                else value = r.value;
                if (levels) last = r.last;
                if (r.failed) status = DEFT_ERR_DEVICE;  // (never expected)
            }
            wave_lds_sync();
            if (caps_sweep) break;
            if (long_list && s + 1 < stages) list_weights();
            if (queues) {
                int open = 0;
                for (int i = lane; i < n; i += 64) open += mark8[i] == 0xff;
                got = cur_items - bits_wave_sum(open);
            }
        }
        wave_lds_sync();
        if constexpr (queues) {
            cur_items -= got;
            cur_time -= value;
            if (case_now == 2) fut_k += 1;  // the new buckets wait in the future queue
            if (case_now != 0 && cur_items == 0) {
                done_k += cur_k;
                cur_k = 0;
            }
            if (lane == 0) {
                q.stage_case[record0 + s] = case_now;
                q.stage_count[record0 + s] = case_now != 0 ? first_items + got : 0;
                q.stage_time[record0 + s] = case_now != 0 ? first_time + value : 0;
                if (j == 1) q.update_k[(record0 + s) / 2] = done_k;  // everything complete is applied in one update
            }
            if (j == 1) done_k = 0;
            continue;
        }
        if (lane == j) kv_l = kl_l = value;
        total += value;
        if (levels) {
            // Algorithm 1: level d keeps the first n - d items and the remaining time R less the drop
            // times of the others.  The levels' answers are nested (fewer items, less time), so the
            // whole list's value is the greatest, and the recursion's answer is the deepest level
            // that has it too: the smallest e such that the items before e reach it (e is beyond
            // the item that completed it) and the time left for them, R - sum of drop[t] over
            // t >= e, is not below it.  The remaining times grow with e: the list is searched from
            // its end, 64 entries at a time, until one falls short.  (R is at most 2^16: a drop time
            // is clamped just above 2^24 and so is the running sum, which keeps everything in 32
            // bits and exact wherever the remaining time is not negative.)
            constexpr int kOver = (1 << 24) + 1;
            int length = 0, remain = 0;
            if (value > 0) {
                length = n;
                remain = C;
                int behind = 0;
                for (int i0 = (n - 1) & ~63; i0 >= 0; i0 -= 64) {
                    const int e = i0 + lane;
                    const int x = bits_wave_suffix_sum(e < n ? min(drop[e], kOver) : 0, lane);
                    const int time_left = C - min(x + behind, kOver);
                    const unsigned long long hit = __builtin_amdgcn_ballot_w64(e > last && e < n && time_left >= value);
                    if (hit == 0ull) break;
                    length = i0 + __builtin_ctzll(hit);
                    remain = __builtin_amdgcn_readlane(time_left, __builtin_ctzll(hit));
                    if ((hit & 1ull) == 0ull) break;
                    behind = min(behind + __builtin_amdgcn_readlane(x, 0), kOver);
                }
            }
            if (lane == 1) {  // slot 1 reports the level: items left off the list, its remaining time
                kv_l = n - length;
                kl_l = remain;
            }
        }
    }
    if constexpr (queues) {
        if (lane < 2) q.tail[(size_t)inst * 2 + lane] = lane == 0 ? cur_k : fut_k;
        if (lane == 0) q.status[inst] = status;
        return;
    }
    if (caps_sweep) total = bits_wave_max(kv_l);

    for (int i = lane; i < a.item_stride; i += 64) {
        int asg = caps_sweep ? 0 : -1;
        if (i < n) asg = caps_sweep ? (int)l.marks[i] : (int)(int8_t)mark8[i];
        out_asg[i] = asg;
    }
    if (lane < a.knap_stride) {
        a.knap_value[(size_t)inst * a.knap_stride + lane] = kv_l;
        a.knap_load[(size_t)inst * a.knap_stride + lane] = kl_l;
    }
    if (lane == 0) {
        a.total_value[inst] = total;
        a.status[inst] = status;
    }
}

// Compiled words-per-lane counts (capacities up to 2048 K - 1) and plane counts (lists of up to
// 2^NP items).
constexpr int kBitsWords[] = {2, 5, 7, 10, 14, 20, 32};
constexpr int kNumBitsWords = 7;
constexpr int kBitsPlanes[] = {6, 9, 9, 12};  // (the second: lists too short for seq_excess.h)

template <bool QUEUES>
using BitsKernel = void (*)(BatchArgs, BitsQueueArgs<QUEUES>, BitsLayout, unsigned long long *);

// The kernel of a variant (4 times the index in kBitsWords, plus the index in kBitsPlanes), among those of the
// word counts W .. END - 1 that a translation unit compiles.
template <int W, int END, bool QUEUES>
const void *bits_kernel_of(int variant)
{
    if constexpr (W < END) {
        constexpr int K = kBitsWords[W];
        if (variant / 4 != W) return bits_kernel_of<W + 1, END, QUEUES>(variant);
        const BitsKernel<QUEUES> fn = variant % 4 == 0   ? &seq_bits_kernel<K, kBitsPlanes[0], QUEUES, false>
                              : variant % 4 == 1 ? &seq_bits_kernel<K, kBitsPlanes[1], QUEUES, false>
                              : variant % 4 == 2 ? &seq_bits_kernel<K, kBitsPlanes[2], QUEUES, true>
                                                 : &seq_bits_kernel<K, kBitsPlanes[3], QUEUES, true>;
        return reinterpret_cast<const void *>(fn);
    }
    return nullptr;
}
constexpr int kBitsShort = 3;  // word counts of the shorter rows

}  // namespace

}  // namespace deft
