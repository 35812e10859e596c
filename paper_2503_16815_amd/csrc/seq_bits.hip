// The bit-set kernels (seq_bits_kernel.h) for the shorter rows, and the plan and launch all of
// them share.
#include "seq_bits_kernel.h"

namespace deft {

namespace {

// LDS is handed out in granules of 1280 bytes, 128 of them per compute unit.
constexpr int kLdsGranule = 1280, kLdsGranulesPerCu = 128;

BitsLayout bits_layout(const SeqBitsPlan &p, bool caps_sweep)
{
    BitsLayout lay;
    lay.row_words = p.row_words;
    lay.n_pad = p.n_pad;
    lay.mark_words = caps_sweep ? p.n_pad : p.n_pad / 4;
    lay.plane_words = p.row_words * bits_plane_stride(p.planes);
    lay.share = 1;
    lay.turns = 1;
    lay.wave_words = 2 * p.row_words + 4 + (p.n_pad + 8) + p.n_pad / 2 + lay.mark_words;
    return lay;
}

int64_t bits_lds_bytes(const BitsLayout &lay, int waves)
{
    return ((int64_t)4 + lay.plane_words + (int64_t)waves * lay.wave_words) * 4;
}

// The planes that a call's lists of up to `items` need (index in kBitsPlanes); `fewest`: from so many on, stages by what they
// leave out.  By the call and not by the handle, whose lists may be longer elsewhere: planes cost registers and LDS, and those
// stages cost the row's sweep its registers where they are never tried.  8192 instances on a handle for 314 items, us with the handle's kernel and the call's: 80 items
// SEQUENTIAL 121 and 94, RECURSIVE 96 and 68, CAPACITY_SWEEP 106 and 80; 38 items 61 and 43; a sweep of 128 items 130 and 102.
int bits_which(int items, int fewest) { return items <= 64 ? 0 : items > 512 ? 3 : items < fewest ? 1 : 2; }

void bits_lists(SeqBitsPlan *p, int items, int fewest)
{
    const int which = bits_which(items, fewest);
    p->variant = p->variant / 4 * 4 + which;
    p->planes = kBitsPlanes[which];
    p->n_pad = (items + 7) & ~7;
}

// Instances a compute unit holds when `waves` of them share a workgroup (0: they do not fit).
int bits_per_cu(const SeqBitsPlan &p, int64_t lds, int waves)
{
    if (lds > p.lds_limit) return 0;
    const int by_lds = kLdsGranulesPerCu / (int)((lds + kLdsGranule - 1) / kLdsGranule) * waves;
    const int by_regs = 4 * bits_waves_per_simd(p.words_per_lane, p.planes) / waves * waves;
    return by_lds < by_regs ? by_lds : by_regs;
}

const void *bits_kernel(const SeqBitsPlan &p, bool queues)
{
    if (p.variant >= 4 * kBitsShort) return seq_bits_long_kernel(p.variant, queues);
    return queues ? seq_bits_queues_kernel(p.variant) : bits_kernel_of<0, kBitsShort, false>(p.variant);
}

}  // namespace

bool seq_bits_plan(int32_t max_capacity, int32_t max_items, int32_t lds_per_wg_bytes, int32_t compute_units, SeqBitsPlan *p)
{
    for (int i = 0; i < kNumBitsWords; ++i) {
        const int K = kBitsWords[i];
        if ((int64_t)max_capacity > (int64_t)K * 2048 - 1) continue;
        const int grain = bits_grain(K);
        p->variant = 4 * i;
        p->words_per_lane = K;
        bits_lists(p, max_items, kBitsExcessItems);
        p->row_words = (max_capacity / 2048 + grain) / grain * grain * 64;
        p->lds_limit = lds_per_wg_bytes - 256;
        p->compute_units = compute_units;
        p->lds_bytes = (int32_t)bits_lds_bytes(bits_layout(*p, true), 1);
        return p->lds_bytes <= p->lds_limit;
    }
    return false;
}

hipError_t seq_bits_prepare(const SeqBitsPlan &p)
{
    // the attribute belongs to the kernel, not to the handle: the most any handle may ask for
    // (a compute unit's LDS less a small allowance)
    for (SeqBitsPlan q = p; q.variant >= p.variant / 4 * 4; --q.variant) {  // (shorter lists have kernels of their own)
        for (const bool queues : {false, true}) {
            const hipError_t e = hipFuncSetAttribute(bits_kernel(q, queues), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - 256);
            if (e != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

namespace {

template <bool QUEUES>
hipError_t bits_launch(SeqBitsPlan p, const BatchArgs &a, const BitsQueueArgs<QUEUES> &q, hipStream_t st, unsigned long long *swept_cells)
{
    const bool caps_sweep = a.mode == DEFT_MODE_CAPACITY_SWEEP;
    bits_lists(&p, a.item_stride, kBitsExcessItems);
    BitsLayout lay = bits_layout(p, caps_sweep);
    const auto launch = [&](unsigned blocks, int waves) {
        const auto kernel = reinterpret_cast<BitsKernel<QUEUES>>(const_cast<void *>(bits_kernel(p, QUEUES)));
        const size_t lds = (size_t)bits_lds_bytes(lay, lay.share > 1 ? 1 : waves);
        hipLaunchKernelGGL(kernel, dim3(blocks), dim3(64 * waves), lds, st, a, q, lay, swept_cells);
        return hipGetLastError();
    };
    if (caps_sweep && a.item_stride >= kBitsExcessItems) {
        // Lists that are answered capacity by capacity: as many wavefronts an instance, up to four, as the whole batch leaves
        // room for.  1024 instances of 314 items and eleven capacities: one 79 us, three 38.
        const int by_lds = kLdsGranulesPerCu / (int)((bits_lds_bytes(lay, 1) + kLdsGranule - 1) / kLdsGranule);
        int share = a.knap_stride < 4 ? a.knap_stride : 4;
        for (; share > 1; --share) {
            const int by_regs = 4 * bits_waves_per_simd(p.words_per_lane, p.planes) / share;
            if ((int64_t)(by_lds < by_regs ? by_lds : by_regs) * p.compute_units >= a.batch) break;
        }
        lay.turns = (int16_t)((a.knap_stride + share - 1) / share);
        const int fewest = bits_tried_caps(lay.turns, p.words_per_lane).fewest;
        if (a.item_stride >= fewest && share > 1) {
            lay.share = (int16_t)share;
            return launch((unsigned)a.batch, share);
        }
        if (a.item_stride < fewest) {
            bits_lists(&p, a.item_stride, fewest);
            lay = bits_layout(p, caps_sweep);
        }
    }
    // Instances per workgroup: they share one copy of the walk's planes, the largest part of an
    // instance's LDS, but walk one at a time.  So: as few as still let the whole batch run at
    // once, else as many as put the most instances on a compute unit.
    int waves = 1, most = 0;
    for (const int w : {1, 2, 4}) {
        const int64_t lds = bits_lds_bytes(lay, w);
        const int held = bits_per_cu(p, lds, w);
        if (held > most) most = held, waves = w;
        if ((int64_t)held * p.compute_units >= a.batch) break;
    }
    return launch((unsigned)((a.batch + waves - 1) / waves), waves);
}

}  // namespace

hipError_t seq_bits_launch(const SeqBitsPlan &p, const BatchArgs &a, hipStream_t st, unsigned long long *swept_cells)
{
    return bits_launch<false>(p, a, BitsNoArgs{}, st, swept_cells);
}

hipError_t seq_bits_queues_launch(const SeqBitsPlan &p, const ScheduleArgs &q, hipStream_t st, unsigned long long *swept_cells)
{
    BatchArgs a{};
    a.mode = DEFT_MODE_SEQUENTIAL;
    a.batch = q.batch;
    a.item_stride = q.n_buckets;
    a.knap_stride = 2;
    a.max_capacity = q.max_capacity;
    a.weights = a.values = q.comm_time;  // the value of a bucket is its communication time
    a.drop_time = q.drop_time;
    return bits_launch<true>(p, a, q, st, swept_cells);
}

}  // namespace deft
