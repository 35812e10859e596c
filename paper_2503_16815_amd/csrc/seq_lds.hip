// Sequential mode with the capacity row resident in LDS: variant choice for the
// create-time limits, and the launch of the kernels in seq_lds_kernel.h.
#include "seq_lds_kernel.h"

namespace deft {

// LDS is handed out in granules of 1280 bytes, 128 of them per compute unit (measured:
// three 53760-byte workgroups run together on a CU, three 54016-byte ones do not, whatever
// the occupancy query says).
constexpr int kLdsGranule = 1280, kLdsGranulesPerCu = 128;

bool seq_lds_plan(int32_t max_capacity, int32_t max_items, int32_t max_knapsacks, int32_t max_batch,
                  int32_t lds_per_wg_bytes, SeqLdsPlan *plan)
{
    const int32_t n_pad = (max_items + 7) & ~7;  // list entries per stage (whole 64-byte lines)
    for (int i = 0; i < kNumVariants; ++i) {
        const Variant &v = variant_table<false>()[i];
        const int guard = v.guard;
        // register slots needed by lane 0, rounded up to whole chunks
        const int64_t slots = ((int64_t)max_capacity / v.threads + v.chunk) / v.chunk * v.chunk;
        if (slots > v.cells) continue;
        // after a stage's sweep the row's LDS stages the walk's data: two ints per list
        // entry and one 64-bit word per lane; a long item list on a short row gets the LDS
        // it needs for that, up to the variant's full row
        int64_t row_cells = slots * v.threads;
        const int64_t staging = 2 * (int64_t)n_pad + 2 * v.threads;
        if (row_cells < staging) row_cells = (staging + v.threads - 1) / v.threads * v.threads;
        if (row_cells > (int64_t)v.cells * v.threads) continue;
        const int64_t per_inst = (guard + row_cells) * 4;
        const int inst_per_wg = v.threads == 64 ? 4 : 1;
        const int64_t lds = per_inst * inst_per_wg;
        if (lds > lds_per_wg_bytes) continue;
        plan->variant = i;
        plan->threads = v.threads;
        plan->cells_per_thread = v.cells;
        plan->keep_words = (v.cells + 31) / 32;
        plan->guard_cells = guard;
        plan->row_cells = (int32_t)row_cells;
        plan->n_pad = n_pad;
        plan->lds_bytes = (int32_t)lds;
        plan->wg_threads = v.threads == 64 ? 256 : v.threads;
        plan->inst_per_wg = inst_per_wg;
        plan->wg_per_cu = 0;
        plan->keep_words_per_inst = (int64_t)max_items * plan->keep_words * v.threads;
        plan->keep_bytes = plan->keep_words_per_inst * 4 * max_batch;
        plan->scratch_bytes = plan->keep_bytes + (int64_t)max_batch * max_knapsacks * n_pad * (int64_t)sizeof(OfferedItem);
        return true;
    }
    return false;
}

hipError_t seq_lds_prepare(SeqLdsPlan *plan)
{
    int nb = 0;
    hipError_t e = prepare_variant<false>(*plan, &nb);
    if (e == hipSuccess) e = seq_lds_pool_prepare(*plan);
    if (e != hipSuccess) return e;
    const int by_lds = kLdsGranulesPerCu / ((plan->lds_bytes + kLdsGranule - 1) / kLdsGranule);
    plan->wg_per_cu = nb < by_lds ? nb : by_lds;
    return plan->wg_per_cu > 0 ? hipSuccess : hipErrorInvalidConfiguration;
}

// Calls that may have stages worth trying by enumeration (seq_lds_kernel.h) run the kernels that do: those of this many
// cells (items times capacity), and twice kPoolItems items or kPoolCells cells.  With unrelated values, us by the sweep and so:
// 6 instances of 380 items at capacity 18914 630 and 70, 212 of 600 at 6695 646 and 103, 3082 of 55 at 20469 1189 and 400,
// 2461 of 241 at 2529 390 and 180, 56 of 155 at 5108 110 and 40; 160 of 100 at 14000, values near the weights, 165 and 188,
// 8 of those 153 and 82, 1000 of them 468 and 314.  Below the line 160 of 66 at 9000 94 and 121, 7 of 123 at 3537 104 and 119,
// 476 of 402 at 699 264 and 287; calls of 16 to 24 us would pay 2 for the larger kernel.  Nor where the row's LDS does not
// hold the items and the shortest lists, so that no stage could be tried: 2048 of 700 items at 940, values the
// weights or less than three above them, 0.99 ms, and 1.08 on the larger kernel.
constexpr int64_t kPoolCallCells = 650000;

hipError_t seq_lds_launch(const SeqLdsPlan &p, const BatchArgs &a, void *scratch, hipStream_t st,
                          unsigned long long *swept_cells)
{
    const int64_t cells = (int64_t)a.item_stride * a.max_capacity;
    const bool room = (int64_t)p.row_cells * 4 >= pool_items_bytes(a.item_stride) + pool_space_bytes(a.item_stride, kPool);
    if (room && (cells >= kPoolCells || (a.item_stride >= 2 * kPoolItems && cells >= kPoolCallCells)))
        return seq_lds_pool_launch(p, a, scratch, st, swept_cells);
    return launch_variant<false>(p, a, scratch, st, swept_cells);
}

}  // namespace deft
