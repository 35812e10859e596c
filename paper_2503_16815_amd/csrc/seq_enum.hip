// The sequential mode by enumeration (seq_enum.h) ahead of the streamed rows: one wavefront per instance goes through all
// its stages; an instance with a stage that is not settled is left to the rows as a whole.
// Measured, the two launches of a call against the streamed sweep alone: 256 GPT-2 instances in 1 us units (C = 381000)
// 2.31 -> 0.19 ms, in 10 us units (C = 38100) 0.45 -> 0.18, nine in 1 us units 1.69 -> 0.06.  What bounds it is the
// instance with the most to look through (the median is done after 40 us).
#include "instance_check.h"
#include "seq_enum.h"

namespace deft {

namespace {

__global__ void __launch_bounds__(64) seq_enum_kernel(BatchArgs a, int space_bytes)
{
    extern __shared__ __align__(16) char lds_pool[];
    const int inst = blockIdx.x, lane = threadIdx.x;
    const int status = check_instance(a, inst, false);
    clear_outputs(a, inst, status);
    if (lane == 0) a.left[inst] = 0;
    if (status != DEFT_OK) return;
    const int n = a.n_items[inst], m = a.n_knapsacks[inst];
    const int32_t *W = a.weights + (size_t)inst * a.item_stride;
    const int32_t *V = a.values + (size_t)inst * a.item_stride;
    const int32_t *cap = a.capacities + (size_t)inst * a.knap_stride;
    int2 *items = reinterpret_cast<int2 *>(lds_pool);
    char *space = lds_pool + pool_items_bytes(n);
    const int chunks = (n + 63) >> 6;
    unsigned long long open = 0;  // bit c of a lane: item 64 c + lane is not placed and worth something
    bool related = true;          // every value is its weight: all selections that fill a window are as good
    for (int c = 0; c < chunks; ++c) {
        const int i = c * 64 + lane;
        const int2 it = i < n ? make_int2(W[i], V[i]) : make_int2(1, 0);
        items[i] = it;
        if (it.y > 0) open |= 1ull << c;
        related = related && (i >= n || it.x == it.y);
    }
    if (__ballot(!related) == 0ull) {
        if (lane == 0) a.left[inst] = 1;
        return;
    }
    pool_sync();
    long long total = 0, deadline = wall_clock64();
    for (int s = 0; s < m; ++s) {
        const int j = a.fill_order ? a.fill_order[(size_t)inst * a.knap_stride + s] : s;
        const int C = cap[j];
        if (__ballot(open != 0) == 0ull) break;  // the remaining stages stay empty
        // Half of what the sweep of a stage takes where it takes least, 4 us an item and 2 for every 100000 cells more
        // (a tick is 10 ns).
        deadline += (long long)n * (200 + C / 1000);
        PoolAnswer answer;
        if (!pool_solve(items, space, space_bytes, INT_MAX, n, C, open, deadline, lane, answer)) {
            if (lane == 0) a.left[inst] = 1;
            return;
        }
        open &= ~answer.chosen;
        for (unsigned long long bits = answer.chosen; bits; bits &= bits - 1)
            a.assignment[(size_t)inst * a.item_stride + __builtin_ctzll(bits) * 64 + lane] = j;
        if (lane == j) {
            a.knap_value[(size_t)inst * a.knap_stride + j] = answer.value;
            a.knap_load[(size_t)inst * a.knap_stride + j] = answer.load;
        }
        total += answer.value;
    }
    if (lane == 0) a.total_value[inst] = total;
}

// How long the lists may get.  A batch of no more instances than compute units: as long as an LDS holds.  Else two
// instances share one.  (Of GPT-2 windows one in a hundred needs more than 512 entries, one in three hundred more than 1280.)
constexpr int kEntriesAlone = 3000, kEntriesShared = 1280;
int enum_entries(int items, int batch, int compute_units)
{
    const int room = (160 * 1024 - 512 - pool_items_bytes(items) - pool_space_bytes(items, 0)) / (3 * kPoolEntryBytes);
    const int entries = batch <= compute_units ? kEntriesAlone : kEntriesShared;
    return entries < room ? entries : room;
}


}  // namespace

hipError_t seq_enum_prepare()
{
    // (the attribute belongs to the kernel, not to the handle: a compute unit's LDS less what check_instance takes)
    return hipFuncSetAttribute(reinterpret_cast<const void *>(&seq_enum_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                               160 * 1024 - 512);
}

hipError_t seq_enum_launch(const BatchArgs &a, int32_t compute_units, hipStream_t st)
{
    const int space = pool_space_bytes(a.item_stride, enum_entries(a.item_stride, a.batch, compute_units));
    hipLaunchKernelGGL(seq_enum_kernel, dim3((unsigned)a.batch), dim3(64), (size_t)(pool_items_bytes(a.item_stride) + space), st, a, space);
    return hipGetLastError();
}

}  // namespace deft
