// HIP-event timing of solve calls: one pair of events around each call and one
// pair around every launch of the DP sweep kernel, all recorded on the caller's
// stream; nothing is waited for until the figures are read.  And the count of the cells that the
// job's sweeps go through where the bit-set kernels answered, which mostly do without.
#include <new>

#include "kernels.h"

namespace deft {

hipEvent_t Profiler::Pool::get(int i)
{
    if (i >= cap) {
        int ncap = cap ? cap : 64;
        while (ncap <= i) ncap *= 2;
        hipEvent_t *n = new (std::nothrow) hipEvent_t[ncap];
        if (!n) return nullptr;
        for (int k = 0; k < cap; ++k) n[k] = ev[k];
        for (int k = cap; k < ncap; ++k) {
            if (hipEventCreate(&n[k]) != hipSuccess) {
                (void)hipGetLastError();
                for (int z = cap; z < k; ++z) (void)hipEventDestroy(n[z]);
                delete[] n;
                return nullptr;
            }
        }
        delete[] ev;
        ev = n;
        cap = ncap;
    }
    return ev[i];
}

void Profiler::Pool::destroy()
{
    for (int k = 0; k < cap; ++k) (void)hipEventDestroy(ev[k]);
    delete[] ev;
    ev = nullptr;
    cap = 0;
}

void Profiler::record(Pool &p, int idx, hipStream_t st)
{
    hipEvent_t e = p.get(idx);
    if (!e || hipEventRecord(e, st) != hipSuccess) {
        (void)hipGetLastError();
        failed_ = true;
    }
}

bool Profiler::begin(hipStream_t st)
{
    record(call_, ncall_, st);
    if (failed_) return false;
    ++ncall_;
    return true;
}

void Profiler::end(hipStream_t st)
{
    record(call_, ncall_, st);
    ++ncall_;
}

void Profiler::sweep_begin(hipStream_t st)
{
    record(sweep_, nsweep_, st);
    ++nsweep_;
}

void Profiler::sweep_end(hipStream_t st) { sweep_begin(st); }

void Profiler::counted(hipStream_t st)
{
    record(count_, 0, st);
    counted_ = true;
}

deft_status_t Profiler::read(deft_knapsack_profile_t *out)
{
    if (ncall_ < 2 || (ncall_ & 1) || (nsweep_ & 1)) return DEFT_ERR_INVALID_ARG;
    if (failed_) { reset(); return DEFT_ERR_DEVICE; }
    deft_status_t rc = DEFT_OK;
    float total = 0.f, sweep = 0.f;
    if (hipEventSynchronize(call_.ev[ncall_ - 1]) != hipSuccess) rc = DEFT_ERR_DEVICE;
    if (counted_ && hipEventSynchronize(count_.ev[0]) != hipSuccess) rc = DEFT_ERR_DEVICE;
    for (int i = 0; rc == DEFT_OK && i < ncall_; i += 2) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, call_.ev[i], call_.ev[i + 1]) != hipSuccess) rc = DEFT_ERR_DEVICE;
        total += ms;
    }
    for (int i = 0; rc == DEFT_OK && i < nsweep_; i += 2) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, sweep_.ev[i], sweep_.ev[i + 1]) != hipSuccess) rc = DEFT_ERR_DEVICE;
        sweep += ms;
    }
    if (rc != DEFT_OK) (void)hipGetLastError();
    out->total_ms = total;
    out->sweep_ms = sweep;
    out->sweep_launches = nsweep_ / 2;
    out->other_ms = total - sweep;
    reset();
    return rc;
}

void Profiler::destroy()
{
    call_.destroy();
    sweep_.destroy();
    count_.destroy();
    reset();
}

namespace {

__device__ __forceinline__ int count_sum(int x)
{
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
    return x;
}

// C - w + 1 for every item that the sweep of a stage goes through: its list up to where it sees that C (every capacity of a
// capacity sweep) can be reached, which is with the last item of the selection; it looks after every eighth item, every
// second one of a list of at most 64.  Nothing for stages whose list fits together or holds at most six items.  All of
// it follows from the outputs.  A wavefront per instance, outside the timed part of a profiled call.
__global__ void __launch_bounds__(256) bits_count_sweeps(BatchArgs a, unsigned long long *cells)
{
    constexpr int kFewest = 7;
    const int inst = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (inst >= a.batch || a.status[inst] != DEFT_OK || (a.left && a.left[inst] != 0)) return;
    const bool caps_sweep = a.mode == DEFT_MODE_CAPACITY_SWEEP;
    const int n = a.n_items[inst], m = a.n_knapsacks[inst];
    const int32_t *W = a.weights + (size_t)inst * a.item_stride, *asg = a.assignment + (size_t)inst * a.item_stride;
    const int32_t *cap = a.capacities + (size_t)inst * a.knap_stride, *val = a.knap_value + (size_t)inst * a.knap_stride;
    const int32_t *ord = a.fill_order ? a.fill_order + (size_t)inst * a.knap_stride : nullptr;
    unsigned long long total = 0, open = ~0ull;  // open: the knapsacks that this stage and those after it fill
    for (int s = 0; s < (caps_sweep ? min(m, 1) : m); ++s) {
        const int j = ord ? ord[s] : s;
        int C = cap[j];
        bool reached = val[j] == C;
        for (int k = 1; caps_sweep && k < m; ++k) C = max(C, cap[k]), reached = reached && val[k] == cap[k];
        auto listed = [&](int i) {
            return i < n && W[i] <= C && (caps_sweep || asg[i] < 0 || ((open >> asg[i]) & 1ull) != 0);
        };
        auto taken = [&](int i) { return i < n && (caps_sweep ? asg[i] != 0 : asg[i] == j); };
        int last = -1, cnt = 0, upto = 0, sum = 0, weight = 0;
        for (int i0 = 0; i0 < n; i0 += 64) {
            const unsigned long long mine = __ballot(taken(i0 + lane));
            if (mine != 0ull) last = i0 + 63 - (int)__builtin_clzll(mine);
        }
        for (int i0 = 0; i0 < n; i0 += 64) {
            const int i = i0 + lane;
            const unsigned long long in = __ballot(listed(i));
            cnt += (int)__popcll(in);
            upto += (int)__popcll(in & __ballot(i <= last));
            sum += count_sum(listed(i) ? W[i] : 0);
        }
        if (caps_sweep ? cnt > 0 : sum > C && cnt >= kFewest) {
            const int look = !caps_sweep && cnt <= 64 ? 2 : 8;
            const int items = reached ? min(cnt, (upto + look - 1) / look * look) : cnt;
            for (int i0 = 0, before = 0; i0 < n; i0 += 64) {
                const unsigned long long in = __ballot(listed(i0 + lane));
                const int rank = before + (int)__popcll(in & ((1ull << lane) - 1ull));
                weight += count_sum(((in >> lane) & 1ull) != 0 && rank < items ? W[i0 + lane] : 0);
                before += (int)__popcll(in);
            }
            total += (unsigned long long)items * (unsigned)(C + 1) - (unsigned long long)(unsigned)weight;
        }
        open &= ~(1ull << j);
    }
    if (lane == 0 && total != 0) atomicAdd(cells, total);
}

}  // namespace

hipError_t bits_count_launch(const BatchArgs &a, hipStream_t st, unsigned long long *cells)
{
    hipLaunchKernelGGL(bits_count_sweeps, dim3((unsigned)((a.batch + 3) / 4)), dim3(256), 0, st, a, cells);
    return hipGetLastError();
}

}  // namespace deft
