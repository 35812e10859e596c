// The sequential mode on the LDS-resident row with stages tried by enumeration first: the kernels of
// seq_lds_kernel.h instantiated with POOL = true, under the same plan and scratch.
#include "seq_lds_kernel.h"

namespace deft {

hipError_t seq_lds_pool_prepare(const SeqLdsPlan &plan)
{
    if (plan.threads == 64) return hipSuccess;  // (no such kernel)
    int nb = 0;
    const hipError_t e = prepare_variant<false, true>(plan, &nb);
    if (e != hipSuccess) return e;
    return nb > 0 ? hipSuccess : hipErrorInvalidConfiguration;
}

hipError_t seq_lds_pool_launch(const SeqLdsPlan &p, const BatchArgs &a, void *scratch, hipStream_t st,
                               unsigned long long *swept_cells)
{
    return launch_variant<false, true>(p, a, scratch, st, swept_cells);
}

}  // namespace deft
