// The bit-set kernels of the longer rows: a translation unit of their own, compiled beside the
// shorter ones.
#include "seq_bits_kernel.h"

namespace deft {

const void *seq_bits_long_kernel(int variant, bool queues)
{
    return queues ? seq_bits_long_queues_kernel(variant) : bits_kernel_of<kBitsShort, kNumBitsWords, false>(variant);
}

}  // namespace deft
