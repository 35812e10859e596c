// The bit-set kernels of the task queues, longer rows (a translation unit of its own, compiled beside the others).
#include "seq_bits_kernel.h"

namespace deft {

const void *seq_bits_long_queues_kernel(int variant) { return bits_kernel_of<kBitsShort, kNumBitsWords, true>(variant); }

}  // namespace deft
