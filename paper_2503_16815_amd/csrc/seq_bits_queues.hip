// The bit-set kernels of the task queues, shorter rows (a translation unit of its own, compiled beside the others).
#include "seq_bits_kernel.h"

namespace deft {

const void *seq_bits_queues_kernel(int variant) { return bits_kernel_of<0, kBitsShort, true>(variant); }

}  // namespace deft
