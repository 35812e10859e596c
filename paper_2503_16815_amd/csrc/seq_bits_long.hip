// The bit-set kernels of the longer rows: a translation unit of their own, compiled beside the
// shorter ones.
#include "seq_bits_kernel.h"

namespace deft {

void *seq_bits_long_kernel(int variant)
{
    BitsKernel fn = nullptr;
    switch (variant) {
    case 9: fn = &seq_bits_kernel<10, 6>; break;
    case 10: fn = &seq_bits_kernel<10, 9>; break;
    case 11: fn = &seq_bits_kernel<10, 12>; break;
    case 12: fn = &seq_bits_kernel<14, 6>; break;
    case 13: fn = &seq_bits_kernel<14, 9>; break;
    case 14: fn = &seq_bits_kernel<14, 12>; break;
    case 15: fn = &seq_bits_kernel<20, 6>; break;
    case 16: fn = &seq_bits_kernel<20, 9>; break;
    case 17: fn = &seq_bits_kernel<20, 12>; break;
    case 18: fn = &seq_bits_kernel<32, 6>; break;
    case 19: fn = &seq_bits_kernel<32, 9>; break;
    case 20: fn = &seq_bits_kernel<32, 12>; break;
    default: break;
    }
    return reinterpret_cast<void *>(fn);
}

}  // namespace deft
