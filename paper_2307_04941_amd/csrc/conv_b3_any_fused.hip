// Instantiations of the kernel that takes fp32 products as bf16 part products, with the fused output stage:
// the forms for any number of channels (HWCN).
#include "conv_b3.h"

namespace mg3m {

KernelFn conv_kernel_b3_any_fused(int load, int tile) {
  switch (load) {
    case kB3Group: return b3_kernel_for_tile<kB3Group, true>(tile);
    case kB3GroupN: return b3_kernel_for_tile<kB3GroupN, true>(tile);
    case kB3GroupC: return b3_kernel_for_tile<kB3GroupC, true>(tile);
    case kB3Row: return b3_kernel_for_tile<kB3Row, true>(tile);
    case kB3RowN: return b3_kernel_for_tile<kB3RowN, true>(tile);
    default: return nullptr;
  }
}

}  // namespace mg3m
