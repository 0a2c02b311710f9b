// Instantiations of the kernel that takes fp32 products as bf16 part products:
// the forms for any number of channels (HWCN).
#include "conv_b3.h"

namespace mg3m {

KernelFn conv_kernel_b3_any(int load, int tile) {
  switch (load) {
    case kB3Group: return b3_kernel_for_tile<kB3Group, false>(tile);
    case kB3GroupN: return b3_kernel_for_tile<kB3GroupN, false>(tile);
    case kB3GroupC: return b3_kernel_for_tile<kB3GroupC, false>(tile);
    case kB3Row: return b3_kernel_for_tile<kB3Row, false>(tile);
    case kB3RowN: return b3_kernel_for_tile<kB3RowN, false>(tile);
    default: return nullptr;
  }
}

}  // namespace mg3m
