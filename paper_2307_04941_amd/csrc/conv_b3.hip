// Instantiations of the kernel that takes fp32 products as bf16 part products:
// the forms whose stages are one filter tap, HWCN and NCHW.
#include "conv_b3.h"

namespace mg3m {

KernelFn conv_kernel_b3(int load, int tile) {
  switch (load) {
    case kB3Slab: return b3_kernel_for_tile<kB3Slab, false>(tile);
    case kB3SlabW: return b3_kernel_for_tile<kB3SlabW, false>(tile);
    default: return conv_kernel_b3_any(load, tile);
  }
}

}  // namespace mg3m
