// Instantiations of the kernel that takes fp32 products as bf16 part products,
// one per tile shape.
#include "conv_b3.h"

namespace mg3m {

KernelFn conv_kernel_b3(int tile) { return pick_b3<false>(tile, std::make_integer_sequence<int, kNumTilesB3>{}); }

}  // namespace mg3m
