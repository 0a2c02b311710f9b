// Instantiations of the kernel of bf16 part products with the fused output
// stage (add, ReLU), one per tile shape.
#include "conv_b3.h"

namespace mg3m {

KernelFn conv_kernel_b3_fused(int tile) {
  return pick_b3<true>(tile, std::make_integer_sequence<int, kNumTilesB3>{});
}

}  // namespace mg3m
