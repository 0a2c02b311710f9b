// Instantiations of the persistent 1x1 kernel of bf16 part products.
#include "conv_b3_res.h"

namespace mg3m {

KernelFn conv_kernel_b3_res(bool fused) { return fused ? &conv_igemm_b3_res<true> : &conv_igemm_b3_res<false>; }

}  // namespace mg3m
