// The fused projection, bf16 weights, and its dispatch by weight type (the
// kernel: proj_conv_kernel.hpp; the fp8 instances: proj_conv_fp8.hip).
#include "proj_conv_kernel.hpp"

namespace sr {

hipError_t launch_proj_conv(int weight_dtype, int d_head, const ProjConvBatch& b, hipStream_t s) {
  if (b.n_layers < 1 || b.n_layers > kProjBatch) return hipErrorInvalidValue;
  for (int l = 1; l < b.n_layers; ++l)
    if (b.layer[l].T != b.layer[0].T || b.layer[l].K != b.layer[0].K || b.layer[l].N != b.layer[0].N)
      return hipErrorInvalidValue;
  if (weight_dtype == SR_BF16) return by_head<bf16_t>(d_head, b, s);
  if (weight_dtype == SR_FP8_E4M3) return launch_proj_conv_fp8(d_head, b, s);
  return hipErrorInvalidValue;
}

hipError_t launch_proj_conv(int weight_dtype, int d_head, const ProjConvArgs& a, hipStream_t s) {
  ProjConvBatch b{};
  b.layer[0] = a;
  b.n_layers = 1;
  b.tq_off[1] = a.tq_blocks;
  return launch_proj_conv(weight_dtype, d_head, b, s);
}

}  // namespace sr
