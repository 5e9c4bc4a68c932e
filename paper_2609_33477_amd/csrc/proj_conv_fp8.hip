// The fused projection's fp8-weight instances (compiled apart from the bf16
// ones: each takes a minute).
#include "proj_conv_kernel.hpp"

namespace sr {

hipError_t launch_proj_conv_fp8(int d_head, const ProjConvBatch& b, hipStream_t s) { return by_head<fp8_t>(d_head, b, s); }

}  // namespace sr
