// Fused unroll: the instantiations for 64 hidden units, fp32 weights (see unroll_fused_kernel.h).
#include "unroll_fused_kernel.h"

namespace marl {

hipError_t launch_unroll_fused_h64_f32(const FusedCall &call) { return fused_dispatch<64, 2>(call); }

}  // namespace marl
