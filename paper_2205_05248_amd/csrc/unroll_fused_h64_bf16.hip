// Fused unroll: the instantiations for 64 hidden units, bf16 weights (see unroll_fused_kernel.h).
#include "unroll_fused_kernel.h"

namespace marl {

hipError_t launch_unroll_fused_h64_bf16(const FusedCall &call) { return fused_dispatch<64, 1>(call); }

}  // namespace marl
