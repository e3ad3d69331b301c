// Fused unroll: which networks it serves, and the dispatch to the per-shape instantiations (unroll_fused_h128.hip,
// unroll_fused_h64_bf16.hip, unroll_fused_h64_f32.hip; the kernel is unroll_fused_kernel.h).
#include "unroll_fused_kernel.h"

namespace marl {

namespace {

template <int H, int P> bool fits(const NetFrags &net)
{
    const int ks1 = obs_k_steps(P, net.D);
    return ks1 <= Fused16<H, P>::kKs1Max && unroll_lds_bytes<H, P>(ks1) <= (size_t)kLdsLimit;
}

}  // namespace

bool unroll_fused_fits(const NetFrags &net)
{
    if (net.A > 64) return false;
    if (net.H == 64 && net.planes == 2) return fits<64, 2>(net);
    if (net.H == 64 && net.planes == 1) return fits<64, 1>(net);
    if (net.H == 128 && net.planes == 1) return fits<128, 1>(net);
    return false;      // H = 128 with fp32 weights: W_ih alone exceeds a compute unit's LDS
}

hipError_t launch_unroll_fused(const NetFrags &online, const NetFrags &target, bool two_nets, int B, int T,
                               const int32_t *episode_index, int pool_episodes, const float *obs, const uint8_t *avail, const int32_t *actions, const float *reward,
                               const uint8_t *terminated, const uint8_t *filled, float gamma, float *q_taken,
                               float *next_max, float *td_target, float *q_all, hipStream_t stream, TdMode mode,
                               int32_t *next_action, float *h_save, void *x_save, const NextQ &next_q)
{
    if ((mode == kTdSelect || mode == kTdValue) && (two_nets || !next_action)) return hipErrorInvalidValue;
    if (mode == kTdDouble && (!two_nets || !next_action || !next_q.q)) return hipErrorInvalidValue;
    if (mode == kTdSave && (two_nets || !h_save || !x_save)) return hipErrorInvalidValue;
    if (mode == kTdKeep && (!h_save || !x_save)) return hipErrorInvalidValue;
    const FusedCall call{online, target, two_nets, B, T, episode_index, pool_episodes, obs, avail, actions, reward, terminated, filled, gamma,
                         q_taken, next_max, td_target, q_all, stream, mode, next_action, h_save, x_save, next_q};
    if (online.H == 64 && online.planes == 2) return launch_unroll_fused_h64_f32(call);
    if (online.H == 64 && online.planes == 1) return launch_unroll_fused_h64_bf16(call);
    if (online.H == 128 && online.planes == 1) return launch_unroll_fused_h128(call);
    return hipErrorInvalidValue;
}

}  // namespace marl
