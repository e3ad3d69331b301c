// Recurrence of the two-kernel unroll on tiles of 16 (episode, agent) rows: 128 hidden units, fp32.  The gate inputs
// W_ih x + b of every slot lie in the scratch buffer that the input projection has written (kernels.hip); one workgroup
// walks the T+1 slots of its tile for one network.
//
// What bounds it is the chain h -> W_hh h -> gates -> h, once per slot: two planes of W_hh (192 KB) fit the registers
// of eight waves (96 each, one block of 16 hidden units per wave, two waves per SIMD) but not those of four, which is
// what tiles of 32 rows with 32 hidden units per wave asked for: that form spilled.  A wave reads its own gate inputs
// from memory, a slot ahead, and adds them after the products, so that the loads have a slot and the products to
// arrive; a wave of its own touches the lines a few slots earlier, so that they come from L2.  No LDS for them, and
// one LDS-only barrier per slot.  Double-estimator targets of 61 episodes x 70 slots x 5 agents: 543 us with the form on 32 rows, 209
// with this one (one network after the other, two projections of 27 us included), 118 with both networks in one launch,
// of which the recurrence is 91, 1.3 us a slot.
//
// Eleven waves leave a wave 168 registers, too few for the epilogue of 49 to 64 actions: 10 to 13 registers of its wave spill,
// 39 and 56 where it also keeps the target's Q values (with 33 to 48 actions 2 and 4 there).  The case above with 48 / 49 actions:
// 150 / 218 us, and 171 / 350 with q_all; 629 / 628 and 729 / 733 with the form on 32 rows.
//
// Wave roles, in the step of slot s:  0..7 the recurrence of slot s;  8 fc2 and the TD step of slot s-1;  9 the
// per-slot inputs of the TD step of slot s;  10 the touches of slot s + 1 + kTouchAhead.
#include <hip/hip_runtime.h>

#include "unroll16_td.h"

namespace marl {

namespace {

struct Recur16 {
    static constexpr int H = 128, P = 2, KS = H / 32, FBK = H / 16;
    static constexpr int NC = FBK;                                    // recurrence waves
    static constexpr int kEpilogue = NC, kToucher = NC + 2, kWaves = NC + 3;
    static constexpr int kGateBytes = (H / 32) * GiLayout<P>::kBlockBytes, kSlotBytes = 3 * kGateBytes;      // of 32 rows
    static constexpr int kLead = 1;
};

}  // namespace

// The gate inputs carry no __restrict__: under kTdDouble the target network's Q values go where they were (td.next_q.q is
// gi_target).  A workgroup stores to its half of the record of slot t in step t + 1.  Its recurrence waves have asked for the gate
// inputs there in step t - 1 and used them in step t, before the barrier that ends it; what reads the record later (the last slot
// again in step T, the touches past the end) uses nothing of it.
template <int AB, bool QALL, int MODE>
__global__ __launch_bounds__(64 * Recur16::kWaves, 3) void recurrent16_td_kernel(NetFrags online, NetFrags target, const char *gi_online,
                                                                                 const char *gi_target, int two_nets, int B, int T,
                                                                                 TdArrays td)
{
    using Sh = Recur16;
    constexpr int H = Sh::H, P = Sh::P, KS = Sh::KS, LEAD = Sh::kLead;
    constexpr bool kValue = MODE == kTdValue, kDouble = MODE == kTdDouble;
    __shared__ bf16x8 h_lds[2][KS][P][64];
    __shared__ __attribute__((aligned(16))) char epi_lds[kEpiBytes];
    __shared__ __attribute__((aligned(16))) float b2_lds[64];

    const bool is_target = blockIdx.y == 1;
    const NetFrags net = is_target ? target : online;
    const int lane = threadIdx.x & 63, q4 = lane >> 4, c = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int N = net.N, A = net.A, S = T + 1;
    const int rt = blockIdx.x, rows = B * N;
    // the scratch buffer is cut into records of (32 rows, slot): this tile is one half of each of its own
    const char *const gi_tile = (is_target ? gi_target : gi_online) + (size_t)(rt >> 1) * S * Sh::kSlotBytes;
    const int half = rt & 1;

    if (wave < Sh::NC) {
        // ---------------------------------------------------------------- recurrence wave: hidden units 16 w .. 16 w + 15
        const int w = wave;
        WFrag<P> whh[3][KS];
#pragma unroll
        for (int gate = 0; gate < 3; ++gate)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                whh[gate][ks] = load_wfrag<P>(net.whh_16 + ((size_t)((gate * Sh::FBK + w) * KS + ks) * P) * 64 + lane);
        const f32x4 bias_hn = load_feature4(net.bias_hn, w, q4);
        // GiLayout<2>: features 32 blk + 8 j + 4 g + 0..3 of row m at block blk, vector j, lane 32 g + m
        const uint32_t gi_lane = (uint32_t)((w >> 1) * GiLayout<P>::kBlockBytes + (2 * (w & 1) + (q4 >> 1)) * 1024
                                            + ((q4 & 1) * 32 + 16 * half + c) * 16);
        struct GateIn { f32x4 r, z, n; };
        auto fetch = [&](GateIn &in, int slot) {
            const char *at = gi_tile + (size_t)slot * Sh::kSlotBytes;
            in.r = *reinterpret_cast<const f32x4 *>(at + gi_lane);
            in.z = *reinterpret_cast<const f32x4 *>(at + Sh::kGateBytes + gi_lane);
            in.n = *reinterpret_cast<const f32x4 *>(at + 2 * Sh::kGateBytes + gi_lane);
        };
        f32x4 h = {0.0f, 0.0f, 0.0f, 0.0f};
        auto publish = [&](int buf) {                  // the wave's units as its half of every lane's 16 bytes of k-step w / 2
            typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
            bf16x4 hi, lo;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                hi[r] = (__bf16)h[r];
                lo[r] = (__bf16)(h[r] - (float)hi[r]);
            }
            char *at = reinterpret_cast<char *>(&h_lds[buf][w / 2][0][lane]) + (w & 1) * 8;
            *reinterpret_cast<bf16x4 *>(at) = hi;
            *reinterpret_cast<bf16x4 *>(at + 1024) = lo;
        };
        GateIn set_a, set_b;
        fetch(set_a, 0);
        publish(0);
#pragma unroll
        for (int gate = 0; gate < 3; ++gate)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) settle(whh[gate][ks]);
        asm volatile("" ::"v"(bias_hn));
        for (int i = 0; i < LEAD; ++i) lds_barrier();
        auto step = [&](const GateIn &in, GateIn &next, int it) {
            fetch(next, min(it + 1, T));
            f32x4 acc_r = {0.0f, 0.0f, 0.0f, 0.0f}, acc_z = {0.0f, 0.0f, 0.0f, 0.0f}, acc_n = bias_hn;
            f32x4 *const acc[3] = {&acc_r, &acc_z, &acc_n};
            Frag<P> hb[KS];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                hb[ks].hi = h_lds[it & 1][ks][0][lane];
                hb[ks].lo = h_lds[it & 1][ks][1][lane];
            }
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const WFrag<P> *const wf[3] = {&whh[0][ks], &whh[1][ks], &whh[2][ks]};
                mma16_across<P, 3>(acc, wf, hb[ks]);
            }
            h = gru_blend4(acc_r + in.r, acc_z + in.z, in.n, acc_n, h);
            publish((it & 1) ^ 1);
            lds_barrier();
        };
        int it = 0;
        for (; it + 1 <= T; it += 2) {
            step(set_a, set_b, it);
            step(set_b, set_a, it + 1);
        }
        if (it <= T) step(set_a, set_b, it);
        lds_barrier();                                 // the epilogue's last slot
        return;
    }
    if (wave == Sh::kToucher) {
        // ---------------------------------------------------------------- touches: one 4-byte load per 128 bytes
        // of the tile's half record: 3 gates x 4 blocks x 4 vectors x 2 lane groups of 256 bytes each
        const char *const at0 = gi_tile + (size_t)(lane >> 2) * 1024 + (lane >> 1 & 1) * 512 + half * 256 + (lane & 1) * 128;
        uint32_t set[kTouchAhead][3] = {};
        auto touch = [&](int k, int s) {
#pragma unroll
            for (int j = 0; j < 3; ++j) asm volatile("" ::"v"(set[k][j]));
            const char *at = at0 + (size_t)min(max(s + 1 + kTouchAhead, 0), T) * Sh::kSlotBytes;
#pragma unroll
            for (int j = 0; j < 3; ++j) set[k][j] = *reinterpret_cast<const uint32_t *>(at + j * Sh::kGateBytes);
            lds_barrier();
        };
        int s = -LEAD;
        static_assert(kTouchAhead == 4, "the loop is unrolled over the register sets");
        for (; s + 3 <= T + 1; s += 4) {
            touch(0, s);
            touch(1, s + 1);
            touch(2, s + 2);
            touch(3, s + 3);
        }
        for (; s <= T + 1; ++s) lds_barrier();
        return;
    }
    // ---------------------------------------------------------------- epilogue and loader wave
    const int row = rt * 16 + c;
    const bool valid = row < rows;                     // rows past the end compute on row 0's inputs; results dropped
    const int b = valid ? row / N : 0, n = valid ? row % N : 0;
    const int bi = td.episode_index ? min(max(td.episode_index[b], 0), td.pool_episodes - 1) : b;
    TdTile16<AB, MODE> tile;
    tile.init(td, net, T, lane, b, bi, n, valid, epi_lds);
    if (wave == Sh::kEpilogue) {
        td_epilogue16<H, P, AB, QALL, MODE>(net, tile, !is_target && !kValue, kDouble ? !is_target : is_target || !two_nets,
                                            kDouble && is_target, LEAD, h_lds, b2_lds);
        return;
    }
    using SlotRaw = typename TdTile16<AB, MODE>::SlotRaw;
    SlotRaw epi_a{}, epi_b{};
    const bool want_target = kDouble ? !is_target : is_target || !two_nets;
    auto loader_loop = [&](auto wide) {
        auto loader_step = [&](const SlotRaw &ready, SlotRaw &refill, int s) {
            refill = tile.fetch(min(max(s + 1, 0), T), wide);
            tile.stage(ready, s, wide, want_target);
            lds_barrier();
        };
        int s = -LEAD;
        for (; s + 1 <= T + 1; s += 2) {
            loader_step(epi_a, epi_b, s);
            loader_step(epi_b, epi_a, s + 1);
        }
        if (s <= T + 1) loader_step(epi_a, epi_b, s);
    };
    if (A >= 4) loader_loop(std::true_type{});
    else loader_loop(std::false_type{});
}

hipError_t launch_recurrent16(const NetFrags &online, const NetFrags &target, bool two_nets, const char *gi_online, const char *gi_target,
                              int B, int T, const TdArrays &td, hipStream_t stream)
{
    if (online.H != Recur16::H || online.planes != Recur16::P) return hipErrorInvalidValue;
    if (td.mode == kTdDouble && (!two_nets || !td.next_q.q)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((B * online.N + 15) / 16), two_nets ? 2u : 1u), block(64 * Recur16::kWaves);
    const int two = two_nets ? 1 : 0;
#define MARL_REC16(ABLK, QA, MD)                                                                                               \
    hipLaunchKernelGGL((recurrent16_td_kernel<ABLK, QA, MD>), grid, block, 0, stream, online, target, gi_online, gi_target, two, B, T, td)
#define MARL_REC16_Q(ABLK)                                                                                                     \
    do {                                                                                                                       \
        if (td.mode == kTdDouble) { if (td.q_all) MARL_REC16(ABLK, true, kTdDouble); else MARL_REC16(ABLK, false, kTdDouble); } \
        else if (td.mode == kTdValue) MARL_REC16(ABLK, false, kTdValue);                                                            \
        else if (td.mode == kTdSelect) { if (td.q_all) MARL_REC16(ABLK, true, kTdSelect); else MARL_REC16(ABLK, false, kTdSelect); } \
        else if (td.mode != kTdPlain) return hipErrorInvalidValue;                                                             \
        else if (td.q_all) MARL_REC16(ABLK, true, kTdPlain);                                                                   \
        else MARL_REC16(ABLK, false, kTdPlain);                                                                                \
    } while (0)
    switch ((online.A + 15) / 16) {
    case 1: MARL_REC16_Q(1); break;
    case 2: MARL_REC16_Q(2); break;
    case 3: MARL_REC16_Q(3); break;
    case 4: MARL_REC16_Q(4); break;
    default: return hipErrorInvalidValue;
    }
#undef MARL_REC16_Q
#undef MARL_REC16
    return hipGetLastError();
}

}  // namespace marl
