// Fused unroll + TD kernel for gfx950: one workgroup walks the T+1 slots of one tile of 16
// (episode, agent) rows for one network.  Every weight matrix stays on chip for the whole
// episode and no intermediate is written to global memory; per slot a workgroup reads its 16
// observation rows and the TD inputs, and writes the TD outputs.
//
// Where the weights live (H = 128, bf16: 278 KB in total):
//   W_hh   registers of the compute waves (each owns H/64 feature blocks of 16 hidden units, all three gates)
//   W_ih   LDS, copied once at kernel start; each compute wave reads the fragments of its own
//          blocks from there every slot (A operands come from LDS at 16 bytes per lane)
//   W1     registers of the fc1 waves (each owns H/16/NF feature blocks x ceil(D/32) k-steps)
//   W2     registers of the epilogue wave
//
// The work of a slot is cut into pipeline stages that run concurrently on different wavefronts,
// each on a different slot, and meet at ONE LDS-only barrier per slot.  In the step in which the
// recurrence handles slot s:
//
//   loader wave    writes the observations of slot s+2 (loaded during the previous step) to LDS
//                  as bf16 operand fragments and issues the loads of slot s+3;
//   fc1 waves      x = ReLU(W1 o + b1[agent]) for slot s+1, observation fragments from LDS, x to
//                  LDS as the next operand; the first one also touches the observations of a
//                  later slot so that the loader's loads hit L2;
//   compute waves  slot s of the GRU: W_ih x + W_hh h + b for their hidden units, gates, new hidden
//                  state to LDS as operand;
//   epilogue wave  fc2 / TD step of slot s-1.
//
// Only the GRU is a dependent chain; the other stages are throughput work that hides under it.
// Tiles of 16 rows (16x16x32 MFMAs) rather than 32 give twice as many workgroups, so that
// episode batches of a few thousand rows still occupy every compute unit, and halve the length
// of the chain per slot.
//
// Every LDS buffer is double-buffered on the parity of the slot it holds; a buffer written in
// step s was last read in step s-1 and is first read in step s+1.
//
// What bounds a step is instruction issue on the SIMDs that the roles share (64 units, two planes, 80 observations: by
// cycle counters every wave works 1700 to 2050 of a step's 2080 clocks, the loader all of them).  The loader waited out a
// trip to memory in each step until its loads were straight-line code and the flags it fetches were put together where
// they are staged; with that and W_ih in registers for 64 units, 32 episodes x 120 slots x 8 agents 103.3 -> 96.7 us,
// 64 x 200 x 32 with 128 units 279 -> 275 us, keeping activations 370 -> 335 us.  (With the target half of the TD inputs put
// together only where it is read, and the first layer's weights prepared per k-step: 92 and 256 to 268 us, box to box.)
#include <hip/hip_runtime.h>

#pragma once
#include "unroll16_td.h"

namespace marl {


// LDS of a launch: the shared layout, then the staging area of the epilogue's inputs.
template <int H, int P> using UnrollShape = Fused16<H, P, H == 64>;
template <int H, int P> using UnrollGru = GruWave<H, P, H == 64>;
template <int H, int P> constexpr size_t unroll_lds_bytes(int ks1) { return UnrollShape<H, P>::lds_bytes(ks1) + kEpiBytes; }

template <int H, int P, int AB, bool QALL, int MODE>
__global__ __launch_bounds__(fused_threads(H), 2) void unroll_fused_kernel(
    NetFrags online, NetFrags target, int two_nets, int B, int T, const int32_t *__restrict__ episode_index,
    int pool_episodes, const float *__restrict__ obs,
    const uint8_t *__restrict__ avail, const int32_t *__restrict__ actions, const float *__restrict__ reward,
    const uint8_t *__restrict__ terminated, const uint8_t *__restrict__ filled, float gamma,
    float *__restrict__ q_taken, float *__restrict__ next_max, float *__restrict__ td_target, float *__restrict__ q_all,
    int32_t *__restrict__ next_action, float *__restrict__ h_save, void *__restrict__ x_save, NextQ next_q)
{
    using Sh = UnrollShape<H, P>;
    constexpr int KS = Sh::KS, LEAD = kFusedLead;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    typedef bf16x8 (*FragBuf)[KS][P][64];
    const FragBuf h_lds = reinterpret_cast<FragBuf>(lds + Sh::oH);
    const FragBuf x_lds = reinterpret_cast<FragBuf>(lds + Sh::oX);
    bf16x8 *const obuf = reinterpret_cast<bf16x8 *>(lds + Sh::oObs);        // [((slot & 1) ks1 + ks) P + p][64]
    bf16x8 *const wih_lds = reinterpret_cast<bf16x8 *>(lds + Sh::oWih);     // [((blk KS + ks) P + p)][64]

    // Workgroup -> (tile, network).  With two networks the online and the target workgroup of a tile
    // sit eight apart in a block of sixteen consecutive workgroups: consecutive workgroups go round
    // the eight XCDs, so the pair shares one XCD's L2 (the second read of an observation line hits
    // there) and is dispatched at about the same time.
    const int rt = two_nets ? (int)(blockIdx.x >> 4) * 8 + (int)(blockIdx.x & 7) : (int)blockIdx.x;
    const bool is_target = two_nets && ((blockIdx.x >> 3) & 1);
    const int rows = B * online.N;
    if (rt * 16 >= rows) return;                          // padding of the last block of sixteen
    const NetFrags net = is_target ? target : online;     // by value: uniform, lives in scalar registers
    const int lane = threadIdx.x & 63, q4 = lane >> 4, c = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int N = net.N, D = net.D, A = net.A, S = T + 1;
    const int ks1 = obs_k_steps(P, D);
    const int row = rt * 16 + c;
    const bool valid = row < rows;                     // rows past the end compute on row 0's inputs; results dropped
    const int b = valid ? row / N : 0, n = valid ? row % N : 0;         // position in the batch: outputs
    // episode of the input arrays: the batch position itself, or the listed episode of a larger pool
    const int bi = episode_index ? min(max(episode_index[b], 0), pool_episodes - 1) : b;

    constexpr bool kValue = MODE == kTdValue, kSave = MODE == kTdSave, kDouble = MODE == kTdDouble;
    TdTile16<AB, MODE> tile;
    tile.init(TdArrays{episode_index, pool_episodes, avail, actions, reward, terminated, filled, gamma, q_taken, next_max, td_target,
                       q_all, MODE, next_action, next_q},
              net, T, lane, b, bi, n, valid, lds + Sh::lds_bytes(ks1));

    // W_ih -> LDS, all waves (or not at all: it may be in registers).  Its first readers start after kFusedLead barriers.
    for (int i = threadIdx.x; i < Sh::kWihVecs; i += fused_threads(H)) wih_lds[i] = net.wih_16[i];
    // Steps run s = -LEAD .. T+1, one barrier at the end of each: LEAD + T + 2 barriers per wave.

    if (wave < Sh::NC) {
        // ---------------------------------------------------------------- compute wave
        const int w = wave;
        UnrollGru<H, P> gru;
        gru.load(net, w, lane, q4);
        if (w == 0 && !Sh::kWihInRegs) UnrollGru<H, P>::stage_gate_biases(lds, net, lane);
        f32x4 hv[Sh::NBC];                           // this wave's units of the hidden state, fp32
#pragma unroll
        for (int j = 0; j < Sh::NBC; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) hv[j][r] = 0.0f;
        UnrollGru<H, P>::publish(h_lds[0], w, lane, hv);
        // kTdSave / kTdKeep: this lane's units of its row's state, slot by slot (the online network's)
        constexpr bool kStores = MODE == kTdSave || MODE == kTdKeep;
        const bool stores = kStores && !is_target;
        float *h_row = nullptr;
        if constexpr (kStores) {
            h_row = h_save + ((size_t)b * S * N + n) * H + 16 * Sh::NBC * w + 4 * q4;
            if (valid && stores)
#pragma unroll
                for (int j = 0; j < Sh::NBC; ++j) *reinterpret_cast<f32x4 *>(h_row + 16 * j) = hv[j];
        }
        gru.settle_weights();
        for (int i = 0; i < LEAD; ++i) lds_barrier();
        for (int it = 0; it <= T + 1; ++it) {
            if (it <= T) {
                const int cur = it & 1;
                gru.step(lds, w, lane, q4, h_lds[cur], x_lds[cur], hv);
                UnrollGru<H, P>::publish(h_lds[cur ^ 1], w, lane, hv);
                if constexpr (kStores) {
                    if (valid && stores && it < T)
#pragma unroll
                        for (int j = 0; j < Sh::NBC; ++j)
                            *reinterpret_cast<f32x4 *>(h_row + (size_t)(it + 1) * N * H + 16 * j) = hv[j];
                }
            }
            lds_barrier();
        }
    } else if (wave == Sh::kEpilogue) {
        // ---------------------------------------------------------------- epilogue wave
        td_epilogue16<H, P, AB, QALL, MODE>(net, tile, !is_target && !kValue && !kSave, (kDouble ? !is_target : is_target || !two_nets) && !kSave,
                                            kDouble && is_target, LEAD, h_lds,
                                            reinterpret_cast<float *>(lds + Sh::oB2));
    } else if (wave == Sh::kLoader) {
        // ---------------------------------------------------------------- loader wave
        // Straight-line steps with the same memory operations in each, so that a wait counts exactly: every step it loads
        // a slot (the ends a slot again) and puts down one (what lies outside 0 .. T nobody reads).
        const float *base = obs + ((size_t)bi * S * N + n) * D;              // the lane's row at slot 0
        const size_t slot_stride = (size_t)N * D;
        using SlotRaw = typename TdTile16<AB, MODE>::SlotRaw;
        const bool want_target = kDouble ? !is_target : is_target || !two_nets;
        auto loader_loop = [&](auto k_steps, auto is_short, auto wide) {
            constexpr int KN = decltype(k_steps)::value;
            ObsStageK<P, KN, decltype(is_short)::value> st;
            st.init(D, q4);
            // Two register sets in turn: a step first issues the loads of the slot it will write in the next step, into
            // the set that step will read, then converts the set loaded a step ago.  The loads have a whole step to arrive.
            ObsRegsK<KN> set_a{}, set_b{};
            SlotRaw epi_a{}, epi_b{};                // the epilogue's inputs of a slot, in turn like the observation sets
            auto loader_step = [&](const ObsRegsK<KN> &ready, ObsRegsK<KN> &refill, const SlotRaw &epi_ready, SlotRaw &epi_refill, int s) {
                const int ws = s + 2, ls = ws + 1;
                st.load(refill, base + (size_t)min(max(ls, 0), T) * slot_stride);
                epi_refill = tile.fetch(min(max(s + 1, 0), T), wide);        // slot s + 1: staged in the next step, read by the epilogue in step s + 2
                __builtin_amdgcn_sched_barrier(0);
                st.write(ready, obuf + (size_t)((ws & 1) * KN) * P * 64 + lane);     // registers -> LDS
                tile.stage(epi_ready, s, wide, want_target);
                lds_barrier();
            };
            int s = -LEAD;
            for (; s + 1 <= T + 1; s += 2) {
                loader_step(set_a, set_b, epi_a, epi_b, s);
                loader_step(set_b, set_a, epi_b, epi_a, s + 1);
            }
            if (s <= T + 1) loader_step(set_a, set_b, epi_a, epi_b, s);
        };
        using Yes = std::true_type;
        using No = std::false_type;
        auto with_width = [&](auto k_steps, auto is_short) {
            if (A >= 4) loader_loop(k_steps, is_short, Yes{});
            else loader_loop(k_steps, is_short, No{});
        };
        if (D < 8) with_width(std::integral_constant<int, 1>{}, Yes{});
        else with_k_steps<P>(ks1, [&](auto k_steps) { with_width(k_steps, No{}); });
    } else {
        // ---------------------------------------------------------------- fc1 wave
        const int f = wave - Sh::kFc1;
        Fc1Wave<H, P> fc1;
        f32x4 b1v[Sh::NBF];
        Fc1Wave<H, P>::load_bias(net, f, n, q4, b1v);
#pragma unroll
        for (int j = 0; j < Sh::NBF; ++j) asm volatile("" ::"v"(b1v[j]));
        const float *touch_row = obs + ((size_t)bi * S * N + n) * D;
        ObsTouch<H, P, 2> tch;
        tch.init(D, q4);
        // 128 units: four bytes of availability, the last of the array at most (fewer in all: any others).  Of a single byte the
        // compiler clears the other bits of its register, in one place per four touches, and waits there for the touch before: a
        // trip to memory, in some instances before the barrier.  (24 episodes x 200 slots x 5 agents keeping activations, 60 / 190 / 225
        // observations 229 / 239 / 233 -> 212 / 221 / 231 us; 64 units: no faster, 32 x 120 x 8 in fp32 91.6 -> 92.9.)
        const uint32_t avail_size = (uint32_t)(episode_index ? pool_episodes : B) * (uint32_t)S * (uint32_t)(N * A);
        const uint8_t *const avail_bytes = avail_size < 4 ? reinterpret_cast<const uint8_t *>(obs) : avail;
        const uint32_t avail_last = max(avail_size, 4u) - 4u;
        const uint32_t avail_row = ((uint32_t)(bi * S) * N + n) * A;
        auto touch = [&](int c, int s) {             // the slot the loader will load kTouchAhead steps from now
            const int slot = min(max(s + 3 + kTouchAhead, 0), T);                            // ends: touched twice
            tch.consume(c);
            tch.touch(c, touch_row + (size_t)slot * N * D);
            // and what the epilogues will read for that slot: the row's availability and action
            if constexpr (MODE != kTdSave) {
                if constexpr (H == 128)
                    __builtin_memcpy(&tch.set[c][tch.TLO], avail_bytes + min(avail_row + (uint32_t)slot * (uint32_t)(N * A), avail_last), 4);
                else
                    tch.set[c][tch.TLO] = avail[(((size_t)bi * S + slot) * N + n) * A];
                tch.set[c][tch.TLO + 1] = (uint32_t)actions[((size_t)bi * T + min(slot, T - 1)) * N + n];
            }
        };
        // kTdSave / kTdKeep: the lane's x of its row, slot by slot (the online network's).  The host bounds 4 H samples to 2^30.
        constexpr bool kStores = MODE == kTdSave || MODE == kTdKeep;
        constexpr uint32_t kElem = P == 1 ? 2u : 4u;
        const __amdgpu_buffer_rsrc_t x_buf =
            __builtin_amdgcn_make_buffer_rsrc(x_save, 0, kStores ? (int)((uint32_t)rows * S * H * kElem) : 0, kRawBuffer);
        // (rows that are not kept: beyond the buffer, in any slot)
        const uint32_t x_row = valid && !is_target ? (((uint32_t)b * S * N + n) * H + 4 * q4) * kElem : 0x80000000u, x_slot = (uint32_t)N * H * kElem;
        auto fc1_loop = [&](auto k_steps) {
            constexpr int KN = decltype(k_steps)::value;
            fc1.template load_k<KN>(net, f, lane);
            auto fc1_step = [&](int s) {
                const int slot = s + 1;
                if (slot >= 0 && slot <= T) {
                    const bf16x8 *const o = obuf + (size_t)((slot & 1) * KN) * P * 64;
                    if constexpr (kStores) fc1.template step_k<KN, true>(o, f, lane, b1v, x_lds[slot & 1], &x_buf, x_row + (uint32_t)slot * x_slot);
                    else fc1.template step_k<KN>(o, f, lane, b1v, x_lds[slot & 1]);
                }
                lds_barrier();
            };
            int s = -LEAD;
            // With two networks only the online workgroup touches: its partner on the tile reads the
            // same lines a few steps later and finds them in L2.  A partner that runs ahead misses,
            // waits for HBM and falls back behind, so the pair settles into that order by itself.
            if (f == 0 && !is_target) {
                static_assert(kTouchAhead == 4, "the loop is unrolled over the register sets");
                for (; s + 3 <= T + 1; s += 4) {
                    touch(0, s);     fc1_step(s);
                    touch(1, s + 1); fc1_step(s + 1);
                    touch(2, s + 2); fc1_step(s + 2);
                    touch(3, s + 3); fc1_step(s + 3);
                }
            }
            for (; s <= T + 1; ++s) fc1_step(s);
        };
        with_k_steps<P>(ks1, fc1_loop);
    }
}

// ------------------------------------------------------------------------------------------ launch
// Arguments of launch_unroll_fused.
struct FusedCall {
    const NetFrags &online, &target;
    bool two_nets;
    int B, T;
    const int32_t *episode_index;
    int pool_episodes;
    const float *obs;
    const uint8_t *avail;
    const int32_t *actions;
    const float *reward;
    const uint8_t *terminated, *filled;
    float gamma;
    float *q_taken, *next_max, *td_target, *q_all;
    hipStream_t stream;
    TdMode mode;
    int32_t *next_action;
    float *h_save;
    void *x_save;
    const NextQ &next_q;
};

hipError_t launch_unroll_fused_h128(const FusedCall &call);
hipError_t launch_unroll_fused_h64_bf16(const FusedCall &call);
hipError_t launch_unroll_fused_h64_f32(const FusedCall &call);

template <int H, int P>
hipError_t fused_dispatch(const FusedCall &call)
{
    const auto &[online, target, two_nets, B, T, episode_index, pool_episodes, obs, avail, actions, reward, terminated, filled, gamma, q_taken,
                 next_max, td_target, q_all, stream, mode, next_action, h_save, x_save, next_q] = call;
    const int tiles = (B * online.N + 15) / 16;
    const dim3 grid(two_nets ? (unsigned)((tiles + 7) / 8) * 16u : (unsigned)tiles), block(fused_threads(H));
    const size_t lds = unroll_lds_bytes<H, P>(obs_k_steps(P, online.D));
    const int two = two_nets ? 1 : 0;
    const int ab = (online.A + 15) / 16;
#define MARL_FUSED(ABLK, QA, MD)                                                                                    \
    do {                                                                                                            \
        auto kernel = unroll_fused_kernel<H, P, ABLK, QA, MD>;                                                      \
        hipError_t err = allow_large_lds<unroll_fused_kernel<H, P, ABLK, QA, MD>>(kLdsLimit);                       \
        if (err != hipSuccess) return err;                                                                          \
        launch_kernel(kernel, grid, block, lds, stream, online, target, two, B, T, episode_index, pool_episodes,      \
                           obs, avail, actions,                                                                      \
                           reward, terminated, filled, gamma, q_taken, next_max, td_target, q_all, next_action,     \
                           h_save, x_save, next_q);                                                                 \
    } while (0)
#define MARL_FUSED_Q(ABLK)                                                                                          \
    do {                                                                                                            \
        if (mode == kTdSave) MARL_FUSED(ABLK, false, kTdSave);                                                      \
        else if (mode == kTdKeep) { if (q_all) MARL_FUSED(ABLK, true, kTdKeep); else MARL_FUSED(ABLK, false, kTdKeep); } \
        else if (mode == kTdDouble) { if (q_all) MARL_FUSED(ABLK, true, kTdDouble); else MARL_FUSED(ABLK, false, kTdDouble); } \
        else if (mode == kTdValue) MARL_FUSED(ABLK, false, kTdValue);                                               \
        else if (mode == kTdSelect) { if (q_all) MARL_FUSED(ABLK, true, kTdSelect); else MARL_FUSED(ABLK, false, kTdSelect); } \
        else if (q_all) MARL_FUSED(ABLK, true, kTdPlain);                                                           \
        else MARL_FUSED(ABLK, false, kTdPlain);                                                                     \
    } while (0)
    switch (ab) {
    case 1: MARL_FUSED_Q(1); break;
    case 2: MARL_FUSED_Q(2); break;
    case 3: MARL_FUSED_Q(3); break;
    case 4: MARL_FUSED_Q(4); break;
    default: return hipErrorInvalidValue;
    }
#undef MARL_FUSED_Q
#undef MARL_FUSED
    return hipGetLastError();
}


}  // namespace marl
