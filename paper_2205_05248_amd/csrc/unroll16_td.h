// The TD step of the unroll kernels on tiles of 16 (episode, agent) rows (unroll_fused.hip, unroll_recur16.hip): its
// per-slot inputs on their way through LDS, and the epilogue wave that turns the hidden state of a slot into
// q_taken / masked maximum / TD target.
#pragma once
#include <type_traits>

#include "fused16_roles.h"

namespace marl {

// The epilogue's per-slot inputs: the taken action, the flags, the reward and the availability bytes.
// They are global loads whose latency is longer than a step, and the epilogue's own instruction stream cannot
// hide it: its stores and loads are conditional, so any wait it needs covers everything in flight.  A loader
// wave fetches them instead, a step earlier, the same number of loads every step
// (positions clamped into the arrays, rows past the end read row 0), and hands them over in LDS:
// epi[slot & 1][word][lane], words: 0 action, 1 flags (filled(t) | terminated(t-1) << 8 | filled(t-1) << 16),
// 2 reward(t-1), 3 the lane's availability slots of slot t (avail_mask16, formed by the loader).
// With two networks each workgroup's epilogue uses one half only: both are fetched (a load left out by a branch would make
// the waits for the others inexact), but the target's half is put together only where it is wanted.
// wide: at least four actions, whose availability is read four bytes at a time.
constexpr int kEpiWords = 4;
constexpr size_t kEpiBytes = 2 * kEpiWords * 64 * 4;

template <int AB, int MODE> struct TdTile16 {
    static constexpr bool kValue = MODE == kTdValue, kSave = MODE == kTdSave;
    struct SlotIn { int u; uint32_t flags; float reward; uint32_t slots; };
    struct SlotRaw { int u; uint32_t filled, terminated_prev, filled_prev; float reward; uint32_t avail_raw[AB]; };

    TdArrays td;
    uint32_t *epi;
    int N, A, T, lane, q4;
    bool valid;
    // 32-bit element offsets (the host bounds every array to 2^30 elements)
    uint32_t btn0;          // outputs [B, T, N]:       + t N
    uint32_t qa0;           // q_all [B, T+1, N, A]:    + t N A
    uint32_t act0;          // actions of the episode:  + t N
    uint32_t av0;           // avail of the episode:    + t N A
    uint32_t bt0;           // per-episode flags:       + t
    uint32_t next_row;      // the row's place in a record of the target network's Q values
    size_t next_tile;

    // b, n: the lane's row of the batch; bi: the episode of the input arrays that it reads
    __device__ __forceinline__ void init(const TdArrays &arrays, const NetFrags &net, int T_, int lane_, int b, int bi, int n, bool valid_,
                                         char *epi_lds)
    {
        td = arrays;
        epi = reinterpret_cast<uint32_t *>(epi_lds);
        N = net.N; A = net.A; T = T_; lane = lane_; q4 = lane_ >> 4; valid = valid_;
        const int S = T + 1;
        btn0 = (uint32_t)(b * T) * N + n;
        qa0 = ((uint32_t)(b * S) * N + n) * A;
        act0 = (uint32_t)(bi * T) * N + n;
        av0 = ((uint32_t)(bi * S) * N + n) * A;
        bt0 = (uint32_t)(bi * T);
        if constexpr (MODE == kTdDouble) {
            const uint32_t row = (uint32_t)b * N + n;
            next_tile = (row >> 5) * arrays.next_q.tile_stride;
            next_row = next_q_row(arrays.next_q, row);
        }
    }

    template <class Wide>
    __device__ __forceinline__ SlotRaw fetch(int t, Wide) const        // t in 0 .. T
    {
        SlotRaw in{};
        if constexpr (!kSave) {
            const uint32_t tq = (uint32_t)min(t, T - 1), tp = (uint32_t)max(t - 1, 0);
            in.u = kValue ? td.next_action[btn0 + tp * N] : td.actions[act0 + tq * N];
            in.filled = td.filled[bt0 + tq];
            in.terminated_prev = td.terminated[bt0 + tp];
            in.filled_prev = td.filled[bt0 + tp];
            in.reward = td.reward[bt0 + tp];
            if constexpr (Wide::value && !kValue) issue_avail_loads16<AB>(td.avail + (av0 + (uint32_t)t * N * A), A, q4, in.avail_raw);
        }
        return in;
    }

    template <class Wide>
    __device__ __forceinline__ void stage(const SlotRaw &in, int t, Wide, bool want_target) const
    {
        if constexpr (!kSave) {
            uint32_t *at = epi + (size_t)(t & 1) * kEpiWords * 64 + lane;
            // The flags pass through the empty asm so that they are put together here: done where they are loaded, the loader
            // waited for them there, a trip to memory in every step.
            uint32_t filled = in.filled, terminated_prev = in.terminated_prev, filled_prev = in.filled_prev;
            asm volatile("" : "+v"(filled), "+v"(terminated_prev), "+v"(filled_prev));
            at[0] = (uint32_t)in.u;
            at[64] = filled | terminated_prev << 8 | filled_prev << 16;
            if (want_target) {
                at[128] = __builtin_bit_cast(uint32_t, in.reward);
                if constexpr (Wide::value && !kValue) at[192] = avail_mask16<AB>(in.avail_raw, A, q4, valid);
            }
        }
    }

    __device__ __forceinline__ SlotIn staged(int t) const
    {
        const uint32_t *at = epi + (size_t)(t & 1) * kEpiWords * 64 + lane;
        SlotIn in;
        in.u = (int)at[0];
        in.flags = at[64];
        in.reward = __builtin_bit_cast(float, at[128]);
        in.slots = at[192];
        return in;
    }
};

// The epilogue wave: fc2 (W2 in registers) on the hidden state that the recurrence published during the step before,
// and the TD step on the result.  `lead` barriers before slot 0, then T + 2 more.  emit_online: q_taken (and q_all);
// emit_target: next_max and td_target, or (kTdSelect, kTdDouble) the index of the best action instead; store_next
// (kTdDouble): the Q values of every slot but the first.
template <int H, int P, int AB, bool QALL, int MODE>
__device__ __forceinline__ void td_epilogue16(const NetFrags &net, const TdTile16<AB, MODE> &tile, bool emit_online, bool emit_target,
                                              bool store_next, int lead, bf16x8 (*h_lds)[H / 32][P][64], float *b2_lds)
{
    constexpr int KS = H / 32;
    constexpr bool kSelect = MODE == kTdSelect || MODE == kTdDouble, kValue = MODE == kTdValue;
    const int lane = tile.lane, q4 = tile.q4, N = tile.N, A = tile.A, T = tile.T;
    const bool valid = tile.valid;
    const TdArrays &td = tile.td;
    WFrag<P> w2[AB][KS];
#pragma unroll
    for (int ab = 0; ab < AB; ++ab)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) w2[ab][ks] = load_wfrag<P>(net.w2_16 + ((size_t)(ab * KS + ks) * P) * 64 + lane);
    if (lane < 16 * AB) b2_lds[lane] = lane < A ? net.b2[lane] : 0.0f;
    // the weights have arrived before the loop starts: a wait for them inside it would also cover the loop's own loads
#pragma unroll
    for (int ab = 0; ab < AB; ++ab)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) settle(w2[ab][ks]);
    for (int i = 0; i < lead; ++i) lds_barrier();
    for (int it = 0; it <= T + 1; ++it) {
        if (it >= 1) {
            const int t = it - 1, cur = it & 1;          // h_t was published during iteration t
            const auto in = tile.staged(t);
            const bool on_filled = (in.flags & 0xFFu) != 0, terminated_prev = (in.flags >> 8 & 0xFFu) != 0, tg_filled = (in.flags >> 16 & 0xFFu) != 0;
            f32x4 qv[AB];
#pragma unroll
            for (int ab = 0; ab < AB; ++ab) qv[ab] = load_feature4(b2_lds, ab, q4);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                Frag<P> hb;
                hb.hi = h_lds[cur][ks][0][lane];
                if constexpr (P == 2) hb.lo = h_lds[cur][ks][1][lane];
                f32x4 *accs[AB];
                const WFrag<P> *wf[AB];
#pragma unroll
                for (int ab = 0; ab < AB; ++ab) {
                    accs[ab] = &qv[ab];
                    wf[ab] = &w2[ab][ks];
                }
                mma16_across<P, AB>(accs, wf, hb);
            }
            if (emit_online) {
                if constexpr (QALL) {
                    if (valid) store_q_row16<AB>(td.q_all + (tile.qa0 + (uint32_t)t * N * A), qv, A, q4);
                }
                if (t < T) {
                    const int u = min(max(in.u, 0), A - 1);
                    const float qu = pick_action_value16<AB>(qv, u, q4);
                    if (valid && q4 == 0) td.q_taken[tile.btn0 + (uint32_t)t * N] = on_filled ? qu : 0.0f;
                }
            }
            if constexpr (MODE == kTdDouble) {
                if (store_next && valid && t >= 1) {
                    float *const at = td.next_q.q + tile.next_tile + (size_t)t * td.next_q.slot_stride + tile.next_row;
#pragma unroll
                    for (int ab = 0; ab < AB; ++ab)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int action = 16 * ab + 4 * q4 + r;
                            if (action < A) at[(uint32_t)action * td.next_q.action_stride] = qv[ab][r];
                        }
                }
            }
            if (emit_target && t >= 1) {
                const uint32_t o = tile.btn0 + (uint32_t)(t - 1) * N;
                float best_q;
                if constexpr (kValue) {               // the value of the action the other network chose
                    const float picked = pick_action_value16<AB>(qv, min(max(in.u, 0), A - 1), q4);
                    best_q = in.u >= 0 ? picked : 0.0f;      // -1: the other network found no action available
                } else {
                    const uint32_t slots =
                        A >= 4 ? in.slots
                               : avail_mask_small16(td.avail + (valid ? tile.av0 + (uint32_t)t * N * A : 0u), A, q4, valid);
                    if constexpr (kSelect) {
                        int best;
                        masked_argmax16<AB, true>(qv, slots, q4, best_q, best);
                        if (valid && q4 == 0) td.next_action[o] = best;
                    } else {
                        best_q = masked_max16<AB>(qv, slots);
                    }
                }
                if (!kSelect && valid && q4 == 0) {
                    const float keep = terminated_prev ? 0.0f : 1.0f;
                    const float y = in.reward + td.gamma * keep * best_q;
                    td.next_max[o] = tg_filled ? best_q : 0.0f;
                    td.td_target[o] = tg_filled ? y : 0.0f;
                }
            }
        }
        lds_barrier();
    }
}

}  // namespace marl
