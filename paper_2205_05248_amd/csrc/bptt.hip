// Backward half of the learner step for the recurrent Q-network: the gradient of
// sum(g * q_taken) with respect to every parameter, g = dL/dq_taken handed in by the caller.
//
//   unroll_fused_kernel<.., kTdSave>   (unroll_fused.hip) forward pass of the online network that keeps x and
//                                      h of every slot in global memory, [B, T+1, N, H]: h in fp32, x in fp32
//                                      or, for a bf16 network, in bf16 (what every reader rounds it to)
//   bptt_back_roles_kernel             one workgroup per 16 (episode, agent) rows walks the slots backwards.
//                                      Per slot it recomputes the gates from x_t and h_{t-1} (two MFMA
//                                      products, as the forward pass), forms the adjoints of the four gate
//                                      pre-activations, and carries dL/dh back through W_hh^T.  The adjoints
//                                      go to global memory.  The recurrence's chain and everything that hangs
//                                      on nothing behind it are on different waves.  128 hidden units, bf16.
//   bptt_back_split_kernel             the same for 64 hidden units, fp32 and bf16; here W_ih^T and, through the
//                                      ReLU, the adjoint of fc1's pre-activation are part of it
//   bptt_back_split8_kernel            the same on tiles of eight rows, for batches that leave compute units free; what goes to
//                                      memory and comes from it is moved by waves of their own
//   tn_gemm_kernel                     the weight gradients are sums over all (row, slot) samples of outer
//                                      products adjoint x activation: C[p][q] = sum_m A[m][p] B[m][q], four
//                                      times (W_ih, W_hh, W1, W2).  The samples are split into chunks, one
//                                      workgroup each, which computes the whole (small) result for its chunk:
//                                      it stages 32 samples at a time through LDS (the contraction index has
//                                      to become the fragments' k), every element read from memory once, and
//                                      writes its partial sum; extra columns of B made up on the fly (a column
//                                      of ones, or the one-hot agent id) yield the bias gradients in the same
//                                      product.
//   tn_gemm_wide_kernel                the same products for a bf16 network: both operands are fetched 16 bytes
//                                      at a time and staged as they lie in memory; the transposing LDS read
//                                      turns the staged rows into fragments.
//   gru_products_kernel                the products of W_ih and W_hh of 128 units, bf16, and, from the same read
//                                      of the adjoints, the adjoint of fc1's pre-activation.
//   tn_reduce_kernel                   adds the chunks' partial sums in a fixed order and writes the result
//                                      into the packed gradient vector.
// A batch with fewer row tiles than compute units leaves most of the chip idle while the reverse recurrence walks the
// slots.  For a bf16 network the slots are therefore walked in two launches (dL/dh handed over in memory), and the
// products over the later half run on a second stream of the handle's beside the earlier half's recurrence
// (launch_qnet_grad); the sum over all chunks, later half first, follows on the caller's stream.
// The precision follows the network's, in every product of the pass: fp32 networks split every operand into two
// bf16 planes (three MFMAs per product), bf16 networks round the operands (adjoints, activations) to bf16.
#include <type_traits>
#include <hip/hip_runtime.h>

#include <algorithm>

#include "fused16_roles.h"
#include "grad_chunks.h"
#include "store_offsets.h"

namespace marl {

struct BpttArgs {
    NetFrags net;
    int B, T, a16;
    const int32_t *actions;      // [B, T, N]
    const uint8_t *filled;       // [B, T]
    const float *grad_q;         // [B, T, N]   dL/dq_taken
    const float *h_all;          // [B, T+1, N, H]   h_all[b, s] = state before slot s
    const void *x_all;           // [B, T+1, N, H]   x of slot s; fp32, or bf16 for a one-plane network
    // The adjoints, fp32 for fp32 networks and bf16 for bf16 networks (whose products round them to bf16 anyway:
    // stored rounded, they cost half the traffic to write here and to read in the weight-gradient products)
    void *da;                    // [B, T, N, 4H]   adjoints of the gate pre-activations: n (input side), r, z, n (hidden side);
                                 //                 128 units: a gate's units in the order of an operand's k-steps
    void *dpre1;                 // [B, T, N, H]    adjoint of fc1's pre-activation
    void *dq;                    // [B, T, N, a16]  adjoint of Q, dense (one non-zero per row)
    // The launch walks slots t_end - 1 .. t_begin.  One launch takes all of them (0, T); two take the later and
    // then the earlier slots and hand dL/dh over in `carry` [rows rounded up to 16][H] fp32, so that the later
    // slots' weight-gradient products can run beside the second launch.
    int t_begin, t_end;
    float *carry;
};

// The wave's block of 16 units as half a fragment in LDS: two adjacent blocks make one k-step, and a wave writes its
// half of every lane's 16 bytes.
template <int P>
__device__ __forceinline__ void publish_block(bf16x8 (*dst)[P][64], int w, int lane, const f32x4 &v)
{
    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
    bf16x4 hi, lo;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        hi[r] = (__bf16)v[r];
        lo[r] = (__bf16)(v[r] - (float)hi[r]);
    }
    char *at = reinterpret_cast<char *>(&dst[w / 2][0][lane]) + (w & 1) * 8;
    *reinterpret_cast<bf16x4 *>(at) = hi;
    if constexpr (P == 2) *reinterpret_cast<bf16x4 *>(at + 1024) = lo;
}

// Four adjoints of one lane -> element offset `at` of the array behind `buf`, fp32 or, for a one-plane network, bf16.
template <int P>
__device__ __forceinline__ void store_adjoints(const f32x4 &v, const __amdgpu_buffer_rsrc_t &buf, uint32_t at, uint32_t drop_mask)
{
    if constexpr (P == 1) {
        typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
        typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
        bf16x4 r;
#pragma unroll
        for (int i = 0; i < 4; ++i) r[i] = (__bf16)v[i];
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, r), buf, (at * 2u) | drop_mask, 0, 0);
    } else {
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), buf, (at * 4u) | drop_mask, 0, 0);
    }
}

// 128 hidden units, one plane (two planes do not fit on chip), cut into two roles.  Only dL/dh_t -> adjoints -> dL/dh_{t-1}
// is a chain; the gates of a slot hang on nothing behind them.  Twelve waves, three per SIMD, 168 registers each: in the step
// of slot t
//
//   gate waves 0..7    (16 units each, W_hh and W_ih in registers) the gates of slot t-1 -> five factors per unit, in LDS; moving two
//                      rows each, what the chain left in LDS in the step before to memory, x and h of slot t-2 to LDS as operand, the
//                      loads of slot t-3
//   chain waves 8..11  (32 units each, W_hh^T in registers) dL/dh_t = carry + W_hh^T adjoints(t+1), then slot t's adjoints from
//                      its factors, to LDS as operand; to memory what LDS has no room for, n's and the adjoint of Q
//
// and ONE barrier per slot.  Every LDS buffer is double-buffered on the parity of its slot: written in one step, read in the
// next, written again only in the one after.  The adjoint of fc1's pre-activation, which nothing in the chain hangs on either,
// is formed from the stored adjoints where the W_ih product reads them (gru_products_kernel): its weights have no room here.
//
// What bounds it: instruction issue on the SIMDs, some 290 vector and 72 matrix instructions each per slot, which overlap only
// where waves are in different parts of their step: gate waves 4..7 move first and multiply then, the others the other way round.
// A hundred slots of 64 episodes x 32 agents, kernel trace: one role of eight waves with two barriers a slot, which formed that
// adjoint too, 249 us; two roles, stores of 8 bytes a lane, and the rows' scalars read by every gate wave 192; adjoints stored as
// operands lie, 16 bytes a lane, and the scalars read by the chain 160; the gate waves' accesses row by row 154; their two
// orders 145.  The gates' products a slot ahead of their factors in all gate waves: 206 instead of 192, more registers than there
// are.  Both roles' registers are full: what is asked for is asked for little by little (sched_barrier), or the weights spill.
struct BpttRoles {
    static constexpr int H = 128, KS = H / 32, FBK = H / 16, kFrag = 1024, kGate = FBK, kChain = KS, kThreads = 64 * (kGate + kChain);
    static constexpr int kFactors = 5;
    static constexpr int oH = 0, oX = oH + 2 * KS * kFrag, oDa = oX + 2 * KS * kFrag, kDaBytes = 3 * KS * kFrag;      // r, z, n hidden side
    static constexpr int oFac = oDa + 2 * kDaBytes, kFacBytes = kFactors * FBK * 1024;
    static constexpr int oBias = oFac + 2 * kFacBytes;             // biases r, z, n input side, n hidden side
    static constexpr int oHf = oBias + 4 * H * 4, kHfPitch = H * 4 + 16, kHfBytes = 16 * kHfPitch;      // h in fp32, row by row, for the blend
    // W2, whose row of the chosen action the chain adds: bf16 (what the table holds exactly)
    static constexpr int oW2 = oHf + 2 * kHfBytes, kW2Pitch = 2 * H + 16;
    static constexpr int lds_bytes(int A) { return oW2 + A * kW2Pitch; }
};

__global__ __launch_bounds__(BpttRoles::kThreads, BpttRoles::kThreads / 256) void bptt_back_roles_kernel(BpttArgs a)
{
    using Bs = BpttRoles;
    constexpr int H = Bs::H, KS = Bs::KS, FBK = Bs::FBK, kFrag = Bs::kFrag;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    float *const bias_lds = reinterpret_cast<float *>(lds + Bs::oBias);

    const NetFrags &net = a.net;
    const int lane = threadIdx.x & 63, q4 = lane >> 4, c = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int N = net.N, A = net.A, T = a.T, S = T + 1;
    const int rows = a.B * N;
    const int row = blockIdx.x * 16 + c;
    const bool valid = row < rows;
    const int b = valid ? row / N : 0, n = valid ? row % N : 0;

    const size_t samples = (size_t)rows * T;
    // Where an operand keeps column `col` of lane quarter `quarter` in k-step ks: the columns change places from quarter to quarter
    // and k-step to k-step, or those who have a row's units side by side would all meet in one bank.
    auto column_at = [](int ks, int quarter, int col) { return quarter * 256 + (((col ^ quarter) * 16) ^ ((ks & 3) * 64)); };
    const int lane_at = column_at(0, q4, c);
    auto operand = [&](int at, int ks) {                           // at: byte offset of the first fragment
        Frag<1> f;
        f.hi = *reinterpret_cast<const bf16x8 *>(lds + at + ks * kFrag + (lane_at ^ ((ks & 3) * 64)));
        return f;
    };
    auto da_at = [](int t) { return Bs::oDa + (t & 1) * Bs::kDaBytes; };
    auto fac_of = [&](int t, int f, int blk) { return reinterpret_cast<f32x4 *>(lds + Bs::oFac + (t & 1) * Bs::kFacBytes + (f * FBK + blk) * 1024) + lane; };
    const uint32_t bt0 = (uint32_t)b * T, btn0 = bt0 * N + n;      // the host bounds 4 H samples to 2^30
    // A store's offset: the lane's own part (kPast, where the store is to be dropped), and the slot's, the same in every lane.

    for (int i = threadIdx.x; i < 4 * H; i += Bs::kThreads) {
        const int gate = i / H, j = i % H;
        const float *src = gate == 0 ? net.bias_r : gate == 1 ? net.bias_z : gate == 2 ? net.bias_in : net.bias_hn;
        bias_lds[i] = src[j];
    }
    for (int i = threadIdx.x; i < A * H; i += Bs::kThreads)
        *reinterpret_cast<__bf16 *>(lds + Bs::oW2 + (i / H) * Bs::kW2Pitch + 2 * (i % H)) = (__bf16)net.w2_plain[i];
    // no adjoints behind the last slot: the first step's products add nothing
    for (int i = threadIdx.x; i < Bs::kDaBytes / 16; i += Bs::kThreads) reinterpret_cast<uint4 *>(lds + da_at(a.t_end))[i] = make_uint4(0, 0, 0, 0);

    if (wave >= Bs::kGate) {
        // ---------------------------------------------------------------- chain wave
        const int w = wave - Bs::kGate;                            // blocks 2 w and 2 w + 1 of sixteen units: one k-step of an operand
        const int unit0 = 32 * w + 4 * q4;                         // the lane's units: these four and those sixteen further on
        const __amdgpu_buffer_rsrc_t da_buf = __builtin_amdgcn_make_buffer_rsrc(a.da, 0, (int)(uint32_t)(samples * 4 * H * 2), kRawBuffer);
        WFrag<1> whhT[2][3 * KS];
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int ks = 0; ks < 3 * KS; ++ks) whhT[j][ks] = load_wfrag<1>(net.whhT_16 + (size_t)((2 * w + j) * 3 * KS + ks) * 64 + lane);
        const uint32_t carry_at = (uint32_t)row * H + unit0;       // rows past the end have room too
        f32x4 carry[2] = {};
        if (a.t_end < T)
#pragma unroll
            for (int j = 0; j < 2; ++j) carry[j] = *reinterpret_cast<const f32x4 *>(a.carry + carry_at + 16 * j);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
#pragma unroll
            for (int ks = 0; ks < 3 * KS; ++ks) settle(whhT[j][ks]);
            asm volatile("" : "+v"(carry[j]));
        }
        // The adjoints lie in memory as in LDS, in the order of an operand's k-steps: the lane's eight units side by side.
        const uint32_t da_lane = valid ? btn0 * 4 * H * 2 + 64 * w + 16 * q4 : kPast, da_slot = (uint32_t)N * 4 * H * 2;
        // wave w writes block w of the row's dQ
        const __amdgpu_buffer_rsrc_t dq_buf = __builtin_amdgcn_make_buffer_rsrc(a.dq, 0, (int)(uint32_t)(samples * a.a16 * 2), kRawBuffer);
        const int action0 = 16 * w + 4 * q4;
        const uint32_t dq_lane = valid && 16 * w < a.a16 ? (btn0 * a.a16 + action0) * 2 : kPast, dq_slot = (uint32_t)N * a.a16 * 2;
        // What a slot's rows add from outside, asked for two steps ahead into two sets in turn.
        struct In { float gq_raw; uint8_t fil; int u; };
        auto fetch = [&](In &in, int t) {
            const uint32_t ts = (uint32_t)max(t, 0), sample = btn0 + ts * N;
            in.fil = a.filled[bt0 + ts];
            in.gq_raw = *reinterpret_cast<const float *>(reinterpret_cast<const char *>(a.grad_q) + sample * 4u);
            in.u = *reinterpret_cast<const int *>(reinterpret_cast<const char *>(a.actions) + sample * 4u);
        };
        auto arrived = [](In &in) {
            asm volatile("" ::"v"((uint32_t)in.fil));
            asm volatile("" : "+v"(in.gq_raw), "+v"(in.u));
        };
        // carry += W_hh^T adjoints(t).  Two k-steps are asked for while the two before are multiplied; left to itself the compiler
        // waits out every pair of reads.
        auto back_product = [&](int t) {
            Frag<1> d[2][2];
            auto request = [&](int pair) {
#pragma unroll
                for (int i = 0; i < 2; ++i) d[pair % 2][i] = operand(da_at(t), 2 * pair + i);
            };
            constexpr int kPairs = 3 * KS / 2;
            request(0);
#pragma unroll
            for (int pair = 0; pair < kPairs; ++pair) {
                if (pair + 1 < kPairs) request(pair + 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) mma16<1>(carry[j], whhT[j][2 * pair + i], d[pair % 2][i]);
            }
        };
        auto step = [&](In &in, int t, bool ask) {                 // (ask: known where it is called)
            // (What passes through the empty asm is used here and not earlier: the compiler would widen `filled` where it is
            // loaded, and wait there.)
            uint32_t fil = in.fil;
            int u = in.u;
            float gq = in.gq_raw;
            asm volatile("" : "+v"(fil), "+v"(u), "+v"(gq));
            gq = (valid && fil) ? gq : 0.0f;
            u = min(max(u, 0), A - 1);
            back_product(t + 1);
            f32x4 dan[2], dar[2], daz[2], dahn[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                f32x4 fac[Bs::kFactors];
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int f = 0; f < Bs::kFactors; ++f) fac[f] = *fac_of(t, f, 2 * w + j);
                const uint2 w2 = *reinterpret_cast<const uint2 *>(lds + Bs::oW2 + u * Bs::kW2Pitch + 2 * (unit0 + 16 * j));
                const f32x4 w2v = {__uint_as_float(w2.x << 16), __uint_as_float(w2.x & 0xFFFF0000u),
                                   __uint_as_float(w2.y << 16), __uint_as_float(w2.y & 0xFFFF0000u)};
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float dht = carry[j][r] + gq * w2v[r];   // Q_t[u] = W2[u] . h_t + b2[u]
                    dan[j][r] = dht * fac[0][r];
                    dahn[j][r] = dan[j][r] * fac[1][r];
                    dar[j][r] = dan[j][r] * fac[2][r];
                    daz[j][r] = dht * fac[3][r];
                    carry[j][r] = dht * fac[4][r];
                }
            }
            typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
            const f32x4 (*const parts[3])[2] = {&dar, &daz, &dahn};
#pragma unroll
            for (int g = 0; g < 3; ++g)
                *reinterpret_cast<bf16x8 *>(lds + da_at(t) + (g * KS + w) * kFrag + (lane_at ^ (w * 64))) = frag_of_pair<1>((*parts[g])[0], (*parts[g])[1]).hi;
            // (the other three go to memory from LDS, for n is no room there.  The slot's part in the lanes' offset, not in the scalar
            // one: behind a 16-byte store with a scalar offset the compiler lets the next instruction overwrite the registers that
            // are being stored, and values of the next instruction's have been stored here.)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, frag_of_pair<1>(dan[0], dan[1]).hi), da_buf, da_lane + (uint32_t)t * da_slot, 0, 0);
            typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
            typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
            bf16x4 dq;                                             // the adjoint of Q_t, dense
#pragma unroll
            for (int r = 0; r < 4; ++r) dq[r] = (__bf16)(u - action0 == r ? gq : 0.0f);
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, dq), dq_buf, dq_lane, (uint32_t)t * dq_slot, 0);
            if (ask) fetch(in, t - 2);
            lds_barrier();
        };
        // Two steps a round; an odd one comes first, from a set of its own.  (A way out of the middle of the loop the compiler leads
        // through the loop's end, and what was asked for last on that way is then waited for at the head of every round.)
        const int odd = (a.t_end - a.t_begin) & 1;
        In first, set_a, set_b;
        fetch(first, a.t_end - 1);
        fetch(set_a, a.t_end - 1 - odd);
        fetch(set_b, a.t_end - 2 - odd);
        arrived(first);
        arrived(set_a);
        arrived(set_b);
        __builtin_amdgcn_s_setprio(2);                             // a SIMD's issue slots go to the chain first
        lds_barrier();                                             // biases, W2, zeros, the last slot's x and h
        lds_barrier();                                             // its factors
        if (odd) step(first, a.t_end - 1, false);
        for (int t = a.t_end - 1 - odd; t >= a.t_begin; t -= 2) {
            step(set_a, t, true);
            __builtin_amdgcn_sched_barrier(0);
            step(set_b, t - 1, true);
        }
        if (a.t_begin > 0) {
            back_product(a.t_begin);
#pragma unroll
            for (int j = 0; j < 2; ++j) *reinterpret_cast<f32x4 *>(a.carry + carry_at + 16 * j) = carry[j];
        }
    } else {
        // ---------------------------------------------------------------- gate wave
        const int w = wave, unit0 = 16 * w + 4 * q4;               // the lane's four units of a product's result
        // What this wave moves: rows 2 w and 2 w + 1, half its lanes each, four units a lane: an access whose neighbouring lanes are
        // different rows, as an operand has them, takes the address unit 64 clocks, one of neighbours side by side 16.
        const int mr = 2 * w + (lane >> 5), j = lane & 31, mrow = blockIdx.x * 16 + mr;
        const bool there = mrow < rows;
        const int mb = there ? mrow / N : 0, mn = there ? mrow % N : 0;
        const __amdgpu_buffer_rsrc_t da_buf = __builtin_amdgcn_make_buffer_rsrc(a.da, 0, (int)(uint32_t)(samples * 4 * H * 2), kRawBuffer);
        // r and z of the row, 16 bytes a lane; n of the hidden side on half the lanes
        const uint32_t da_lane = there ? ((uint32_t)mb * T * N + mn) * 4 * H * 2 + 2 * H + 16 * j : kPast, da_slot = (uint32_t)N * 4 * H * 2;
        const uint32_t last_lane = there && j < 16 ? da_lane + 2 * 2 * H : kPast;
        const int piece_at = column_at(j >> 2 & 3, j & 3, mr);     // of 16 bytes j % 16 of a part, in its fragments
        auto store_left = [&](int t) {                             // adjoints(t), left in LDS by the chain
            typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
            const char *const from = lds + da_at(t) + (j >> 2 & 3) * kFrag + piece_at;
            const u32x4 rz = *reinterpret_cast<const u32x4 *>(from + (j >> 4) * KS * kFrag), nh = *reinterpret_cast<const u32x4 *>(from + 2 * KS * kFrag);
            const uint32_t slot_at = (uint32_t)t * da_slot;
            __builtin_amdgcn_raw_buffer_store_b128(rz, da_buf, t < a.t_end ? da_lane + slot_at : kPast, 0, 0);
            __builtin_amdgcn_raw_buffer_store_b128(nh, da_buf, t < a.t_end ? last_lane + slot_at : kPast, 0, 0);
        };
        WFrag<1> whh[3][KS], wih[3][KS];
#pragma unroll
        for (int gate = 0; gate < 3; ++gate)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const size_t at = (size_t)((gate * FBK + w) * KS + ks) * 64 + lane;
                whh[gate][ks] = load_wfrag<1>(net.whh_16 + at);
                wih[gate][ks] = load_wfrag<1>(net.wih_16 + at);
            }
        // x stays the bf16 that it is in memory: an operand as it lies
        struct In { f32x4 h; uint2 x; };
        const uint32_t saved0 = ((uint32_t)mb * S * N + mn) * H + 4 * j;
        auto fetch = [&](In &in, int t) {
            const uint32_t at = saved0 + (uint32_t)max(t, 0) * (uint32_t)(N * H);
            in.h = *reinterpret_cast<const f32x4 *>(reinterpret_cast<const char *>(a.h_all) + at * 4u);
            in.x = *reinterpret_cast<const uint2 *>(static_cast<const char *>(a.x_all) + at * 2u);
        };
        auto arrived = [](In &in) { asm volatile("" : "+v"(in.h), "+v"(in.x.x), "+v"(in.x.y)); };
        const int moved_at = (j >> 3) * kFrag + column_at(j >> 3, j & 3, mr) + (j >> 2 & 1) * 8;      // block j / 4, quarter j % 4
        auto put_down = [&](const In &in, int t) {
            typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
            bf16x4 hb;
#pragma unroll
            for (int r = 0; r < 4; ++r) hb[r] = (__bf16)in.h[r];
            *reinterpret_cast<bf16x4 *>(lds + Bs::oH + (t & 1) * KS * kFrag + moved_at) = hb;
            *reinterpret_cast<uint2 *>(lds + Bs::oX + (t & 1) * KS * kFrag + moved_at) = in.x;
            *reinterpret_cast<f32x4 *>(lds + Bs::oHf + (t & 1) * Bs::kHfBytes + mr * Bs::kHfPitch + 16 * j) = in.h;
        };
        auto gates = [&](int t) {
            f32x4 acc_r = load_feature4(bias_lds, w, q4), acc_z = load_feature4(bias_lds + H, w, q4);
            f32x4 acc_in = load_feature4(bias_lds + 2 * H, w, q4), acc_hn = load_feature4(bias_lds + 3 * H, w, q4);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const Frag<1> hb = operand(Bs::oH + (t & 1) * KS * kFrag, ks), xb = operand(Bs::oX + (t & 1) * KS * kFrag, ks);
                mma16<1>(acc_r, whh[0][ks], hb);
                mma16<1>(acc_z, whh[1][ks], hb);
                mma16<1>(acc_hn, whh[2][ks], hb);
                mma16<1>(acc_r, wih[0][ks], xb);
                mma16<1>(acc_z, wih[1][ks], xb);
                mma16<1>(acc_in, wih[2][ks], xb);
            }
            const f32x4 hp = *reinterpret_cast<const f32x4 *>(lds + Bs::oHf + (t & 1) * Bs::kHfBytes + c * Bs::kHfPitch + unit0 * 4);
            f32x4 fac[Bs::kFactors];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float rr = sigmoidf_fast(acc_r[r]), zz = sigmoidf_fast(acc_z[r]);
                const float nn = tanhf_fast(acc_in[r] + rr * acc_hn[r]);
                fac[0][r] = (1.0f - zz) * (1.0f - nn * nn);        // dL/dh_t -> n
                fac[1][r] = rr;                                    // n -> n hidden side
                fac[2][r] = acc_hn[r] * rr * (1.0f - rr);          // n -> r
                fac[3][r] = (hp[r] - nn) * zz * (1.0f - zz);       // dL/dh_t -> z
                fac[4][r] = zz;                                    // dL/dh_t -> what passes the cell by
            }
#pragma unroll
            for (int f = 0; f < Bs::kFactors; ++f) *fac_of(t, f, w) = fac[f];
        };
        // in turn: slot t-2's, the one asked for; an odd step comes first, as the chain's
        const int odd = (a.t_end - a.t_begin) & 1;
        In first, set_a, set_b;
        fetch(first, a.t_end - 1);
        fetch(set_a, a.t_end - 2);
#pragma unroll
        for (int gate = 0; gate < 3; ++gate)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) { settle(whh[gate][ks]); settle(wih[gate][ks]); }
        arrived(first);
        put_down(first, a.t_end - 1);
        fetch(first, a.t_end - 3);
        fetch(set_b, a.t_end - 3 - odd);
        lds_barrier();
        gates(a.t_end - 1);
        arrived(set_a);
        put_down(set_a, a.t_end - 2);
        lds_barrier();
        auto step = [&](const In &next, int t) {
            if (w < 4) gates(t - 1);                               // (a SIMD has one wave of either order)
            store_left(t + 1);
            put_down(next, t - 2);
            if (w >= 4) gates(t - 1);
            lds_barrier();
        };
        arrived(first);
        arrived(set_b);
        if (odd) step(first, a.t_end - 1);
        for (int t = a.t_end - 1 - odd; t >= a.t_begin; t -= 2) {
            fetch(set_a, t - 3);
            __builtin_amdgcn_sched_barrier(0);
            step(set_b, t);
            fetch(set_b, t - 4);
            __builtin_amdgcn_sched_barrier(0);
            step(set_a, t - 1);
        }
        store_left(a.t_begin);
    }
}

// The same for 64 hidden units, cut into two roles.  What bounds it is issue and latency, not memory or the matrix
// cores: four waves in one role issue 508 instructions each per slot (two planes; 326 of them vector arithmetic, 72
// products), one wave per SIMD, so that nothing hides a wait: 1.97 us per slot, fp32.  But only
// dL/dh_t -> adjoints -> dL/dh_{t-1} is a chain; the gates of a slot and the adjoint of x hang on nothing behind them.
// Eight waves, two per SIMD, 258 (chain) and 242 (gates) instructions a slot: in the step of slot t
//
//   chain waves 0..3  dL/dh_t = carry + W_hh^T adjoints(t+1), beside it W_ih^T adjoints(t+1) -> dpre1 of slot t+1 (the
//                     same operands, and matrix instructions that do not wait for each other), then slot t's
//                     adjoints from its gate factors, to LDS as operand and to memory
//   gate waves 4..7   the gates of slot t-1 -> factors, in LDS; x and h of slot t-2 to LDS as operand, the loads of
//                     slot t-3
//
// and ONE barrier per slot.  Every LDS buffer is double-buffered on the parity of its slot: written in one step, read
// in the next, written again only in the one after.  All weights are in registers.  Waves w and w + 4 own the same
// 16 units, in the same lanes.  Kernel trace, us per launch, four waves in one role / split with the adjoint of x on the
// gate waves, which then issue more than the chain does / on the chain waves / with the stores' offsets as below:
// 64 episodes x 120 slots x 5 agents fp32 237 / 178 / 165 / 158.  First and last form: 4 x 60 x 3 fp32 115 / 80,
// 37 x 83 x 5 bf16 116 / 82.
// One plane: 126 registers and 68 KB of LDS, two workgroups per compute unit, asked for with the launch bound.  With one
// (136 registers) a batch of a few more than 256 tiles walked all its slots twice over: gradient of 820 episodes x 199
// slots x 5 agents (257 tiles) 1080 -> 1055 us, 4096 x 1 x 5 89 -> 85 us.  The fewer instructions per store help few
// tiles too.  (Two planes need 192 registers.)
template <int P> struct BpttSplit {
    static constexpr int H = 64, KS = H / 32, FBK = H / 16, kFrag = P * 1024;
    static constexpr int kFactors = 5;
    static constexpr int oH = 0, oX = oH + 2 * KS * kFrag, oDa = oX + 2 * KS * kFrag, kDaBytes = 4 * KS * kFrag;
    static constexpr int oFac = oDa + 2 * kDaBytes, kFacBytes = kFactors * FBK * 1024 + FBK * 256;      // five factors of every unit, and four bits a lane: x > 0
    static constexpr int oBias = oFac + 2 * kFacBytes, kBytes = oBias + 4 * H * 4;       // biases r, z, n input side, n hidden side
};

template <int P>
__global__ __launch_bounds__(512, P == 1 ? 4 : 2) void bptt_back_split_kernel(BpttArgs a)
{
    using Bs = BpttSplit<P>;
    constexpr int H = Bs::H, KS = Bs::KS, FBK = Bs::FBK, kFrag = Bs::kFrag;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    typedef bf16x8 (*FragBuf)[P][64];
    float *const bias_lds = reinterpret_cast<float *>(lds + Bs::oBias);

    const NetFrags &net = a.net;
    const int lane = threadIdx.x & 63, q4 = lane >> 4, c = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), w = wave & 3;
    const int N = net.N, A = net.A, T = a.T, S = T + 1;
    const int rows = a.B * N;
    const int row = blockIdx.x * 16 + c;
    const bool valid = row < rows;
    const int b = valid ? row / N : 0, n = valid ? row % N : 0;
    const int unit0 = 16 * w + 4 * q4;                             // the lane's four units

    constexpr uint32_t kElem = P == 1 ? 2u : 4u;                   // bytes per stored adjoint
    const size_t samples = (size_t)rows * T;
    auto operand = [&](int at) {                                   // at: byte offset of a fragment
        Frag<P> f;
        const FragBuf p = reinterpret_cast<FragBuf>(lds + at);
        f.hi = p[0][0][lane];
        if constexpr (P == 2) f.lo = p[0][1][lane];
        return f;
    };
    auto publish = [&](int at, const f32x4 &v) { publish_block<P>(reinterpret_cast<FragBuf>(lds + at), w, lane, v); };
    auto da_at = [](int t) { return Bs::oDa + (t & 1) * Bs::kDaBytes; };
    auto fac_of = [&](int t, int f) { return reinterpret_cast<f32x4 *>(lds + Bs::oFac + (t & 1) * Bs::kFacBytes + (f * FBK + w) * 1024) + lane; };
    auto bits_of = [&](int t) { return reinterpret_cast<uint32_t *>(lds + Bs::oFac + (t & 1) * Bs::kFacBytes + Bs::kFactors * FBK * 1024 + w * 256) + lane; };
    uint32_t drop = valid ? 0u : kDrop;
    asm volatile("" : "+v"(drop));
    const uint32_t bt0 = (uint32_t)b * T, btn0 = bt0 * N + n;      // the host bounds 4 H samples to 2^30

    if (wave < 4) {
        // ---------------------------------------------------------------- chain wave
        const __amdgpu_buffer_rsrc_t da_buf = __builtin_amdgcn_make_buffer_rsrc(a.da, 0, (int)(uint32_t)(samples * 4 * H * kElem), kRawBuffer);
        const __amdgpu_buffer_rsrc_t dq_buf = __builtin_amdgcn_make_buffer_rsrc(a.dq, 0, (int)(uint32_t)(samples * a.a16 * kElem), kRawBuffer);
        const uint32_t drop_dq = (16 * w < a.a16) ? drop : kDrop;  // wave w writes block w of the row's dQ
        const __amdgpu_buffer_rsrc_t pre_buf = __builtin_amdgcn_make_buffer_rsrc(a.dpre1, 0, (int)(uint32_t)(samples * H * kElem), kRawBuffer);
        WFrag<P> whhT[3 * KS], wihT[3 * KS];
#pragma unroll
        for (int ks = 0; ks < 3 * KS; ++ks) {
            whhT[ks] = load_wfrag<P>(net.whhT_16 + ((size_t)(w * 3 * KS + ks) * P) * 64 + lane);
            wihT[ks] = load_wfrag<P>(net.wihT_16 + ((size_t)(w * 3 * KS + ks) * P) * 64 + lane);
        }
        {
            const int i = (int)threadIdx.x, gate = i / H, j = i % H;      // 256 threads, 4 H biases
            const float *src = gate == 0 ? net.bias_r : gate == 1 ? net.bias_z : gate == 2 ? net.bias_in : net.bias_hn;
            bias_lds[i] = src[j];
            static_assert(4 * H == 256, "one bias per thread of the chain waves");
        }
        // no adjoints behind the last slot: the first step's products add nothing
        for (int i = threadIdx.x; i < Bs::kDaBytes / 16; i += 256) reinterpret_cast<uint4 *>(lds + da_at(a.t_end))[i] = make_uint4(0, 0, 0, 0);

        // A slot's inputs are asked for two steps ahead, its action (which picks the row of W2) two more; three register
        // sets take turns in the unrolled loop, for a set that is copied has to have arrived.
        struct In { f32x4 w2; float gq_raw; uint32_t fil; int u, u_ahead; };
        auto action = [&](int t) { return a.actions[btn0 + (uint32_t)max(t, 0) * N]; };
        auto fetch = [&](In &in, int t, int u_raw) {
            const uint32_t at = (uint32_t)max(t, 0);
            in.u = min(max(u_raw, 0), A - 1);
            in.fil = a.filled[bt0 + at];
            in.gq_raw = a.grad_q[btn0 + at * N];
            in.w2 = *reinterpret_cast<const f32x4 *>(net.w2_plain + (uint32_t)(in.u * H + unit0));
            in.u_ahead = action(t - 2);
        };
        const uint32_t carry_at = (uint32_t)row * H + unit0;       // rows past the end have room too
        f32x4 carry = {0.0f, 0.0f, 0.0f, 0.0f};
        if (a.t_end < T) carry = *reinterpret_cast<const f32x4 *>(a.carry + carry_at);
        In set_a, set_b, set_c;
        fetch(set_a, a.t_end - 1, action(a.t_end - 1));
        fetch(set_b, a.t_end - 2, action(a.t_end - 2));
#pragma unroll
        for (int ks = 0; ks < 3 * KS; ++ks) { settle(whhT[ks]); settle(wihT[ks]); }
        asm volatile("" : "+v"(set_a.w2), "+v"(set_a.gq_raw), "+v"(set_a.fil), "+v"(set_a.u), "+v"(set_a.u_ahead), "+v"(carry));
        asm volatile("" : "+v"(set_b.w2), "+v"(set_b.gq_raw), "+v"(set_b.fil), "+v"(set_b.u), "+v"(set_b.u_ahead));

        // Offsets of the stores: the lane's own part, and the slot's, the same in every lane.  The slot's is hidden from the
        // compiler, which would otherwise step an address of its own for every store of the unrolled loop (ten registers,
        // with which two workgroups of a one-plane network do not fit a compute unit).
        const uint32_t da_lane = btn0 * 4 * H + unit0, pre_lane = btn0 * H + unit0, dq_lane = btn0 * a.a16 + unit0;
        auto rows_before = [&](int t) { uint32_t r = (uint32_t)t * N; asm volatile("" : "+s"(r)); return r; };
        uint32_t positive = 0;                                     // x > 0 of the slot whose adjoints were formed last
        auto back_product = [&](int t, uint32_t drop_mask) {       // carry += W_hh^T adjoints(t); dpre1 of slot t
            f32x4 accx = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int ks = 0; ks < 3 * KS; ++ks) {
                const Frag<P> di = operand(da_at(t) + ks * kFrag);
                const Frag<P> dhid = ks < 2 * KS ? di : operand(da_at(t) + (ks + KS) * kFrag);
                mma16<P>(carry, whhT[ks], dhid);
                mma16<P>(accx, wihT[ks], di);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) accx[r] = positive >> r & 1u ? accx[r] : 0.0f;
            store_adjoints<P>(accx, pre_buf, pre_lane + rows_before(t) * H, drop_mask);
        };
        auto step = [&](const In &in, In &nxt, int t) {
            fetch(nxt, t - 2, in.u_ahead);
            f32x4 fac[Bs::kFactors];
#pragma unroll
            for (int f = 0; f < Bs::kFactors; ++f) fac[f] = *fac_of(t, f);
            back_product(t + 1, t + 1 < a.t_end ? drop : kDrop);
            positive = *bits_of(t);
            const float gq = (valid && in.fil) ? in.gq_raw : 0.0f;
            f32x4 dan, dar, daz, dahn;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float dht = carry[r] + gq * in.w2[r];        // Q_t[u] = W2[u] . h_t + b2[u]
                dan[r] = dht * fac[0][r];
                dahn[r] = dan[r] * fac[1][r];
                dar[r] = dan[r] * fac[2][r];
                daz[r] = dht * fac[3][r];
                carry[r] = dht * fac[4][r];
            }
            publish(da_at(t) + 0 * KS * kFrag, dar);
            publish(da_at(t) + 1 * KS * kFrag, daz);
            publish(da_at(t) + 2 * KS * kFrag, dan);
            publish(da_at(t) + 3 * KS * kFrag, dahn);
            const uint32_t tn = rows_before(t), at = da_lane + tn * 4 * H;
            store_adjoints<P>(dan, da_buf, at + 0 * H, drop);
            store_adjoints<P>(dar, da_buf, at + 1 * H, drop);
            store_adjoints<P>(daz, da_buf, at + 2 * H, drop);
            store_adjoints<P>(dahn, da_buf, at + 3 * H, drop);
            f32x4 v;                                               // the adjoint of Q_t, dense
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = in.u - unit0 == r ? gq : 0.0f;
            store_adjoints<P>(v, dq_buf, dq_lane + tn * a.a16, drop_dq);
            lds_barrier();
        };
        lds_barrier();                                             // biases, zeros, the last slot's x and h
        lds_barrier();                                             // its factors
        for (int t = a.t_end - 1;;) {
            step(set_a, set_c, t);
            if (--t < a.t_begin) break;
            step(set_b, set_a, t);
            if (--t < a.t_begin) break;
            step(set_c, set_b, t);
            if (--t < a.t_begin) break;
        }
        back_product(a.t_begin, drop);
        if (a.t_begin > 0) *reinterpret_cast<f32x4 *>(a.carry + carry_at) = carry;
    } else {
        // ---------------------------------------------------------------- gate wave
        WFrag<P> whh[3][KS], wih[3][KS];
#pragma unroll
        for (int gate = 0; gate < 3; ++gate)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const size_t at = ((size_t)((gate * FBK + w) * KS + ks) * P) * 64 + lane;
                whh[gate][ks] = load_wfrag<P>(net.whh_16 + at);
                wih[gate][ks] = load_wfrag<P>(net.wih_16 + at);
            }
        // x of a one-plane network stays the bf16 that it is in memory: an operand as it lies
        using XRegs = std::conditional_t<P == 1, uint2, f32x4>;
        struct In { f32x4 h; XRegs x; };
        const uint32_t saved0 = ((uint32_t)b * S * N + n) * H + unit0;
        auto fetch = [&](In &in, int t) {
            const uint32_t at = saved0 + (uint32_t)max(t, 0) * (uint32_t)(N * H);
            in.h = *reinterpret_cast<const f32x4 *>(a.h_all + at);
            in.x = *reinterpret_cast<const XRegs *>(static_cast<const char *>(a.x_all) + (size_t)at * kElem);
        };
        uint32_t positive = 0;                                     // x > 0 of the slot put down last
        auto put_down = [&](const In &in, int t) {
            publish(Bs::oH + (t & 1) * KS * kFrag, in.h);
            uint32_t bits = 0;
            if constexpr (P == 1) {
                char *at = lds + Bs::oX + (t & 1) * KS * kFrag + (w / 2) * kFrag + lane * 16 + (w & 1) * 8;
                *reinterpret_cast<uint2 *>(at) = in.x;
                bits = (__uint_as_float(in.x.x << 16) > 0.0f ? 1u : 0u) | (__uint_as_float(in.x.x & 0xFFFF0000u) > 0.0f ? 2u : 0u)
                       | (__uint_as_float(in.x.y << 16) > 0.0f ? 4u : 0u) | (__uint_as_float(in.x.y & 0xFFFF0000u) > 0.0f ? 8u : 0u);
            } else {
                publish(Bs::oX + (t & 1) * KS * kFrag, in.x);
#pragma unroll
                for (int r = 0; r < 4; ++r) bits |= in.x[r] > 0.0f ? 1u << r : 0u;
            }
            positive = bits;
        };
        auto gates = [&](const In &in, int t) {
            f32x4 acc_r = load_feature4(bias_lds, w, q4), acc_z = load_feature4(bias_lds + H, w, q4);
            f32x4 acc_in = load_feature4(bias_lds + 2 * H, w, q4), acc_hn = load_feature4(bias_lds + 3 * H, w, q4);
            f32x4 *const acc_h[3] = {&acc_r, &acc_z, &acc_hn}, *const acc_x[3] = {&acc_r, &acc_z, &acc_in};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const WFrag<P> *const wh[3] = {&whh[0][ks], &whh[1][ks], &whh[2][ks]}, *const wx[3] = {&wih[0][ks], &wih[1][ks], &wih[2][ks]};
                mma16_across<P, 3>(acc_h, wh, operand(Bs::oH + ((t & 1) * KS + ks) * kFrag));
                mma16_across<P, 3>(acc_x, wx, operand(Bs::oX + ((t & 1) * KS + ks) * kFrag));
            }
            f32x4 fac[Bs::kFactors];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float rr = sigmoidf_fast(acc_r[r]), zz = sigmoidf_fast(acc_z[r]);
                const float nn = tanhf_fast(acc_in[r] + rr * acc_hn[r]);
                fac[0][r] = (1.0f - zz) * (1.0f - nn * nn);        // dL/dh_t -> n
                fac[1][r] = rr;                                    // n -> n hidden side
                fac[2][r] = acc_hn[r] * rr * (1.0f - rr);          // n -> r
                fac[3][r] = (in.h[r] - nn) * zz * (1.0f - zz);     // dL/dh_t -> z
                fac[4][r] = zz;                                    // dL/dh_t -> what passes the cell by
            }
#pragma unroll
            for (int f = 0; f < Bs::kFactors; ++f) *fac_of(t, f) = fac[f];
            *bits_of(t) = positive;
        };
        In set_a, set_b, set_c;                                    // in turn: slot t-1's, slot t-2's, the one asked for
        fetch(set_c, a.t_end - 1);
        fetch(set_a, a.t_end - 2);
        fetch(set_b, a.t_end - 3);
#pragma unroll
        for (int gate = 0; gate < 3; ++gate)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) { settle(whh[gate][ks]); settle(wih[gate][ks]); }
        for (In *in : {&set_a, &set_b, &set_c}) {
            asm volatile("" : "+v"(in->h));
            if constexpr (P == 1) asm volatile("" : "+v"(in->x.x), "+v"(in->x.y));
            else asm volatile("" : "+v"(in->x));
        }
        put_down(set_c, a.t_end - 1);
        lds_barrier();
        gates(set_c, a.t_end - 1);
        put_down(set_a, a.t_end - 2);
        lds_barrier();
        auto step = [&](const In &at_gates, const In &next, In &asked, int t) {
            fetch(asked, t - 3);
            gates(at_gates, t - 1);
            put_down(next, t - 2);
            lds_barrier();
        };
        for (int t = a.t_end - 1;;) {
            step(set_a, set_b, set_c, t);
            if (--t < a.t_begin) break;
            step(set_b, set_c, set_a, t);
            if (--t < a.t_begin) break;
            step(set_c, set_a, set_b, t);
            if (--t < a.t_begin) break;
        }
    }
}

// The same two roles on tiles of eight rows, for batches that leave compute units free.
//
// An operand's sixteen columns are the eight rows twice: two planes, the high parts and the remainders side by side (c < 8,
// c >= 8), so that W_hi and W_lo take one product each, two instead of three, and the sum of a row's two columns is the whole (W_lo
// times the remainder with it); one plane, the same values twice.  Either way lane (c, q4) then has two of the four units 4 q4 .. +
// 3, those of its side (c / 8), to go on with: half the vector instructions per lane.
//
// What goes to memory and comes from it goes through LDS, and waves of their own move it, two rows each, a row's lanes side by
// side: an access whose neighbouring lanes are different rows, as an operand has them, takes the address unit 64 clocks, one whose
// neighbours lie side by side 8 to 16, and the kernel above has 48 of them a slot (3,000 clocks; a slot took 2,900).  In the
// step of slot t
//
//   chain waves 0..3  as above; adjoints(t) and the adjoint of fc1's pre-activation of slot t+1 to LDS, nothing to memory
//   gate waves 4..7   the gates of slot t-1 -> factors
//   movers 8..11      x and h of slot t-2 to LDS, its rows' scalars, its adjoint of Q to memory; what the chain left in the step
//                     before to memory; the loads of slot t-3
//
// Kernel trace, us per launch: 64 episodes x 120 slots x 5 agents fp32 156 on tiles of 16; of 8 with the accesses as there 111, moved
// by the gate waves 111 (then what a step waits for), by waves of their own 103; 37 x 83 x 5 bf16 82, 56, 63, 46.  Eight gate waves,
// every four with every other slot, as long as they also fetched: 140, 66.
template <int P> struct BpttSplit8 {
    static constexpr int H = 64, KS = H / 32, FBK = H / 16, kThreads = 3 * 256, kElem = P == 1 ? 2 : 4;      // bytes per stored adjoint
    static constexpr int kColumns = P == 2 ? 16 : 8, kFrag = 4 * kColumns * 16;          // of an operand that are kept
    static constexpr int kFactors = 5, kPair = FBK * 512;                                // two floats of every lane and block
    static constexpr int oH = 0, oX = oH + 2 * KS * kFrag, oDa = oX + 2 * KS * kFrag, kDaBytes = 4 * KS * kFrag;
    static constexpr int oFac = oDa + 2 * kDaBytes, kFacBytes = kFactors * kPair;
    // row by row, the pitches 64 bytes past a multiple of 256: h in fp32, for the blend; the adjoints and dpre1 as they are stored
    static constexpr int oHf = oFac + 2 * kFacBytes, kHfPitch = H * 4 + 64, kHfBytes = 8 * kHfPitch;
    static constexpr int oOut = oHf + 2 * kHfBytes, kOutPitch = 4 * H * kElem + 64, kOutBytes = 8 * kOutPitch;
    static constexpr int oPre = oOut + 2 * kOutBytes, kPrePitch = (H * kElem + 255) / 256 * 256 + 64, kPreBytes = 8 * kPrePitch;
    static constexpr int oBias = oPre + 2 * kPreBytes;             // r, z, n input side, n hidden side; zeros
    static constexpr int oRow = oBias + 5 * H * 4, kRowBytes = 8 * 8;                    // per row: dL/dq_taken, its action; of four slots
    // W2, whose row of the chosen action the chain adds; bf16 for a one-plane network (what the table holds exactly)
    static constexpr int oW2 = oRow + 4 * kRowBytes, kW2Pitch = H * kElem + 4 * kElem;
    static constexpr int lds_bytes(int A) { return oW2 + (A * kW2Pitch + 15) / 16 * 16; }
};

template <int P>
__global__ __launch_bounds__(BpttSplit8<P>::kThreads, BpttSplit8<P>::kThreads / 256) void bptt_back_split8_kernel(BpttArgs a)
{
    using Bs = BpttSplit8<P>;
    constexpr int H = Bs::H, KS = Bs::KS, FBK = Bs::FBK, kFrag = Bs::kFrag, kElem = Bs::kElem;
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    extern __shared__ __attribute__((aligned(16))) char lds[];
    float *const bias_lds = reinterpret_cast<float *>(lds + Bs::oBias);

    const NetFrags &net = a.net;
    const int lane = threadIdx.x & 63, q4 = lane >> 4, c = lane & 15, side = c >> 3, r8 = c & 7;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), w = wave & 3;
    const int N = net.N, A = net.A, T = a.T, S = T + 1;
    const int rows = a.B * N, row0 = blockIdx.x * 8;
    const int unit0 = 16 * w + 4 * q4 + 2 * side;                  // the two units of the lane's in a product's result

    struct Pair { float v[2]; };
    // Where an operand keeps column `col` of lane quarter `quarter` in k-step ks: the columns change places from quarter to quarter
    // and k-step to k-step, or the writers, who have a row's units side by side, would all meet in one bank.
    auto column_at = [](int ks, int quarter, int col) { return (quarter * Bs::kColumns + (col ^ (quarter + 4 * (ks & 1)))) * 16; };
    const int operand_at[2] = {column_at(0, q4, c & (Bs::kColumns - 1)), column_at(1, q4, c & (Bs::kColumns - 1))};
    auto operand = [&](int at, int ks) { return *reinterpret_cast<const bf16x8 *>(lds + at + ks * kFrag + operand_at[ks & 1]); };
    // two units as their part of an operand; `where`: publish_at of them
    auto publish_at = [&](int row, int unit) { return (unit >> 5) * kFrag + column_at(unit >> 5, (unit & 15) >> 2, row) + (unit >> 4 & 1) * 8 + (unit & 3) * 2; };
    auto publish = [&](int where, const Pair &x) {
        bf16x2 hi;
        hi[0] = (__bf16)x.v[0]; hi[1] = (__bf16)x.v[1];
        *reinterpret_cast<bf16x2 *>(lds + where) = hi;
        if constexpr (P == 2) {
            bf16x2 lo;
            lo[0] = (__bf16)(x.v[0] - (float)hi[0]); lo[1] = (__bf16)(x.v[1] - (float)hi[1]);
            *reinterpret_cast<bf16x2 *>(lds + (where ^ (8 * 16))) = lo;      // column + 8
        }
    };
    // A row's two columns, of which this lane holds one -> the two units of the lane's side.  (Bits, for of a choice between
    // elements the compiler makes a search for the element, three instructions.)
    uint32_t upper = side ? 0xFFFFFFFFu : 0u;
    asm volatile("" : "+v"(upper));
    auto mine = [&](const f32x4 &acc) {
        Pair x;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t first = __float_as_uint(acc[i]), second = __float_as_uint(acc[2 + i]);
            x.v[i] = __uint_as_float(first ^ (upper & (second ^ first)));
            if constexpr (P == 2) {
                const uint32_t other = second ^ (upper & (first ^ second));                // what the lane of the other column is to have
                x.v[i] += __uint_as_float(__builtin_amdgcn_update_dpp(0, other, 0x128, 0xF, 0xF, true));      // row_ror:8
            }
        }
        return x;
    };
    auto product = [&](f32x4 &acc, const WFrag<P> &wf, const bf16x8 &d) {
        if constexpr (P == 2) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf.lo, d, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf.hi, d, acc, 0, 0, 0);
    };
    auto da_at = [](int t) { return Bs::oDa + (t & 1) * Bs::kDaBytes; };
    auto fac_of = [&](int t, int f) { return reinterpret_cast<f32x2 *>(lds + Bs::oFac + (t & 1) * Bs::kFacBytes + f * Bs::kPair + w * 512) + lane; };
    auto row_of = [&](int t, int r) { return reinterpret_cast<uint2 *>(lds + Bs::oRow + (t & 3) * Bs::kRowBytes) + r; };
    for (int i = threadIdx.x; i < A * H; i += Bs::kThreads) {
        char *const at = lds + Bs::oW2 + (i / H) * Bs::kW2Pitch + (i % H) * kElem;
        if constexpr (P == 1) *reinterpret_cast<__bf16 *>(at) = (__bf16)net.w2_plain[i];
        else *reinterpret_cast<float *>(at) = net.w2_plain[i];
    }

    if (wave < 4) {
        // ---------------------------------------------------------------- chain wave
        WFrag<P> whhT[3 * KS], wihT[3 * KS];
#pragma unroll
        for (int ks = 0; ks < 3 * KS; ++ks) {
            whhT[ks] = load_wfrag<P>(net.whhT_16 + ((size_t)(w * 3 * KS + ks) * P) * 64 + lane);
            wihT[ks] = load_wfrag<P>(net.wihT_16 + ((size_t)(w * 3 * KS + ks) * P) * 64 + lane);
        }
        {
            const int i = (int)threadIdx.x, gate = i / H, j = i % H;      // 256 threads, 4 H biases
            const float *src = gate == 0 ? net.bias_r : gate == 1 ? net.bias_z : gate == 2 ? net.bias_in : net.bias_hn;
            bias_lds[i] = src[j];
            if (i < H) bias_lds[4 * H + i] = 0.0f;
            static_assert(4 * H == 256, "one bias per thread of the chain waves");
        }
        // no adjoints behind the last slot: the first step's products add nothing
        for (int i = threadIdx.x; i < Bs::kDaBytes / 16; i += 256) reinterpret_cast<uint4 *>(lds + da_at(a.t_end))[i] = make_uint4(0, 0, 0, 0);

        const uint32_t carry_at = (uint32_t)(row0 + r8) * H + unit0;      // rows past the end have room too (16 is a multiple of 8)
        Pair carry = {};
        if (a.t_end < T) {
            carry.v[0] = a.carry[carry_at];
            carry.v[1] = a.carry[carry_at + 1];
        }
#pragma unroll
        for (int ks = 0; ks < 3 * KS; ++ks) { settle(whhT[ks]); settle(wihT[ks]); }
        asm volatile("" : "+v"(carry.v[0]), "+v"(carry.v[1]));

        const int mine_at = publish_at(r8, unit0);
        // what is to be stored, for the movers
        auto leave = [&](int at, const Pair &x) {
            if constexpr (P == 1) {
                bf16x2 v;
                v[0] = (__bf16)x.v[0]; v[1] = (__bf16)x.v[1];
                *reinterpret_cast<bf16x2 *>(lds + at + unit0 * kElem) = v;
            } else {
                *reinterpret_cast<f32x2 *>(lds + at + unit0 * kElem) = f32x2{x.v[0], x.v[1]};
            }
        };
        auto back_product = [&](int t) {                           // carry += W_hh^T adjoints(t); dpre1 of slot t, before the ReLU
            f32x4 acch = {0.0f, 0.0f, 0.0f, 0.0f}, accx = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int ks = 0; ks < 3 * KS; ++ks) {
                const bf16x8 di = operand(da_at(t), ks), dhid = ks < 2 * KS ? di : operand(da_at(t), ks + KS);
                product(acch, whhT[ks], dhid);
                product(accx, wihT[ks], di);
            }
            const Pair h = mine(acch);
#pragma unroll
            for (int i = 0; i < 2; ++i) carry.v[i] += h.v[i];
            leave(Bs::oPre + (t & 1) * Bs::kPreBytes + r8 * Bs::kPrePitch, mine(accx));
        };
        auto step = [&](int t) {
            const uint2 about = *row_of(t, r8);
            const float gq = __uint_as_float(about.x);
            const char *const w2_at = lds + Bs::oW2 + (int)about.y * Bs::kW2Pitch + unit0 * kElem;
            f32x2 w2;
            if constexpr (P == 1) {
                const uint32_t two = *reinterpret_cast<const uint32_t *>(w2_at);
                w2 = f32x2{__uint_as_float(two << 16), __uint_as_float(two & 0xFFFF0000u)};
            } else {
                w2 = *reinterpret_cast<const f32x2 *>(w2_at);
            }
            f32x2 fac[Bs::kFactors];
#pragma unroll
            for (int f = 0; f < Bs::kFactors; ++f) fac[f] = *fac_of(t, f);
            back_product(t + 1);
            Pair dan, dar, daz, dahn;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const float dht = carry.v[i] + gq * w2[i];         // Q_t[u] = W2[u] . h_t + b2[u]
                dan.v[i] = dht * fac[0][i];
                dahn.v[i] = dan.v[i] * fac[1][i];
                dar.v[i] = dan.v[i] * fac[2][i];
                daz.v[i] = dht * fac[3][i];
                carry.v[i] = dht * fac[4][i];
            }
            publish(da_at(t) + 0 * KS * kFrag + mine_at, dar);
            publish(da_at(t) + 1 * KS * kFrag + mine_at, daz);
            publish(da_at(t) + 2 * KS * kFrag + mine_at, dan);
            publish(da_at(t) + 3 * KS * kFrag + mine_at, dahn);
            const int out = Bs::oOut + (t & 1) * Bs::kOutBytes + r8 * Bs::kOutPitch;
            leave(out + 0 * H * kElem, dan);
            leave(out + 1 * H * kElem, dar);
            leave(out + 2 * H * kElem, daz);
            leave(out + 3 * H * kElem, dahn);
            lds_barrier();
        };
        lds_barrier();                                             // biases, zeros, the last slot's x and h
        lds_barrier();                                             // its factors
        for (int t = a.t_end - 1; t >= a.t_begin; --t) step(t);
        back_product(a.t_begin);
        lds_barrier();                                             // the last dpre1
        if (a.t_begin > 0) {
            a.carry[carry_at] = carry.v[0];
            a.carry[carry_at + 1] = carry.v[1];
        }
    } else if (wave < 8) {
        // ---------------------------------------------------------------- gate wave
        WFrag<P> whh[3][KS], wih[3][KS];
#pragma unroll
        for (int gate = 0; gate < 3; ++gate)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const size_t at = ((size_t)((gate * FBK + w) * KS + ks) * P) * 64 + lane;
                whh[gate][ks] = load_wfrag<P>(net.whh_16 + at);
                wih[gate][ks] = load_wfrag<P>(net.wih_16 + at);
            }
        // (two planes: the bias of a unit in one of a row's two columns)
        const float *const bias = P == 2 && side ? bias_lds + 4 * H : bias_lds + 16 * w + 4 * q4;
        const int bias_step = P == 2 && side ? 0 : H;
        auto gates = [&](int t) {
            f32x4 acc_r = *reinterpret_cast<const f32x4 *>(bias), acc_z = *reinterpret_cast<const f32x4 *>(bias + bias_step);
            f32x4 acc_in = *reinterpret_cast<const f32x4 *>(bias + 2 * bias_step), acc_hn = *reinterpret_cast<const f32x4 *>(bias + 3 * bias_step);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const bf16x8 hb = operand(Bs::oH + (t & 1) * KS * kFrag, ks), xb = operand(Bs::oX + (t & 1) * KS * kFrag, ks);
                product(acc_r, whh[0][ks], hb);
                product(acc_z, whh[1][ks], hb);
                product(acc_hn, whh[2][ks], hb);
                product(acc_in, wih[2][ks], xb);
                product(acc_r, wih[0][ks], xb);
                product(acc_z, wih[1][ks], xb);
            }
            const f32x2 hp = *reinterpret_cast<const f32x2 *>(lds + Bs::oHf + (t & 1) * Bs::kHfBytes + r8 * Bs::kHfPitch + unit0 * 4);
            const Pair pr = mine(acc_r), pz = mine(acc_z), pin = mine(acc_in), phn = mine(acc_hn);
            f32x2 fac[Bs::kFactors];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const float rr = sigmoidf_fast(pr.v[i]), zz = sigmoidf_fast(pz.v[i]);
                const float nn = tanhf_fast(pin.v[i] + rr * phn.v[i]);
                fac[0][i] = (1.0f - zz) * (1.0f - nn * nn);        // dL/dh_t -> n
                fac[1][i] = rr;                                    // n -> n hidden side
                fac[2][i] = phn.v[i] * rr * (1.0f - rr);           // n -> r
                fac[3][i] = (hp[i] - nn) * zz * (1.0f - zz);       // dL/dh_t -> z
                fac[4][i] = zz;                                    // dL/dh_t -> what passes the cell by
            }
#pragma unroll
            for (int f = 0; f < Bs::kFactors; ++f) *fac_of(t, f) = fac[f];
        };
#pragma unroll
        for (int gate = 0; gate < 3; ++gate)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) { settle(whh[gate][ks]); settle(wih[gate][ks]); }
        lds_barrier();
        gates(a.t_end - 1);
        lds_barrier();
        for (int t = a.t_end - 1; t >= a.t_begin; --t) {
            gates(t - 1);
            lds_barrier();
        }
        lds_barrier();
    } else {
        // ---------------------------------------------------------------- mover
        // What this wave moves: rows 2 w and 2 w + 1, half its lanes each, two units a lane.
        const int mr = 2 * w + (lane >> 5), j = lane & 31, mrow = row0 + mr;
        const bool valid = mrow < rows;
        const int b = valid ? mrow / N : 0, n = valid ? mrow % N : 0;
        const uint32_t bt0 = (uint32_t)b * T, btn0 = bt0 * N + n;  // the host bounds 4 H samples to 2^30
        const size_t samples = (size_t)rows * T;
        auto buffer = [&](void *p, size_t per_sample, bool exists) { return __builtin_amdgcn_make_buffer_rsrc(p, 0, (int)descriptor_bytes(samples * per_sample * kElem, exists), kRawBuffer); };
        const __amdgpu_buffer_rsrc_t dq_buf = buffer(a.dq, a.a16, true), pre_buf = buffer(a.dpre1, H, true);
        // A store's offset: the lane's own part (kPast, where the store is to be dropped), and the slot's, the same in every lane.
        // da: one plane, both rows, 16 bytes a lane; two planes, a row per access, with a descriptor of its own, for kPast may be in
        // the middle of the array.  (A mask over the offsets instead: seven instructions more per slot, 64 x 120 x 5 346.1 -> 347.3 us.)
        __amdgpu_buffer_rsrc_t da_buf[P];
        uint32_t da_lane[P];
        int da_from[P];
#pragma unroll
        for (int i = 0; i < P; ++i) {
            const int r = P == 2 ? 2 * w + i : mr, piece = P == 2 ? lane : j;
            const bool there = row0 + r < rows;
            const int rb = there ? (row0 + r) / N : 0, rn = there ? (row0 + r) % N : 0;
            da_buf[i] = buffer(a.da, 4 * H, P == 1 || there);
            da_lane[i] = P == 2 || there ? ((uint32_t)rb * T * N + rn) * 4 * H * kElem + 16 * piece : kPast;
            asm volatile("" : "+v"(da_lane[i]));                   // (one vector register, not a sum with a scalar that is stepped for itself)
            da_from[i] = Bs::oOut + r * Bs::kOutPitch + 16 * piece;
        }
        const uint32_t pre_lane = valid ? (btn0 * H + 2 * j) * kElem : kPast, dq_lane = valid && 2 * j < a.a16 ? (btn0 * a.a16 + 2 * j) * kElem : kPast;
        const uint32_t da_slot = (uint32_t)N * 4 * H * kElem, pre_slot = (uint32_t)N * H * kElem, dq_slot = (uint32_t)N * a.a16 * kElem;
        auto store2 = [](const Pair &x, const __amdgpu_buffer_rsrc_t &buf, uint32_t lane_at, uint32_t slot_at) {
            if constexpr (P == 1) {
                bf16x2 v;
                v[0] = (__bf16)x.v[0]; v[1] = (__bf16)x.v[1];
                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), buf, lane_at, slot_at, 0);
            } else {
                __builtin_amdgcn_raw_buffer_store_b64(u32x2{__float_as_uint(x.v[0]), __float_as_uint(x.v[1])}, buf, lane_at, slot_at, 0);
            }
        };
        uint32_t positive = 0;                                     // x > 0 of the lane's units, slots put down last in the low bits
        // what the chain left in the step of slot t: adjoints(t), dpre1 of slot t+1
        auto store_pre = [&](int t, int age) {                     // age: slots put down since that one
            const int from = Bs::oPre + (t & 1) * Bs::kPreBytes + mr * Bs::kPrePitch + 2 * j * kElem;
            const uint32_t at = t < a.t_end ? pre_lane : kPast, slot_at = (uint32_t)min(t, T - 1) * pre_slot, on = positive >> (2 * age);
            if constexpr (P == 1) {
                const uint32_t v = *reinterpret_cast<const uint32_t *>(lds + from);
                __builtin_amdgcn_raw_buffer_store_b32(v & ((on & 1u ? 0xFFFFu : 0u) | (on & 2u ? 0xFFFF0000u : 0u)), pre_buf, at, slot_at, 0);
            } else {
                const f32x2 v = *reinterpret_cast<const f32x2 *>(lds + from);
                store2(Pair{on & 1u ? v[0] : 0.0f, on & 2u ? v[1] : 0.0f}, pre_buf, at, slot_at);
            }
        };
        auto store_left = [&](int t) {
#pragma unroll
            for (int i = 0; i < P; ++i) {
                const u32x4 v = *reinterpret_cast<const u32x4 *>(lds + da_from[i] + (t & 1) * Bs::kOutBytes);
                // (the slot's part not as a scalar offset: see the 16-byte stores of bptt_back_roles_kernel)
                __builtin_amdgcn_raw_buffer_store_b128(v, da_buf[i], store_offset(da_lane[i], (uint32_t)t * da_slot, t < a.t_end), 0, 0);
            }
        };

        using XRegs = std::conditional_t<P == 1, uint32_t, f32x2>;
        struct In { f32x2 h; XRegs x; float gq_raw; uint8_t fil; int u; };
        const uint32_t saved0 = ((uint32_t)b * S * N + n) * H + 2 * j;
        auto fetch = [&](In &in, int t) {
            const uint32_t ts = (uint32_t)max(t, 0), at = saved0 + ts * (uint32_t)(N * H), sample = btn0 + ts * N;
            in.h = *reinterpret_cast<const f32x2 *>(reinterpret_cast<const char *>(a.h_all) + at * 4u);
            in.x = *reinterpret_cast<const XRegs *>(static_cast<const char *>(a.x_all) + at * (uint32_t)kElem);
            in.fil = a.filled[bt0 + ts];
            in.gq_raw = *reinterpret_cast<const float *>(reinterpret_cast<const char *>(a.grad_q) + sample * 4u);
            in.u = *reinterpret_cast<const int *>(reinterpret_cast<const char *>(a.actions) + sample * 4u);
        };
        auto arrived = [](In &in) {
            asm volatile("" : "+v"(in.h), "+v"(in.x));
            asm volatile("" ::"v"((uint32_t)in.fil));
            asm volatile("" : "+v"(in.gq_raw), "+v"(in.u));
        };
        const int moved_at = publish_at(mr, 2 * j);
        auto put_down = [&](const In &in, int t) {
            publish(Bs::oH + (t & 1) * KS * kFrag + moved_at, Pair{in.h[0], in.h[1]});
            *reinterpret_cast<f32x2 *>(lds + Bs::oHf + (t & 1) * Bs::kHfBytes + mr * Bs::kHfPitch + 8 * j) = in.h;
            if constexpr (P == 1) {                                // x stays the bf16 that it is in memory: an operand as it lies
                *reinterpret_cast<uint32_t *>(lds + Bs::oX + (t & 1) * KS * kFrag + moved_at) = in.x;
                positive = positive << 2 | (__uint_as_float(in.x << 16) > 0.0f ? 1u : 0u) | (__uint_as_float(in.x & 0xFFFF0000u) > 0.0f ? 2u : 0u);
            } else {
                publish(Bs::oX + (t & 1) * KS * kFrag + moved_at, Pair{in.x[0], in.x[1]});
                positive = positive << 2 | (in.x[0] > 0.0f ? 1u : 0u) | (in.x[1] > 0.0f ? 2u : 0u);
            }
            // (What passes through the empty asm is used here and not earlier: the compiler would widen `filled` where it is
            // loaded, and wait there.)
            uint32_t fil = in.fil;
            int u = in.u;
            float gq = in.gq_raw;
            asm volatile("" : "+v"(fil), "+v"(u), "+v"(gq));
            gq = valid && fil ? gq : 0.0f;
            u = min(max(u, 0), A - 1);
            *row_of(t, mr) = make_uint2(__float_as_uint(gq), (uint32_t)u);      // (every lane of the row has the same to say)
            // the adjoint of Q_t, dense
            store2(Pair{u == 2 * j ? gq : 0.0f, u == 2 * j + 1 ? gq : 0.0f}, dq_buf, t >= a.t_begin ? dq_lane : kPast, (uint32_t)max(t, 0) * dq_slot);
        };
        // In turn: slot t-2's, the one asked for.  Two steps a round; an odd one comes first, from a set of its own.  (A way out of
        // the middle of the loop the compiler leads through the loop's end, and what was asked for last on that way is then waited
        // for at the head of every round.)
        const int odd = (a.t_end - a.t_begin) & 1;
        In first, set_a, set_b;
        fetch(first, a.t_end - 1);
        fetch(set_a, a.t_end - 2);
        arrived(first);
        put_down(first, a.t_end - 1);
        fetch(first, a.t_end - 3);
        fetch(set_b, a.t_end - 3 - odd);
        lds_barrier();
        arrived(set_a);
        put_down(set_a, a.t_end - 2);
        lds_barrier();
        // In the step of slot t slots down to t-1 are put down: slot t+2 is three before the last.
        auto step = [&](const In &next, int t) {
            store_left(t + 1);
            store_pre(t + 2, 3);
            put_down(next, t - 2);
            lds_barrier();
        };
        arrived(first);
        arrived(set_b);
        if (odd) step(first, a.t_end - 1);
        for (int t = a.t_end - 1 - odd; t >= a.t_begin; t -= 2) {
            fetch(set_a, t - 3);
            __builtin_amdgcn_sched_barrier(0);
            step(set_b, t);
            fetch(set_b, t - 4);
            __builtin_amdgcn_sched_barrier(0);
            step(set_a, t - 1);
        }
        store_left(a.t_begin);
        store_pre(a.t_begin + 1, 3);
        lds_barrier();
        store_pre(a.t_begin, 2);
    }
}

// ------------------------------------------------------------------------------------------ weight gradients
struct TnGemmArgs {
    RowMap a, b;
    int M;              // samples
    int P, Q;           // columns of A and of B taken
    int extra_mode;     // columns appended to B: kExtraOnes (one column of ones), kExtraAgent (N one-hot columns of m % N)
    int n_extra, N;
    int qp;             // Q + n_extra rounded up to 16: row pitch of the result
    int pp;             // rows of a partial result (partial_rows)
    int chunk;          // samples per workgroup along the contraction, a multiple of 32
    // elements from a row to the next: inside a group, and from a group's last row to the next group's first
    // (A's rows are one group: the adjoint arrays are)
    unsigned next_a, next_b, wrap_b;
    unsigned wrap_a;    // tn_gemm_wide_kernel only: A in groups too
    float *partial;     // [chunks][pp][qp]
};

constexpr int kTnThreads = 512;        // eight waves: two per SIMD
constexpr int kTnBatchMax = kProductsPerLaunch;        // products of one shape launched together (blockIdx.y picks one)
struct TnGemmBatch { TnGemmArgs g[kTnBatchMax]; };

// One workgroup per chunk of samples computes the whole result, so that every operand element is read from
// memory once.  Wave w owns result row blocks w, w + 8, .. (PBW of them at most) and all column blocks (QBN at most).  Shapes
// (launch_shape): what is staged is sized by PBW and QBN, so the products of 64 hidden units, 192 x 65 and 64 x (D + N), have
// their own; in those of 128 units, 384 x 144 and 128 x 336, half of what they staged and multiplied was padding.  P: bf16
// planes per operand, the network's own: 2 = every value as bf16 high part + bf16 of the remainder, three MFMAs
// per product; 1 = values rounded to bf16, one MFMA.
// ABF: A's elements are bf16 (the adjoints of a bf16 network), else fp32.  BBF: the same for B's (its saved x).
template <int PBW, int QBN, int P, bool ABF, bool BBF = false>
__global__ __launch_bounds__(kTnThreads, 2) void tn_gemm_kernel(const TnGemmBatch batch)
{
    const TnGemmArgs g = batch.g[blockIdx.y];
    constexpr int kPp = 16 * 8 * PBW;                              // result rows, padded = columns of A staged
    constexpr int kSets = (kPp + 16 * QBN + 63) / 64;              // sets of 64 staged columns (A's, then B's)
    constexpr int kSetsPerWave = (kSets + 1) / 2;
    constexpr bool kTwoBuffers = P == 1;                           // a second staging buffer where it fits
    constexpr int kPitch = 80;                                     // bytes per column: 64 + 16 against bank conflicts
    // LDS: P planes (bf16 high part, bf16 of the remainder), each column-major: column c of the staged 32
    // samples is 64 bytes, the lane's eight samples of a fragment 16.
    extern __shared__ __attribute__((aligned(16))) char stage[];
    const int cols = kPp + g.qp;
    const int plane_bytes = cols * kPitch;
    const int lane = threadIdx.x & 63, q4 = lane >> 4, c = lane & 15;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int sg = w & 3, half = w >> 2;                           // the wave stages samples 8 sg + 0..7 of every other column set
    const int n_qb = g.qp / 16;
    [[maybe_unused]] const bool last_block = 16 * (w + 8 * (PBW - 1)) < g.P;        // whether the wave's last row block exists
    const int m_begin = (int)blockIdx.x * g.chunk, m_end = min(g.M, m_begin + g.chunk);     // M < 2^30
    // The 32 samples of a step are eight consecutive ones from each quarter of the chunk: wave group sg walks
    // through its own quarter, so that the rows it reads follow one another from the first step to the last and
    // their addresses are stepped, never recomputed.
    const int n_steps = (m_end - m_begin + 31) / 32;
    const int wave_begin = m_begin + 8 * n_steps * sg, wave_end = min(m_end, wave_begin + 8 * n_steps);

    f32x4 acc[PBW][QBN];
#pragma unroll
    for (int k = 0; k < PBW; ++k)
#pragma unroll
        for (int j = 0; j < QBN; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[k][j][r] = 0.0f;

    // Inputs are asked for kDepth steps before they are used, into kDepth register sets that the unrolled
    // loop addresses statically.  Every load is unconditional (rows past the end of the arrays repeat the last
    // row, columns past an operand's width repeat its first), so the loop is straight-line code.
    constexpr int kDepth = 2;
    // bf16 adjoints (ABF) are not fetched column by column like the rest: a thread takes 16 bytes, eight columns
    // of one sample, and the tile goes to LDS as it lies in memory, sample-major; the transposition into
    // fragments (eight samples of one column per lane) is left to the transposing LDS read.  kAVec such loads
    // per thread cover the step's 32 samples of kPp columns.
    constexpr int kAVec = ABF ? 32 * kPp * 2 / 16 / kTnThreads : 0;
    constexpr int kAChunks = kPp / 8;                              // 16-byte pieces of a staged row of A
    constexpr int kAPitch = kPp * 2 + 32;                          // bytes from a sample's row to the next in LDS
    static_assert(!ABF || (32 * kPp * 2) % (16 * kTnThreads) == 0, "whole loads per thread");
    static_assert(32 * kAPitch <= kPp * kPitch, "the sample-major tile fits where A's columns would lie");
    struct Staged { float col[kSetsPerWave][8]; uint4 a[kAVec > 0 ? kAVec : 1]; };
    Staged rv[kDepth];
    // kPp is a multiple of 128, so set i of either half of the waves is one of A's exactly for i < kPp / 128:
    // known at compile time, and with it the element type, so that a load is one instruction with no branch
    constexpr int kSetsOfA = kPp / 128;
    static_assert(kPp % 128 == 0, "the column sets of A split evenly between the two halves of the waves");
    // Per column set of this wave: the lane's (clamped) column in its operand's rows, and for B's sets what the lane's
    // column is made of: -2 a column of B itself (or one past everything, whose results nobody reads), -1 the
    // appended column of ones, n >= 0 the appended one-hot column of agent n.
    int set_col[kSetsPerWave], made_of[kSetsPerWave];
#pragma unroll
    for (int i = 0; i < kSetsPerWave; ++i) {
        const int col = lane + 64 * (2 * i + half), cb = col - kPp;
        set_col[i] = i < kSetsOfA ? (col < g.P ? col : 0) : (cb < g.Q ? cb : 0);
        made_of[i] = (i >= kSetsOfA && cb >= g.Q && cb < g.Q + g.n_extra) ? (g.extra_mode == kExtraOnes ? -1 : cb - g.Q) : -2;
    }
    // A column past an operand's width is staged with the values of the operand's first column: it only reaches
    // rows or columns of the result that the reduction never reads, and costs no instruction here.

    // The row the next load takes, as addresses in A and B; (group, row in group) by division once, then by
    // stepping: a row further in the group, or from a group's last row to the next group's first.  All of it
    // is the same in every lane and is kept in scalar registers (said so where the compiler cannot tell).
    const unsigned row0 = (unsigned)min(wave_begin, g.M - 1);
    const unsigned gb0 = __builtin_amdgcn_readfirstlane(row0 / (unsigned)g.b.rows_per_group);
    const unsigned ib0 = row0 - gb0 * (unsigned)g.b.rows_per_group;
    long off_a = (long)row0 * g.a.ld;                                        // in elements; A's rows follow one another
    long off_b = (long)gb0 * g.b.group_stride + (long)ib0 * g.b.ld;
    unsigned b_left = (unsigned)g.b.rows_per_group - ib0;            // rows to the end of B's group
    unsigned rows_left = (unsigned)(g.M - 1) - row0;                  // steps that stay inside the arrays
    int sample = wave_begin;                                          // first sample of the step being staged
    unsigned agent0 = (unsigned)wave_begin % (unsigned)g.N;          // its agent, where rows are (.., agent) samples
    const unsigned agent_step = 8u % (unsigned)g.N;
    // wide loads of A: load i of this thread is piece a_piece of row a_k (sample 8 (a_k / 8) + a_k % 8 of the step:
    // the a_k % 8-th of quarter a_k / 8), at a_at bytes from A's base; every step moves eight rows on
    // (a_fetch: the sample the next load takes, a_staged: the one the next deposit puts down, a_end: the end of
    // the quarter's share)
    long a_at[kAVec > 0 ? kAVec : 1];
    int a_fetch[kAVec > 0 ? kAVec : 1], a_staged[kAVec > 0 ? kAVec : 1], a_end[kAVec > 0 ? kAVec : 1], a_lds[kAVec > 0 ? kAVec : 1];
    if constexpr (ABF) {
#pragma unroll
        for (int i = 0; i < kAVec; ++i) {
            const int v = (int)threadIdx.x + kTnThreads * i, k = v / kAChunks, piece = v % kAChunks;
            const int quarter_begin = m_begin + 8 * n_steps * (k >> 3);
            a_fetch[i] = a_staged[i] = quarter_begin + (k & 7);
            a_end[i] = min(m_end, quarter_begin + 8 * n_steps);
            a_at[i] = ((long)min(a_fetch[i], g.M - 1) * g.a.ld + (8 * piece < g.P ? 8 * piece : 0)) * 2;
            a_lds[i] = k * kAPitch + 16 * piece;
        }
    }

    // The loop comes twice.  ENDS = false: every row the workgroup touches, those fetched ahead included, exists
    // and every sample of every step counts - all chunks but the last one or two.  ENDS = true: past the last
    // sample the last row is fetched again (and not used), and samples past the wave's share are cleared (A's
    // values are; B's may stay).
    auto run = [&](auto ends_tag) {
        constexpr bool ENDS = decltype(ends_tag)::value;
        auto fetch = [&](Staged &into) {                             // this wave's next eight rows
            float (&f)[kSetsPerWave][8] = into.col;
            if constexpr (ABF) {
#pragma unroll
                for (int i = 0; i < kAVec; ++i) {
                    into.a[i] = *reinterpret_cast<const uint4 *>(static_cast<const char *>(g.a.base) + a_at[i]);
                    // eight rows on, or (ENDS) stay where the arrays end: what is fetched there again is not used
                    long step_bytes = (long)8 * g.next_a * 2;
                    if constexpr (ENDS) step_bytes = a_fetch[i] + 8 < g.M ? step_bytes : 0;
                    a_at[i] += step_bytes;
                    a_fetch[i] += 8;
                }
            }
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const char *arow = static_cast<const char *>(g.a.base) + off_a * (ABF ? 2 : 4);
                const char *brow = static_cast<const char *>(g.b.base) + off_b * (BBF ? 2 : 4);
#pragma unroll
                for (int i = ABF ? kSetsOfA : 0; i < kSetsPerWave; ++i) {
                    if constexpr (BBF) {
                        if (i >= kSetsOfA) {
                            f[i][r] = __uint_as_float((uint32_t)reinterpret_cast<const uint16_t *>(brow)[set_col[i]]);
                            continue;
                        }
                    }
                    f[i][r] = i < kSetsOfA ? reinterpret_cast<const float *>(arow)[set_col[i]] : reinterpret_cast<const float *>(brow)[set_col[i]];
                }
                // the next row, without a branch (a branch between two loads would make every wait a full one)
                unsigned go = 1u;
                if constexpr (ENDS) { go = rows_left ? 1u : 0u; rows_left -= go; }
                b_left -= go;
                const bool wb = b_left == 0u;
                unsigned sa = g.next_a, sb = wb ? g.wrap_b : g.next_b;      // A's rows are one group (the launcher checks)
                if constexpr (ENDS) { sa = go ? sa : 0u; sb = go ? sb : 0u; }
                off_a += sa; off_b += sb;
                asm volatile("" : "+s"(off_a));      // kept as one running scalar, not turned into a vector address per row
                b_left = wb ? (unsigned)g.b.rows_per_group : b_left;
            }
        };
        // The wave's eight samples of a column are samples 8 sg + 0..7 of the step: as bf16 they are exactly the
        // 16 bytes that lane quarter sg of a fragment of that column reads.  Converted once here, not by every
        // reader.  A loaded value is first passed through an empty asm: that is where the wait for it goes, and
        // it keeps the compiler from turning "loaded value or zero" into a branch around the load.
        auto deposit = [&](char *buf, Staged &from) {
            float (&f)[kSetsPerWave][8] = from.col;
            if constexpr (ABF) {
#pragma unroll
                for (int i = 0; i < kAVec; ++i) {
                    uint4 v = from.a[i];
                    asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w));
                    if constexpr (ENDS) {
                        const uint32_t keep = a_staged[i] < a_end[i] ? 0xFFFFFFFFu : 0u;
                        v.x &= keep; v.y &= keep; v.z &= keep; v.w &= keep;
                    }
                    *reinterpret_cast<uint4 *>(buf + a_lds[i]) = v;
                    a_staged[i] += 8;
                }
            }
#pragma unroll
            for (int i = ABF ? kSetsOfA : 0; i < kSetsPerWave; ++i) {
                const int col = lane + 64 * (2 * i + half);
                if constexpr (BBF) {
                    if (i >= kSetsOfA) {      // bf16 values of B, or the bf16 of an appended column's 1 or 0
                        uint32_t word[4];
                        unsigned agent = agent0;
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            asm volatile("" : "+v"(f[i][2 * j]), "+v"(f[i][2 * j + 1]));
                            uint32_t e[2];
#pragma unroll
                            for (int k = 0; k < 2; ++k) {
                                const int which = g.extra_mode == kExtraOnes ? -1 : (int)agent;
                                e[k] = made_of[i] == which ? 0x3F80u : (made_of[i] == -2 ? __float_as_uint(f[i][2 * j + k]) : 0u);
                                agent = agent + 1 == (unsigned)g.N ? 0u : agent + 1;
                            }
                            word[j] = e[0] | (e[1] << 16);
                        }
                        if (col < cols) *reinterpret_cast<uint4 *>(buf + col * kPitch + 16 * sg) = make_uint4(word[0], word[1], word[2], word[3]);
                        continue;
                    }
                }
                float v[8];
                unsigned agent = agent0;
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    asm volatile("" : "+v"(f[i][r]));
                    if (i < kSetsOfA) {
                        v[r] = (!ENDS || sample + r < wave_end) ? f[i][r] : 0.0f;
                    } else {
                        const int which = g.extra_mode == kExtraOnes ? -1 : (int)agent;
                        v[r] = made_of[i] == which ? 1.0f : (made_of[i] == -2 ? f[i][r] : 0.0f);
                        agent = agent + 1 == (unsigned)g.N ? 0u : agent + 1;
                    }
                }
                if (col < cols) {
                    const Frag<P> fr = to_frag<P>(v);
                    *reinterpret_cast<bf16x8 *>(buf + col * kPitch + 16 * sg) = fr.hi;
                    if constexpr (P == 2) *reinterpret_cast<bf16x8 *>(buf + plane_bytes + col * kPitch + 16 * sg) = fr.lo;
                }
            }
            sample += 8;
            agent0 += agent_step;
            agent0 = agent0 >= (unsigned)g.N ? agent0 - (unsigned)g.N : agent0;
        };

#pragma unroll
        for (int d = 0; d < kDepth; ++d) fetch(rv[d]);
        // fragments: lane (c, q4) takes samples 8 q4 + 0..7 of column 16 block + c
        auto multiply = [&](const char *buf) {
            const char *mine = buf + c * kPitch + 16 * q4;
            WFrag<P> af[PBW];
#pragma unroll
            for (int k = 0; k < PBW; ++k) {
                if constexpr (ABF) {
                    // The transposing read works on blocks of 16 lanes: lane 4 a + e of a block receives, as its
                    // i-th value, element e of the four that lane a + 4 i of the block points at.  With lane a + 4 i
                    // pointing at sample 8 q4 + i, columns 4 a .. 4 a + 3, lane c gets column c of samples
                    // 8 q4 + 0..3; the second read gives samples 8 q4 + 4..7.
                    typedef short s16x4 __attribute__((ext_vector_type(4)));
                    typedef s16x4 __attribute__((address_space(3))) *LdsQuad;
                    const char *at = buf + (8 * q4 + (c >> 2)) * kAPitch + (16 * (w + 8 * k) + 4 * (c & 3)) * 2;
                    const s16x4 first = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsQuad)(at));
                    const s16x4 second = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsQuad)(at + 4 * kAPitch));
                    typedef short s16x8 __attribute__((ext_vector_type(8)));
                    const s16x8 both = __builtin_shufflevector(first, second, 0, 1, 2, 3, 4, 5, 6, 7);
                    af[k].hi = __builtin_bit_cast(bf16x8, both);
                } else {
                    af[k].hi = *reinterpret_cast<const bf16x8 *>(mine + 16 * (w + 8 * k) * kPitch);
                    if constexpr (P == 2) af[k].lo = *reinterpret_cast<const bf16x8 *>(mine + plane_bytes + 16 * (w + 8 * k) * kPitch);
                }
            }
            // (PBW == 2: the first of a wave's row blocks exists, as P is more than 128, the second may not)
            auto product = [&](auto row_blocks) {
#pragma unroll
                for (int j = 0; j < QBN; ++j)
                    if (j < n_qb) {
                        Frag<P> bf;
                        bf.hi = *reinterpret_cast<const bf16x8 *>(mine + (kPp + 16 * j) * kPitch);
                        if constexpr (P == 2) bf.lo = *reinterpret_cast<const bf16x8 *>(mine + plane_bytes + (kPp + 16 * j) * kPitch);
#pragma unroll
                        for (int k = 0; k < decltype(row_blocks)::value; ++k) mma16<P>(acc[k][j], af[k], bf);
                    }
            };
            if constexpr (PBW == 2) {          // (with three row blocks a wave, the accumulators of two ways through spill)
                if (last_block) product(std::integral_constant<int, PBW>{});
                else product(std::integral_constant<int, PBW - 1>{});
            } else {
                product(std::integral_constant<int, PBW>{});
            }
        };
        // Rounds of kDepth steps; steps past the end of the chunk add zeros.  The compiler's wait at the head of
        // the loop is for everything asked for so far, whatever the order of the round.  Where two staging
        // buffers fit, the round is therefore: stage both steps, ask for the next two, multiply both - every
        // load has both multiplications to arrive in.
        for (int s0 = 0; s0 < n_steps; s0 += kDepth) {
            if constexpr (kTwoBuffers) {
                static_assert(kDepth == 2, "one staging buffer per step of a round");
                char *second = stage + P * plane_bytes;
                deposit(stage, rv[0]);
                deposit(second, rv[1]);
                fetch(rv[0]);
                fetch(rv[1]);
                __syncthreads();
                multiply(stage);
                multiply(second);
                __syncthreads();               // every wave is done reading before the next round writes
            } else {
#pragma unroll
                for (int d = 0; d < kDepth; ++d) {
                    __syncthreads();           // one buffer: the previous step has been read by every wave
                    deposit(stage, rv[d]);
                    fetch(rv[d]);              // asked for before the barrier, so that the wait at it is not idle time for memory
                    __syncthreads();
                    multiply(stage);
                }
            }
        }
    };
    // Rows touched: the last quarter's, plus what is fetched ahead of the last step (the loop runs whole rounds).
    const int rounds_end = (n_steps + kDepth - 1) / kDepth * kDepth;
    const bool all_inside = m_begin + 8 * (3 * n_steps + rounds_end + kDepth) <= g.M
                            && rounds_end == n_steps && m_end - m_begin == 32 * n_steps;
    // (two planes: the one general loop only - twice over, the loop did not fit the registers)
    if (P == 1 && all_inside) run(std::integral_constant<bool, P != 1>{});
    else run(std::true_type{});

    // C layout: lane (c, q4) holds result[16 block + 4 q4 + r][16 j + c]
    float *out = g.partial + (size_t)blockIdx.x * g.pp * g.qp;
#pragma unroll
    for (int k = 0; k < PBW; ++k)
#pragma unroll
        for (int j = 0; j < QBN; ++j)
            if (j < n_qb && (PBW == 3 || 16 * (w + 8 * k) < g.P))
#pragma unroll
                for (int r = 0; r < 4; ++r) out[(size_t)(16 * (w + 8 * k) + 4 * q4 + r) * g.qp + 16 * j + c] = acc[k][j][r];
}

// The same product for a bf16 network whose operands allow it (tn_wide_fits): neither operand is fetched
// column by column.  A thread takes 16 bytes of a sample's row (eight bf16 or four fp32 columns), the step's 32
// samples go to LDS as they lie in memory, sample-major and as bf16, and the transposition into fragments
// (eight samples of one column per lane) is left to the transposing LDS read: a tenth of the load
// instructions.  Chunks, the order of samples within a step (eight consecutive ones from each quarter of the
// chunk), the made-up columns and the partial results are those of tn_gemm_kernel.
template <int PBW, int QBN, bool BBF>
__global__ __launch_bounds__(kTnThreads, 2) void tn_gemm_wide_kernel(const TnGemmBatch batch)
{
    const TnGemmArgs g = batch.g[blockIdx.y];
    constexpr int kPp = 16 * 8 * PBW;                              // result rows, padded = columns of A staged
    constexpr int kQp = 16 * QBN;                                  // most columns of B staged
    constexpr int kColsB = BBF ? 8 : 4;                            // columns of B in 16 bytes
    static_assert(kPp / 8 % 16 == 0, "whole loads of A per thread");
    // bytes from a sample's row to the next in LDS: 48 past a multiple of 256, so that the four rows a block of
    // 16 lanes reads together, 32 bytes of each, lie in different banks
    constexpr int kAPitch = kPp * 2 + 48, kBPitch = (kQp * 2 + 255) / 256 * 256 + 48;
    constexpr int kBufBytes = 32 * (kAPitch + kBPitch);
    extern __shared__ __attribute__((aligned(16))) char stage[];
    const int lane = threadIdx.x & 63, q4 = lane >> 4, c = lane & 15;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n_qb = g.qp / 16;
    const int m_begin = (int)blockIdx.x * g.chunk, m_end = min(g.M, m_begin + g.chunk);     // M < 2^30
    const int n_steps = (m_end - m_begin + 31) / 32;

    // Which blocks of the result a wave owns.  Three row blocks (w, w + 8, w + 16) and every column block where the
    // result is tall: a fragment of B then feeds three products.  Where it is 128 rows, all eight row blocks and every
    // eighth column block (w, w + 8) of up to 176 columns; of up to 336 columns, half the row blocks and every fourth column
    // block: 10 fragments per step for 24 products, and 16 registers less of them than with all row blocks and every eighth
    // column block, which spilled 25 (this one spills one).
    constexpr bool kSplitColumns = PBW == 1, kHalves = kSplitColumns && QBN > 16;
    constexpr int kRB = kHalves ? 4 : kSplitColumns ? 8 : PBW, kCB = kHalves ? (QBN + 3) / 4 : kSplitColumns ? (QBN + 7) / 8 : QBN;
    auto row_block = [&](int k) { return kHalves ? 4 * (w >> 2) + k : kSplitColumns ? k : w + 8 * k; };
    auto col_block = [&](int j) { return kHalves ? (w & 3) + 4 * j : kSplitColumns ? w + 8 * j : j; };
    // (the accumulators of the larger shapes leave no room for two ways through)
    constexpr bool kMayBeShort = PBW == 2 || (kSplitColumns && !kHalves);
    [[maybe_unused]] const bool all_blocks = kSplitColumns ? g.P > 64 : 16 * (w + 8 * (PBW - 1)) < g.P;
    f32x4 acc[kRB][kCB];
#pragma unroll
    for (int k = 0; k < kRB; ++k)
#pragma unroll
        for (int j = 0; j < kCB; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[k][j][r] = 0.0f;

    // A thread's loads all take pieces of one row: thread (quarter t / 128, row (t % 128) / 16, first piece t % 16)
    // fetches pieces first + 16 i of row 8 quarter + row of the step, i.e. of that quarter's next sample but
    // `row`, so that one address, one sample number and one end serve them all.  Pieces past the operand's
    // width repeat the first one (their results are rows or columns nobody reads, or they are made up below).
    constexpr int kALoads = kPp / 8 / 16;                          // per thread and step: of A,
    constexpr int kBLoads = (kQp / kColsB + 15) / 16;              // of B
    const int quarter = (int)threadIdx.x >> 7, row_in_quarter = ((int)threadIdx.x & 127) >> 4, first_piece = (int)threadIdx.x & 15;
    const int k_row = 8 * quarter + row_in_quarter;
    const int pieces_b = g.qp / kColsB;
    int sample_next = m_begin + 8 * n_steps * quarter + row_in_quarter;      // the sample the next loads take
    const int share_end = min(m_end, m_begin + 8 * n_steps * (quarter + 1));  // end of the quarter's share of the chunk
    const char *a_row, *b_row;                                     // the next loads' rows
    unsigned a_left, b_left;                                       // rows from the next load's to the end of its group
    unsigned agent;                                                // of the sample being staged next
    {
        const unsigned row = (unsigned)min(sample_next, g.M - 1);
        const unsigned group = row / (unsigned)g.b.rows_per_group, in_group = row - group * (unsigned)g.b.rows_per_group;
        const unsigned group_a = row / (unsigned)g.a.rows_per_group, in_group_a = row - group_a * (unsigned)g.a.rows_per_group;
        a_row = static_cast<const char *>(g.a.base) + ((long)group_a * g.a.group_stride + (long)in_group_a * g.a.ld) * 2;
        b_row = static_cast<const char *>(g.b.base) + ((long)group * g.b.group_stride + (long)in_group * g.b.ld) * (BBF ? 2 : 4);
        a_left = (unsigned)g.a.rows_per_group - in_group_a;
        b_left = (unsigned)g.b.rows_per_group - in_group;
        agent = (unsigned)sample_next % (unsigned)g.N;
    }
    const unsigned agent_step = 8u % (unsigned)g.N;
    int a_piece[kALoads], b_piece[kBLoads];                        // byte offsets within the row
#pragma unroll
    for (int i = 0; i < kALoads; ++i) a_piece[i] = 8 * (first_piece + 16 * i) < g.P ? 16 * (first_piece + 16 * i) : 0;
#pragma unroll
    for (int i = 0; i < kBLoads; ++i) b_piece[i] = kColsB * (first_piece + 16 * i) < g.Q ? 16 * (first_piece + 16 * i) : 0;
    const int a_lds = k_row * kAPitch + 16 * first_piece;          // + 256 i
    const int b_lds = 32 * kAPitch + k_row * kBPitch + 2 * kColsB * first_piece;      // + 32 kColsB i
    const int b_spare = 32 * kAPitch + k_row * kBPitch + (kBPitch - 48);             // 48 bytes that no fragment reads

    constexpr int kDepth = 2;
    struct Staged { uint4 a[kALoads], b[kBLoads]; };
    Staged rv[kDepth];
    int staged_sample = sample_next;                               // the sample the next deposit puts down

    auto run = [&](auto ends_tag) {
        constexpr bool ENDS = decltype(ends_tag)::value;           // the chunk reaches the end of the samples
        auto fetch = [&](Staged &into) {
#pragma unroll
            for (int i = 0; i < kALoads; ++i) into.a[i] = *reinterpret_cast<const uint4 *>(a_row + a_piece[i]);
#pragma unroll
            for (int i = 0; i < kBLoads; ++i) into.b[i] = *reinterpret_cast<const uint4 *>(b_row + b_piece[i]);
            // eight rows on: inside the group, or seven steps inside and one from a group's last row to the
            // next group's first.  (ENDS) Past the arrays' end the rows stay: what is fetched there again is not used.
            bool go = true;
            if constexpr (ENDS) go = sample_next + 8 < g.M;
            const bool wraps = b_left <= 8u, wraps_a = a_left <= 8u;
            const long b_step = (wraps ? (long)7 * g.next_b + g.wrap_b : (long)8 * g.next_b) * (BBF ? 2 : 4);
            const long a_step = (wraps_a ? (long)7 * g.next_a + g.wrap_a : (long)8 * g.next_a) * 2;
            a_row += go ? a_step : 0;
            b_row += go ? b_step : 0;
            a_left = go ? (wraps_a ? a_left + (unsigned)g.a.rows_per_group - 8u : a_left - 8u) : a_left;
            b_left = go ? (wraps ? b_left + (unsigned)g.b.rows_per_group - 8u : b_left - 8u) : b_left;
            sample_next += 8;
        };
        auto deposit = [&](char *buf, Staged &from) {
            uint32_t keep = 0xFFFFFFFFu;       // samples past the chunk's end count for nothing: A's values are cleared, B's may stay
            if constexpr (ENDS) keep = staged_sample < share_end ? 0xFFFFFFFFu : 0u;
            // where the sample's row of appended columns has its 1: the column of ones, its agent's column, or nowhere
            const int one_at = g.extra_mode == kExtraAgent ? g.Q + (int)agent : g.extra_mode == kExtraOnes ? g.Q : -8;
#pragma unroll
            for (int i = 0; i < kALoads; ++i) {
                uint4 v = from.a[i];
                asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w));
                if constexpr (ENDS) { v.x &= keep; v.y &= keep; v.z &= keep; v.w &= keep; }
                *reinterpret_cast<uint4 *>(buf + a_lds + 256 * i) = v;
            }
#pragma unroll
            for (int i = 0; i < kBLoads; ++i) {
                uint4 v = from.b[i];
                asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w));
                const int piece = first_piece + 16 * i, col = kColsB * piece;
                // a piece past B's own columns is made up: the column of ones, or the one-hot columns of the sample's agent
                const bool made_up = col >= g.Q;
                // (the one 1 of its columns, if it has it: `one` columns on from the piece's first)
                const int one = one_at - col;
                const uint64_t bf16_one = 0x3F80ull << (16 * (one & 3));
                const uint64_t low = (unsigned)one < 4u ? bf16_one : 0, high = kColsB == 8 && (unsigned)(one - 4) < 4u ? bf16_one : 0;
                // a spare load (a piece past the staged columns) goes to the padding at the end of the row
                const int at = piece < pieces_b ? b_lds + 32 * kColsB * i : b_spare;
                if constexpr (BBF) {
                    const uint4 out = made_up && piece < pieces_b ? make_uint4((uint32_t)low, (uint32_t)(low >> 32), (uint32_t)high, (uint32_t)(high >> 32)) : v;
                    *reinterpret_cast<uint4 *>(buf + at) = out;
                } else {
                    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
                    bf16x4 r;
                    r[0] = (__bf16)__uint_as_float(v.x); r[1] = (__bf16)__uint_as_float(v.y);
                    r[2] = (__bf16)__uint_as_float(v.z); r[3] = (__bf16)__uint_as_float(v.w);
                    const uint2 real = __builtin_bit_cast(uint2, r);
                    const uint2 out = made_up && piece < pieces_b ? make_uint2((uint32_t)low, (uint32_t)(low >> 32)) : real;
                    *reinterpret_cast<uint2 *>(buf + at) = out;
                }
            }
            staged_sample += 8;
            agent += agent_step;
            agent = agent >= (unsigned)g.N ? agent - (unsigned)g.N : agent;
        };
        // The transposing read works on blocks of 16 lanes: lane 4 a + e of a block receives, as its i-th value,
        // element e of the four that lane a + 4 i of the block points at.  With lane a + 4 i pointing at sample
        // 8 q4 + i, columns 4 a .. 4 a + 3 of a block of 16 columns, lane c gets column c of samples 8 q4 + 0..3;
        // a second read four rows on gives samples 8 q4 + 4..7: the fragment of lane (c, q4).
        auto fragment = [&](const char *rows, int pitch, int first_col) {
            typedef short s16x4 __attribute__((ext_vector_type(4)));
            typedef short s16x8 __attribute__((ext_vector_type(8)));
            typedef s16x4 __attribute__((address_space(3))) *LdsQuad;
            const char *at = rows + (8 * q4 + (c >> 2)) * pitch + (first_col + 4 * (c & 3)) * 2;
            const s16x4 first = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsQuad)(at));
            const s16x4 second = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsQuad)(at + 4 * pitch));
            return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(first, second, 0, 1, 2, 3, 4, 5, 6, 7));
        };
        auto multiply = [&](const char *buf) {
            WFrag<1> af[kRB];
#pragma unroll
            for (int k = 0; k < kRB; ++k) af[k].hi = fragment(buf, kAPitch, 16 * row_block(k));
            if constexpr (kMayBeShort) {
                auto product = [&](auto row_blocks) {
#pragma unroll
                    for (int j = 0; j < kCB; ++j)
                        if (col_block(j) < n_qb) {
                            Frag<1> bf;
                            bf.hi = fragment(buf + 32 * kAPitch, kBPitch, 16 * col_block(j));
#pragma unroll
                            for (int k = 0; k < decltype(row_blocks)::value; ++k) mma16<1>(acc[k][j], af[k], bf);
                        }
                };
                if (all_blocks) product(std::integral_constant<int, kRB>{});
                else product(std::integral_constant<int, kSplitColumns ? kRB / 2 : kRB - 1>{});
            } else {
#pragma unroll
                for (int j = 0; j < kCB; ++j)
                    if (col_block(j) < n_qb) {
                        Frag<1> bf;
                        bf.hi = fragment(buf + 32 * kAPitch, kBPitch, 16 * col_block(j));
#pragma unroll
                        for (int k = 0; k < kRB; ++k) mma16<1>(acc[k][j], af[k], bf);
                    }
            }
        };
#pragma unroll
        for (int d = 0; d < kDepth; ++d) fetch(rv[d]);
        // a round: stage both steps, ask for the next two, multiply both - every load has both multiplications to arrive in
        for (int s0 = 0; s0 < n_steps; s0 += kDepth) {
            deposit(stage, rv[0]);
            deposit(stage + kBufBytes, rv[1]);
            fetch(rv[0]);
            fetch(rv[1]);
            __syncthreads();
            multiply(stage);
            multiply(stage + kBufBytes);
            __syncthreads();                   // every wave is done reading before the next round writes
        }
    };
    // Rows touched: the last quarter's, plus what is fetched ahead of the last step (the loop runs whole rounds).
    const int rounds_end = (n_steps + kDepth - 1) / kDepth * kDepth;
    const bool all_inside = m_begin + 8 * (3 * n_steps + rounds_end + kDepth) <= g.M
                            && rounds_end == n_steps && m_end - m_begin == 32 * n_steps;
    if (all_inside) run(std::false_type{});
    else run(std::true_type{});

    // C layout: lane (c, q4) holds result[16 block + 4 q4 + r][16 j + c]
    float *out = g.partial + (size_t)blockIdx.x * g.pp * g.qp;
#pragma unroll
    for (int k = 0; k < kRB; ++k)
#pragma unroll
        for (int j = 0; j < kCB; ++j)
            if (col_block(j) < n_qb && (PBW == 3 || 16 * row_block(k) < g.P))
#pragma unroll
                for (int r = 0; r < 4; ++r) out[(size_t)(16 * row_block(k) + 4 * q4 + r) * g.qp + 16 * col_block(j) + c] = acc[k][j][r];
}

template <int PBW, int QBN> constexpr size_t tn_wide_lds()
{
    return (size_t)2 * 32 * ((16 * 8 * PBW * 2 + 48) + ((16 * QBN * 2 + 255) / 256 * 256 + 48));
}

// Whether tn_gemm_wide_kernel can take a product: bf16 adjoints, and every row of both operands a whole number
// of 16-byte pieces at 16-byte aligned addresses, B's own columns ending on a piece.
bool tn_wide_fits(const TnProduct &t, long M)
{
    if (!t.a.bf16) return false;
    const int cols_b = t.b.bf16 ? 8 : 4, bytes_b = t.b.bf16 ? 2 : 4;
    if (reinterpret_cast<uintptr_t>(t.a.base) % 16 != 0 || t.a.ld % 8 != 0 || t.a.ld < (t.P + 7) / 8 * 8) return false;
    if (t.a.rows_per_group < M && (t.a.rows_per_group < 8 || (t.a.group_stride * 2) % 16 != 0)) return false;
    if (t.Q == 0) return t.b.ld >= cols_b && t.b.ld % cols_b == 0 && reinterpret_cast<uintptr_t>(t.b.base) % 16 == 0
                         && (t.b.rows_per_group >= M || (t.b.rows_per_group >= 8 && (t.b.group_stride * bytes_b) % 16 == 0));
    if (reinterpret_cast<uintptr_t>(t.b.base) % 16 != 0 || t.b.ld % cols_b != 0 || t.Q % cols_b != 0 || t.b.ld < cols_b) return false;
    if (t.b.rows_per_group < M && (t.b.rows_per_group < 8 || (t.b.group_stride * bytes_b) % 16 != 0)) return false;
    return true;
}

// The products of the two GRU matrices of 128 units, one plane, and the adjoint of fc1's pre-activation, from the stored
// adjoints: W_ih  sum da[n, r, z]^T [x | 1],  W_hh  sum da[r, z, n_h]^T [h_{t-1} | 1],  dpre1 = (x > 0) W_ih^T da[n, r, z].
// Four workgroups share a chunk of samples, each with half the columns of one of the two products, those of W_ih with dpre1's
// units of the same half beside it: the four read the same adjoints at about the same time, on one XCD, so that they come from
// memory once.  All of a product's columns in one workgroup leave no registers for dpre1's weights.
struct GruProductArgs {
    const bf16x8 *wihT;
    const char *da, *x, *h;        // rows of the window's first sample: adjoints [4 H] bf16, x [H] bf16, h_{t-1} [H] fp32
    char *dpre1;                   // its row of [H] bf16
    uint32_t dpre1_bytes;          // from there to the array's end
    float *partial[2];             // [chunks][384][144] of W_ih, W_hh
    int M, chunk, chunks;          // samples, samples of a chunk (a multiple of 64)
    // A window's samples come in groups, the rows of an episode; `adj` and `act` rows from a group's first to the next one's.
    uint32_t group, adj_group, act_group;
    // 32 rows on: whole groups and rows of one
    uint32_t step_rows, adj_step, act_step;
};

constexpr int kGruRows = 384, kGruColumns = 144;                   // of a partial result
constexpr int kGruShare = 4;                                       // workgroups of a chunk

struct GruTile {
    static constexpr int H = 128, KS = H / 32;
    static constexpr int kAPitch = 3 * H * 2 + 48;                 // 12 words past a multiple of 64: as in tn_gemm_wide_kernel
    static constexpr int kBPitch = 64 * 2 + 16;                    // four rows' 32 bytes in different banks here too
    static constexpr int oB = 32 * kAPitch, kBufBytes = oB + 32 * kBPitch;
    static constexpr int oDp = 2 * kBufBytes, kDpPitch = 64 * 2 + 16, kDpBytes = 32 * kDpPitch;
    static constexpr int kBytes = oDp + 2 * kDpBytes;
};

// WIH: the W_ih product and dpre1; else the W_hh product.
template <bool WIH>
__device__ __forceinline__ void gru_products(const GruProductArgs &g, int chunk_index, int half, char *lds)
{
    using Tl = GruTile;
    constexpr int H = Tl::H, KS = Tl::KS;
    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
    const int lane = threadIdx.x & 63, q4 = lane >> 4, c = lane & 15;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m_begin = chunk_index * g.chunk, m_end = min(g.M, m_begin + g.chunk);
    const int n_steps = (m_end - m_begin + 31) / 32;

    // Thread (row of the step, piece): three times 16 bytes of the sample's adjoints, four columns of x or h.
    const int k_row = (int)threadIdx.x >> 4, piece = (int)threadIdx.x & 15;
    int sample = m_begin + k_row;                                  // the sample the next loads take
    uint32_t in_group, adj_row, act_row;                           // where its rows are
    {
        const uint32_t first = (uint32_t)min(sample, g.M - 1), group = first / g.group;
        in_group = first - group * g.group;
        adj_row = group * g.adj_group + in_group;
        act_row = group * g.act_group + in_group;
    }
    const char *const da = g.da + (WIH ? 0 : 2 * H);               // columns n, r, z or r, z, n of the hidden side
    const char *const act = WIH ? g.x + 128 * half : g.h + 256 * half;
    const uint32_t dp_column = 128u * half + 8u * piece;
    const __amdgpu_buffer_rsrc_t dp_buf = __builtin_amdgcn_make_buffer_rsrc(g.dpre1, 0, WIH ? (int)g.dpre1_bytes : 0, kRawBuffer);

    typedef std::conditional_t<WIH, uint2, uint4> BRegs;
    struct Staged { uint4 a[3]; BRegs b; uint32_t dp_at; };        // dp_at: where the sample's dpre1 goes, kDrop past the chunk's end
    auto fetch = [&](Staged &into) {
        into.dp_at = sample < m_end ? adj_row * (2u * H) + dp_column : kDrop;
        const uint32_t a_at = adj_row * (8u * H) + 16u * piece, b_at = act_row * ((WIH ? 2u : 4u) * H) + (WIH ? 8u : 16u) * piece;
#pragma unroll
        for (int i = 0; i < 3; ++i) into.a[i] = *reinterpret_cast<const uint4 *>(da + 256 * i + a_at);
        into.b = *reinterpret_cast<const BRegs *>(act + b_at);
        // 32 rows on; past the last sample its row stays (what is fetched there again does not count).  Masks: of conditions the
        // compiler makes branches, and a branch between loads makes every wait a full one.
        uint32_t go = sample + 32 < g.M ? 0xFFFFFFFFu : 0u, wraps = in_group + g.step_rows >= g.group ? 0xFFFFFFFFu : 0u;
        asm volatile("" : "+v"(go), "+v"(wraps));
        adj_row += go & (g.adj_step + (wraps & (g.adj_group - g.group)));
        act_row += go & (g.act_step + (wraps & (g.act_group - g.group)));
        in_group += go & (g.step_rows - (wraps & g.group));
        sample += 32;
    };
    const int a_lds = k_row * Tl::kAPitch + 16 * piece, b_lds = Tl::oB + k_row * Tl::kBPitch + 8 * piece;
    // what the thread has to do with dpre1 of the steps staged last: where it goes, which of its four units were on
    uint32_t dp_at[2] = {kDrop, kDrop}, dp_on[2][2] = {};
    auto deposit = [&](int which, Staged &from) {
        char *const buf = lds + which * Tl::kBufBytes;
        const uint32_t keep = from.dp_at != kDrop ? 0xFFFFFFFFu : 0u;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            uint4 v = from.a[i];
            asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w));
            v.x &= keep; v.y &= keep; v.z &= keep; v.w &= keep;
            *reinterpret_cast<uint4 *>(buf + a_lds + 256 * i) = v;
        }
        if constexpr (WIH) {
            uint2 v = from.b;
            asm volatile("" : "+v"(v.x), "+v"(v.y));
            *reinterpret_cast<uint2 *>(buf + b_lds) = v;
            auto on = [](uint32_t two) {
                return (__uint_as_float(two << 16) > 0.0f ? 0xFFFFu : 0u) | (__uint_as_float(two & 0xFFFF0000u) > 0.0f ? 0xFFFF0000u : 0u);
            };
            dp_on[which][0] = on(v.x);
            dp_on[which][1] = on(v.y);
            dp_at[which] = from.dp_at;
        } else {
            uint4 v = from.b;
            asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w));
            bf16x4 r;
            r[0] = (__bf16)__uint_as_float(v.x); r[1] = (__bf16)__uint_as_float(v.y);
            r[2] = (__bf16)__uint_as_float(v.z); r[3] = (__bf16)__uint_as_float(v.w);
            *reinterpret_cast<bf16x4 *>(buf + b_lds) = r;
        }
    };
    auto store_dpre1 = [&]() {                                     // of the two steps multiplied last
#pragma unroll
        for (int which = 0; which < 2; ++which) {
            typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
            uint2 v = *reinterpret_cast<const uint2 *>(lds + Tl::oDp + which * Tl::kDpBytes + k_row * Tl::kDpPitch + 8 * piece);
            const u32x2 out = {v.x & dp_on[which][0], v.y & dp_on[which][1]};
            __builtin_amdgcn_raw_buffer_store_b64(out, dp_buf, dp_at[which], 0, 0);
        }
    };

    // Wave w: row blocks w, w + 8, w + 16 of the result, all four column blocks, and the column of ones (its fragment is the same
    // for every sample: no operand to stage).  dpre1: units of block w % 4 of the half, samples 16 (w / 4) .. + 15 of the step.
    f32x4 acc[3][5] = {};
    WFrag<1> wihT[WIH ? 3 * KS : 1];
    const int dp_block = w & 3, dp_half = w >> 2;
    if constexpr (WIH) {
#pragma unroll
        for (int ks = 0; ks < 3 * KS; ++ks) wihT[ks] = load_wfrag<1>(g.wihT + (size_t)((4 * half + dp_block) * 3 * KS + ks) * 64 + lane);
    }
    Frag<1> ones;
#pragma unroll
    for (int i = 0; i < 8; ++i) ones.hi[i] = (__bf16)(c == 0 ? 1.0f : 0.0f);

    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    typedef s16x4 __attribute__((address_space(3))) *LdsQuad;
    auto fragment = [&](const char *rows, int pitch, int first_col) {      // the transposing read, as in tn_gemm_wide_kernel
        const char *at = rows + (8 * q4 + (c >> 2)) * pitch + (first_col + 4 * (c & 3)) * 2;
        const s16x4 first = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsQuad)(at));
        const s16x4 second = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsQuad)(at + 4 * pitch));
        return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(first, second, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    auto multiply = [&](int which) {
        const char *const buf = lds + which * Tl::kBufBytes;
        WFrag<1> af[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) af[k].hi = fragment(buf, Tl::kAPitch, 16 * (w + 8 * k));
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            Frag<1> bf;
            bf.hi = fragment(buf + Tl::oB, Tl::kBPitch, 16 * j);
#pragma unroll
            for (int k = 0; k < 3; ++k) mma16<1>(acc[k][j], af[k], bf);
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) mma16<1>(acc[k][4], af[k], ones);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (WIH) {
            // the adjoints of a sample are an operand as they lie; the weights' fragments take the gates in the order r, z, n
            const char *const sample_row = buf + (16 * dp_half + c) * Tl::kAPitch + 16 * q4;
            f32x4 dp = {0.0f, 0.0f, 0.0f, 0.0f};
            Frag<1> d[2][KS];                                      // a gate's four k-steps, asked for while the one before is multiplied
            auto request = [&](int gate) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    d[gate % 2][ks].hi = *reinterpret_cast<const bf16x8 *>(sample_row + ((gate + 1) % 3 * KS + ks) * 64);
                }
            };
            request(0);
#pragma unroll
            for (int gate = 0; gate < 3; ++gate) {
                if (gate < 2) request(gate + 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) mma16<1>(dp, wihT[gate * KS + ks], d[gate % 2][ks]);
            }
            bf16x4 r;
#pragma unroll
            for (int i = 0; i < 4; ++i) r[i] = (__bf16)dp[i];
            *reinterpret_cast<bf16x4 *>(lds + Tl::oDp + which * Tl::kDpBytes + (16 * dp_half + c) * Tl::kDpPitch + (16 * dp_block + 4 * q4) * 2) = r;
        }
    };

    // Rounds of two steps: stage both, ask for two more, multiply both.  The loads are two rounds ahead, in four register sets
    // (W_ih: one round, in two; its weights have taken the room).
    constexpr int kAhead = WIH ? 1 : 2;
    Staged set_a, set_b, set_c, set_d;
    for (Staged *set : {&set_a, &set_b, &set_c, &set_d}) {
        if (kAhead == 1 && set == &set_c) break;
        fetch(*set);
        __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (WIH) {
#pragma unroll
        for (int ks = 0; ks < 3 * KS; ++ks) settle(wihT[ks]);
    }
    auto round = [&](Staged &one, Staged &two) {
        if constexpr (WIH) store_dpre1();
        deposit(0, one);
        deposit(1, two);
        __builtin_amdgcn_sched_barrier(0);
        fetch(one);
        __builtin_amdgcn_sched_barrier(0);
        fetch(two);
        __builtin_amdgcn_sched_barrier(0);
        lds_barrier();
        multiply(0);
        __builtin_amdgcn_sched_barrier(0);
        multiply(1);
        lds_barrier();                                             // every wave is done reading before the next round writes
    };
    for (int s = 0; s < n_steps;) {
        round(set_a, set_b);
        s += 2;
        if constexpr (kAhead == 2) {
            if (s >= n_steps) break;
            round(set_c, set_d);
            s += 2;
        }
    }
    if constexpr (WIH) store_dpre1();

    // C layout: lane (c, q4) holds the result's rows at positions 16 block + 4 q4 + r of the stored adjoints, columns 16 j + c.
    // Position 32 s + 8 p + 4 b + r of a gate is its unit 32 s + 16 b + 4 p + r.
    const int unit = 32 * (w >> 1) + 16 * (q4 & 1) + 4 * (2 * (w & 1) + (q4 >> 1));
    float *const out = g.partial[WIH ? 0 : 1] + (size_t)chunk_index * kGruRows * kGruColumns;
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int j = 0; j < 5; ++j)
            if (j < 4 || half == 1)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    out[(size_t)(H * k + unit + r) * kGruColumns + (j < 4 ? 64 * half + 16 * j : H) + c] = acc[k][j][r];
}

__global__ __launch_bounds__(kTnThreads, 2) void gru_products_kernel(const GruProductArgs g)
{
    extern __shared__ __attribute__((aligned(16))) char lds[];
    // Workgroup -> (chunk, share): consecutive workgroups go round the eight XCDs, so the four of a chunk are eight apart.
    const int chunk_index = (int)(blockIdx.x / (8 * kGruShare)) * 8 + (int)(blockIdx.x & 7), share = (int)(blockIdx.x >> 3) & (kGruShare - 1);
    if (chunk_index >= g.chunks) return;
    if (share < 2) gru_products<true>(g, chunk_index, share & 1, lds);
    else gru_products<false>(g, chunk_index, share & 1, lds);
}

// Sum of the chunks, in a fixed order, into the packed gradient vector.  Result row p goes to row
// (p + row_shift) % P of the destination matrix (the adjoint array lists the gates as n, r, z, the
// parameters as r, z, n); columns < Q go to dst_w[row * ld_w + column]; the appended column of ones
// goes to dst_b[row]; appended agent columns continue the row of dst_w (they are W1's id columns).
struct TnReduceArgs {
    const float *partial;
    int chunks, P, p_pad, qp;
    int Q, n_extra, extra_mode;
    int row_shift, w_cols, ld_w;
    float *dst_w, *dst_b;
};
struct TnReduceBatch { TnReduceArgs r[kTnBatchMax]; };

// A result is four running sums over interleaved chunks (j, j + 4, ...), added in a fixed order.
// kWaves = 1: one thread has all four, sixteen loads in flight.  What bounds it where the results are few is the trips to
// memory of that thread, eight for 128 chunks (9.9 us a launch on 64 episodes x 120 slots x 5 agents, 64 units, for 15 MB).
// kWaves = 4: four waves share 64 results, one sum each; iterations there 408 -> 404 us, 37 x 83 x 5 bf16 232 -> 228.
// Four only up to kReduceFew results a launch (one wave per SIMD of the chip): with 147,000 (64 x 200 x 32, 128 units) the
// loads of one thread per result already fill the memory path (iteration 1350 us, with four waves 1352).  The four
// products of 128 units together have more results than that (99,000 and the first layer's), those of 64 units fewer.
constexpr int kReduceThreads = 256;
constexpr long kReduceFew = 65536;

template <int kWaves>
__global__ __launch_bounds__(kReduceThreads) void tn_reduce_kernel(const TnReduceBatch batch)
{
    constexpr int kResults = kReduceThreads / kWaves, kSums = 4 / kWaves;        // results of a workgroup, sums of a thread
    const TnReduceArgs g = batch.r[blockIdx.y];
    const int cols = g.Q + g.n_extra;
    if ((int)blockIdx.x * kResults >= g.P * cols) return;                        // the whole workgroup
    const int part = threadIdx.x / kResults, lane = threadIdx.x % kResults;
    const int at = blockIdx.x * kResults + lane;
    const int idx = min(at, g.P * cols - 1);
    const int p = idx / cols, q = idx % cols;
    const float *src = g.partial + (size_t)p * g.qp + q;
    const size_t step = (size_t)g.p_pad * g.qp;
    float s[kSums] = {};
    int ch = part;
    for (; ch + kWaves * 15 < g.chunks; ch += kWaves * 16) {
        float v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = src[(size_t)(ch + kWaves * i) * step];
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i % kSums] += v[i];
    }
    for (; ch < g.chunks; ch += kWaves * 8) {                                    // the rest, eight at a time
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = src[(size_t)min(ch + kWaves * i, g.chunks - 1) * step];
#pragma unroll
        for (int i = 0; i < 8; ++i) s[i % kSums] += ch + kWaves * i < g.chunks ? v[i] : 0.0f;
    }
    float total;
    if constexpr (kWaves == 4) {
        __shared__ float sums[4][kResults];
        sums[part][lane] = s[0];
        __syncthreads();
        if (part != 0) return;
        total = (sums[0][lane] + sums[1][lane]) + (sums[2][lane] + sums[3][lane]);
    } else {
        total = (s[0] + s[1]) + (s[2] + s[3]);
    }
    if (at >= g.P * cols) return;
    const int row = (p + g.row_shift) % g.P;
    if (q < g.Q || g.extra_mode == kExtraAgent) g.dst_w[(size_t)row * g.ld_w + q] = total;
    else g.dst_b[row] = total;
}

hipError_t launch_reduce(const TnReduceBatch &batch, int count, hipStream_t stream)
{
    long results = 0;
    int most = 0;
    for (int i = 0; i < count; ++i) {
        const int n = batch.r[i].P * (batch.r[i].Q + batch.r[i].n_extra);
        results += n;
        most = std::max(most, n);
    }
    if (results <= kReduceFew)
        hipLaunchKernelGGL(tn_reduce_kernel<4>, dim3((most + kReduceThreads / 4 - 1) / (kReduceThreads / 4), count), dim3(kReduceThreads), 0, stream, batch);
    else
        hipLaunchKernelGGL(tn_reduce_kernel<1>, dim3((most + kReduceThreads - 1) / kReduceThreads, count), dim3(kReduceThreads), 0, stream, batch);
    return hipGetLastError();
}

// kExtraAgent: the bias gradient is the sum of the agent columns just written.
__global__ void bias_from_columns_kernel(const float *w, int rows, int ld, int first, int count, float *dst)
{
    const int row = blockIdx.x * blockDim.x + threadIdx.x;
    if (row >= rows) return;
    float s = 0.0f;
    for (int e = 0; e < count; ++e) s += w[(size_t)row * ld + first + e];
    dst[row] = s;
}

// ------------------------------------------------------------------------------------------ host side
namespace {

size_t align_up(size_t v) { return (v + 255) / 256 * 256; }

// Rows of a product's partial result: P rounded up to 16, or the whole tile of the largest shape.
int partial_rows(int P) { return P > 256 ? 384 : (P + 15) / 16 * 16; }

struct Plan {
    size_t off_h, off_x, off_da, off_dpre1, off_dq, off_carry, off_partial, partial_bytes, bytes;
    int a16;
    GradChunks cut;
};

Plan make_plan(const NetFrags &net, int B, int T)
{
    Plan p{};
    const size_t adj = net.planes == 1 ? 2 : 4;                    // bytes per stored adjoint
    const size_t R = (size_t)B * net.N, S = (size_t)T + 1, H = net.H;
    p.a16 = (net.A + 15) / 16 * 16;
    p.cut = grad_chunks(net.planes, (long)R, T);
    size_t off = 0;
    p.off_h = off;      off = align_up(off + R * S * H * 4);
    p.off_x = off;      off = align_up(off + R * S * H * adj + 4);         // x: bf16 for a one-plane network
    p.off_da = off;     off = align_up(off + R * T * 4 * H * adj + 4);
    p.off_dpre1 = off;  off = align_up(off + R * T * H * adj + 4);
    p.off_dq = off;     off = align_up(off + R * T * p.a16 * adj + 4);
    // room for the partial sums of all four products, whichever way the slots are walked
    auto part = [&](size_t P, size_t Qt) { return (size_t)p.cut.room * partial_rows((int)P) * ((Qt + 15) / 16 * 16) * 4; };
    const size_t need = 2 * part(3 * H, H + 1) + part(H, (size_t)net.D + net.N) + part(net.A, H + 1);
    p.partial_bytes = need;
    p.off_carry = off;  off = align_up(off + (R + 15) / 16 * 16 * H * 4);
    p.off_partial = off; off = align_up(off + need);
    p.bytes = off;
    return p;
}

template <auto kKernel>
hipError_t back_dispatch(const BpttArgs &a, int tile_rows, int threads, size_t lds_bytes, hipStream_t stream)
{
    const int tiles = (a.B * a.net.N + tile_rows - 1) / tile_rows;
    hipError_t err = allow_large_lds<kKernel>(kLdsLimit);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(kKernel, dim3(tiles), dim3(threads), lds_bytes, stream, a);
    return hipGetLastError();
}

}  // namespace

size_t tn_partial_bytes(long M, int chunk, int P, int q_total)
{
    const size_t chunks = (size_t)((M + chunk - 1) / chunk);
    return chunks * (size_t)partial_rows(P) * (size_t)((q_total + 15) / 16 * 16) * sizeof(float);
}

namespace {

// Fills a product's kernel arguments; false where no kernel takes it.
bool tn_args(int planes, const TnProduct &t, long M, int chunk, float *partial, TnGemmArgs *out)
{
    TnGemmArgs g{};
    g.a = t.a; g.b = t.b; g.M = (int)M; g.P = t.P; g.Q = t.Q; g.extra_mode = t.extra_mode; g.n_extra = t.n_extra;
    g.N = t.N > 0 ? t.N : 1;
    g.qp = (t.Q + t.n_extra + 15) / 16 * 16;
    g.pp = partial_rows(t.P);
    g.chunk = chunk;
    g.partial = partial;
    // steps from row to row in elements, 32 bits each; an operand that is one group never takes the second
    auto steps = [&](const RowMap &m, unsigned *next, unsigned *wrap) {
        const long n = (long)m.ld;
        const long w = m.rows_per_group >= M ? n : m.group_stride - (long)(m.rows_per_group - 1) * m.ld;
        if (n < 0 || w < 0 || n >= (1L << 31) || w >= (1L << 31)) return false;
        *next = (unsigned)n; *wrap = (unsigned)w;
        return true;
    };
    if (!steps(t.a, &g.next_a, &g.wrap_a) || !steps(t.b, &g.next_b, &g.wrap_b)) return false;
    *out = g;
    return has_product_kernel(planes, t.a.bf16 != 0, t.b.bf16 != 0, t.P, g.qp);
}

TnReduceArgs reduce_args(const TnProduct &t, const float *partial, int chunks)
{
    TnReduceArgs r{};
    r.partial = partial; r.chunks = chunks; r.P = t.P; r.p_pad = partial_rows(t.P); r.qp = (t.Q + t.n_extra + 15) / 16 * 16;
    r.Q = t.Q; r.n_extra = t.n_extra; r.extra_mode = t.extra_mode;
    r.row_shift = t.row_shift; r.w_cols = t.Q; r.ld_w = t.ld_w; r.dst_w = t.dst_w; r.dst_b = t.dst_b;
    return r;
}

// Products that go together in one launch.
struct TnLaunch {
    TnGemmBatch batch{};
    int count = 0, max_qp = 0;
    void add(const TnGemmArgs &g) { batch.g[count++] = g; max_qp = std::max(max_qp, g.qp); }
};

template <auto kKernel>
hipError_t launch_tn(const TnLaunch &l, int chunks, size_t lds, hipStream_t stream)
{
    const hipError_t err = allow_large_lds<kKernel>(kLdsLimit);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(kKernel, dim3(chunks, l.count), dim3(kTnThreads), lds, stream, l.batch);
    return hipGetLastError();
}

template <int PBW, int QBN, bool BBF>
hipError_t launch_tn_shape(const TnLaunch &l, int planes, bool wide_loads, int chunks, hipStream_t stream)
{
    if (wide_loads) return launch_tn<tn_gemm_wide_kernel<PBW, QBN, BBF>>(l, chunks, tn_wide_lds<PBW, QBN>(), stream);
    const size_t lds = (size_t)2 * (128 * PBW + l.max_qp) * 80;      // 80 bytes per staged column; two planes, or two buffers of one
    if constexpr (!BBF)
        if (planes == 2) return launch_tn<tn_gemm_kernel<PBW, QBN, 2, false>>(l, chunks, lds, stream);
    return launch_tn<tn_gemm_kernel<PBW, QBN, 1, true, BBF>>(l, chunks, lds, stream);
}

// rows: row_class of all of them.  wide_loads: every one fits tn_gemm_wide_kernel.
hipError_t launch_shape(const TnLaunch &l, int rows, bool b_bf16, int planes, bool wide_loads, int chunks, hipStream_t stream)
{
    if (l.count == 0) return hipSuccess;
    if (rows == 1) return l.max_qp <= 176 ? launch_tn_shape<1, 11, false>(l, planes, wide_loads, chunks, stream)
                                          : launch_tn_shape<1, 21, false>(l, planes, wide_loads, chunks, stream);
    if (rows == 3) return b_bf16 ? launch_tn_shape<3, 9, true>(l, planes, wide_loads, chunks, stream)
                                 : launch_tn_shape<3, 9, false>(l, planes, wide_loads, chunks, stream);
    if (l.max_qp <= 80) return b_bf16 ? launch_tn_shape<2, 5, true>(l, planes, wide_loads, chunks, stream)
                                      : launch_tn_shape<2, 5, false>(l, planes, wide_loads, chunks, stream);
    return b_bf16 ? launch_tn_shape<2, 9, true>(l, planes, wide_loads, chunks, stream)
                  : launch_tn_shape<2, 9, false>(l, planes, wide_loads, chunks, stream);
}

}  // namespace

// Launches the products of `list` (all over the same M samples, chunks of `chunk`): those of one shape go
// together in one launch (up to kTnBatchMax), then their partial sums are reduced, again in one launch.
hipError_t launch_tn_products(int planes, const TnProduct *list, int count, long M, int chunk, float *partial,
                              size_t partial_bytes, hipStream_t stream)
{
    const int chunks = (int)((M + chunk - 1) / chunk);
    int done = 0;
    while (done < count) {
        TnLaunch rows[3];
        TnReduceBatch red{};
        int n_red = 0;
        size_t used = 0;
        int taken = done;
        bool a_in_groups = false, wide_loads = planes == 1 && list[done].a.bf16;
        for (; taken < count; ++taken) {
            const TnProduct &t = list[taken];
            TnGemmArgs g{};
            if (!tn_args(planes, t, M, chunk, reinterpret_cast<float *>(reinterpret_cast<char *>(partial) + used), &g)) return hipErrorInvalidValue;
            // A in groups: the wide kernel only
            if (t.a.rows_per_group < M && !(planes == 1 && tn_wide_fits(t, M))) return hipErrorInvalidValue;
            // bf16 adjoints are read 16 bytes (eight columns) at a time
            if (t.a.bf16 && (reinterpret_cast<uintptr_t>(t.a.base) % 16 != 0 || t.a.ld % 8 != 0 || t.a.ld < (t.P + 7) / 8 * 8)) return hipErrorInvalidValue;
            // B in bf16: such products go in launches of their own
            if ((t.b.bf16 != 0) != (list[done].b.bf16 != 0)) break;
            const size_t bytes = tn_partial_bytes(M, chunk, t.P, t.Q + t.n_extra);
            if (bytes > partial_bytes) return hipErrorInvalidValue;
            if (used + bytes > partial_bytes || n_red == kTnBatchMax) break;
            used += bytes;
            a_in_groups = a_in_groups || t.a.rows_per_group < M;
            wide_loads = wide_loads && tn_wide_fits(t, M);
            rows[row_class(t.P) - 1].add(g);
            red.r[n_red++] = reduce_args(t, g.partial, chunks);
        }
        if (a_in_groups && !wide_loads) return hipErrorInvalidValue;
        hipError_t err = hipSuccess;
        for (int k = 3; k >= 1 && err == hipSuccess; --k) err = launch_shape(rows[k - 1], k, list[done].b.bf16 != 0, planes, wide_loads, chunks, stream);
        if (err != hipSuccess) return err;
        err = launch_reduce(red, n_red, stream);
        if (err != hipSuccess) return err;
        for (int i = done; i < taken; ++i)
            if (list[i].extra_mode == kExtraAgent) {
                const TnProduct &t = list[i];
                hipLaunchKernelGGL(bias_from_columns_kernel, dim3((t.P + 255) / 256), dim3(256), 0, stream, t.dst_w, t.P, t.ld_w, t.Q,
                                   t.n_extra, t.dst_b);
                err = hipGetLastError();
                if (err != hipSuccess) return err;
            }
        done = taken;
    }
    return hipSuccess;
}

// The products of `list` (every one fits the wide kernel; same M and chunk), without the sum of their chunks:
// product i's partial sums go to partial[i].  One launch per shape and element type of B.
hipError_t launch_tn_gemms_wide(const TnProduct *list, int count, long M, int chunk, float *const *partial, hipStream_t stream)
{
    const int chunks = (int)((M + chunk - 1) / chunk);
    TnLaunch rows[3][2];                // by row class and element type of B
    for (int i = 0; i < count; ++i) {
        const TnProduct &t = list[i];
        TnGemmArgs g{};
        TnLaunch &l = rows[row_class(t.P) - 1][t.b.bf16 ? 1 : 0];
        if (!tn_wide_fits(t, M) || !tn_args(1, t, M, chunk, partial[i], &g) || l.count == kTnBatchMax) return hipErrorInvalidValue;
        l.add(g);
    }
    hipError_t err = hipSuccess;
    for (int k = 3; k >= 1; --k)
        for (int b = 1; b >= 0 && err == hipSuccess; --b) err = launch_shape(rows[k - 1][b], k, b != 0, 1, true, chunks, stream);
    return err;
}

// The GRU matrices' products and dpre1 over the samples of slots [t0, t1), 128 units and one plane; without the sum of the chunks.
hipError_t launch_gru_products(const BpttArgs &a, int t0, int t1, const SampleChunks &cut, float *partial_ih, float *partial_hh, hipStream_t stream)
{
    const NetFrags &net = a.net;
    const size_t H = net.H, N = net.N, T = a.T, first = (size_t)t0 * N;
    GruProductArgs g{};
    g.wihT = net.wihT_16;
    g.da = static_cast<const char *>(a.da) + first * 4 * H * 2;
    g.x = static_cast<const char *>(a.x_all) + first * H * 2;
    g.h = reinterpret_cast<const char *>(a.h_all + first * H);
    g.dpre1 = static_cast<char *>(a.dpre1) + first * H * 2;
    g.dpre1_bytes = (uint32_t)((a.B * T * N - first) * H * 2);
    g.partial[0] = partial_ih; g.partial[1] = partial_hh;
    g.M = (int)cut.samples; g.chunk = cut.chunk; g.chunks = cut.chunks;
    g.group = (uint32_t)((t1 - t0) * N); g.adj_group = (uint32_t)(T * N); g.act_group = (uint32_t)((T + 1) * N);
    const uint32_t groups = 32 / g.group;
    g.step_rows = 32 % g.group;
    g.adj_step = groups * g.adj_group + g.step_rows; g.act_step = groups * g.act_group + g.step_rows;
    const hipError_t err = allow_large_lds<gru_products_kernel>(kLdsLimit);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(gru_products_kernel, dim3((cut.chunks + 7) / 8 * 8 * kGruShare), dim3(kTnThreads), GruTile::kBytes, stream, g);
    return hipGetLastError();
}

bool qnet_grad_fits(const NetFrags &net)
{
    return unroll_fused_fits(net) && net.D + net.N <= 336;        // the widest product the gradient kernel stages
}

size_t qnet_grad_workspace_bytes(const NetFrags &net, int B, int T) { return make_plan(net, B, T).bytes; }

// grad: packed like the weights (W1, b1, W_ih, W_hh, b_ih, b_hh, W2, b2), device, fully overwritten.
void qnet_grad_activation_slots(const NetFrags &net, int B, int T, void *workspace, float **h_all, void **x_all)
{
    const Plan plan = make_plan(net, B, T);
    *h_all = reinterpret_cast<float *>(static_cast<char *>(workspace) + plan.off_h);
    *x_all = static_cast<char *>(workspace) + plan.off_x;
}

hipError_t launch_qnet_grad(const NetFrags &net, int B, int T, const float *obs, const int32_t *actions,
                            const uint8_t *filled, const float *grad_q, void *workspace, float *grad, hipStream_t stream,
                            bool activations_kept, const SideStream *side, int n_cu)
{
    const Plan plan = make_plan(net, B, T);
    char *ws = static_cast<char *>(workspace);
    float *h_all = reinterpret_cast<float *>(ws + plan.off_h);
    void *x_all = ws + plan.off_x;
    char *da = ws + plan.off_da, *dpre1 = ws + plan.off_dpre1, *dq = ws + plan.off_dq;
    float *partial = reinterpret_cast<float *>(ws + plan.off_partial);
    const int adj_bf16 = net.planes == 1 ? 1 : 0, adj_bytes = adj_bf16 ? 2 : 4;
    const int N = net.N, D = net.D, A = net.A, H = net.H, S = T + 1;

    // forward pass that keeps x and h, unless the caller's unroll has left them in the workspace
    hipError_t err = hipSuccess;
    if (!activations_kept)
        err = launch_unroll_fused(net, net, false, B, T, nullptr, B, obs, nullptr, actions, nullptr, nullptr, filled,
                                  0.0f, nullptr, nullptr, nullptr, nullptr, stream, kTdSave, nullptr, h_all, x_all);
    if (err != hipSuccess) return err;

    BpttArgs a{};
    a.net = net; a.B = B; a.T = T; a.a16 = plan.a16; a.actions = actions; a.filled = filled; a.grad_q = grad_q;
    a.h_all = h_all; a.x_all = x_all; a.da = da; a.dpre1 = dpre1; a.dq = dq;
    a.carry = reinterpret_cast<float *>(ws + plan.off_carry);
    const bool roles = H == 128 && net.planes == 1;
    bool eights = false;                                           // 64 units: tiles of eight rows
    auto reverse = [&](int t_begin, int t_end, hipStream_t on) {
        a.t_begin = t_begin; a.t_end = t_end;
        if (H == 64 && net.planes == 2) return eights ? back_dispatch<bptt_back_split8_kernel<2>>(a, 8, BpttSplit8<2>::kThreads, BpttSplit8<2>::lds_bytes(A), on)
                                                      : back_dispatch<bptt_back_split_kernel<2>>(a, 16, 512, BpttSplit<2>::kBytes, on);
        if (H == 64 && net.planes == 1) return eights ? back_dispatch<bptt_back_split8_kernel<1>>(a, 8, BpttSplit8<1>::kThreads, BpttSplit8<1>::lds_bytes(A), on)
                                                      : back_dispatch<bptt_back_split_kernel<1>>(a, 16, 512, BpttSplit<1>::kBytes, on);
        if (roles) return back_dispatch<bptt_back_roles_kernel>(a, 16, BpttRoles::kThreads, BpttRoles::lds_bytes(A), on);
        return hipErrorInvalidValue;
    };

    // offsets of the tensors in the packed vector
    float *gW1 = grad, *gb1 = gW1 + (size_t)H * (D + N), *gWih = gb1 + H, *gWhh = gWih + (size_t)3 * H * H;
    float *gbih = gWhh + (size_t)3 * H * H, *gbhh = gbih + 3 * H, *gW2 = gbhh + 3 * H, *gb2 = gW2 + (size_t)A * H;
    // The four products over the samples (b, t, n) of slots [t0, t1): every operand's rows come in groups of
    // (t1 - t0) N, one per episode.
    struct Four { TnProduct p[4]; };
    auto products_of = [&](int t0, int t1) {
        const int rows = (t1 - t0) * N;
        const size_t first = (size_t)t0 * N;                                 // rows of an episode before the window
        // (all slots: the adjoint arrays' rows follow one another across episodes, one group)
        const bool whole = t0 == 0 && t1 == T;
        const int rows_adj = whole ? (int)std::min<long>((long)B * N * T, 1 << 30) : rows;
        const RowMap da_i{da + first * 4 * H * adj_bytes, whole ? 0 : (long)T * N * 4 * H, rows_adj, 4 * H, adj_bf16};      // columns n, r, z
        RowMap da_h = da_i; da_h.base = da + (first * 4 * H + H) * adj_bytes;                            // columns r, z, n (hidden side)
        const RowMap x_rows{static_cast<const char *>(x_all) + first * H * adj_bytes, (long)S * N * H, rows, H, adj_bf16};      // stored as the adjoints are
        const RowMap h_prev{h_all + first * H, (long)S * N * H, rows, H, 0};
        const RowMap h_new{h_all + (first + N) * H, (long)S * N * H, rows, H, 0};
        const RowMap pre_rows{dpre1 + first * H * adj_bytes, whole ? 0 : (long)T * N * H, rows_adj, H, adj_bf16};
        const RowMap obs_rows{obs + first * D, (long)S * N * D, rows, D, 0};
        const RowMap dq_rows{dq + first * plan.a16 * adj_bytes, whole ? 0 : (long)T * N * plan.a16, rows_adj, plan.a16, adj_bf16};
        // W_ih and b_ih: the adjoint columns are n, r, z -> parameter rows r, z, n: shift by 2H
        return Four{{
            {da_i, x_rows, 3 * H, H, kExtraOnes, 1, N, 2 * H, H, gWih, gbih},
            {da_h, h_prev, 3 * H, H, kExtraOnes, 1, N, 0, H, gWhh, gbhh},
            {pre_rows, obs_rows, H, D, kExtraAgent, N, N, 0, D + N, gW1, gb1},
            {dq_rows, h_new, A, H, kExtraOnes, 1, N, 0, H, gW2, gb2},
        }};
    };

    // The reverse recurrence is one workgroup per 8 or 16 rows: a batch with fewer tiles than compute units leaves the
    // rest of the chip idle for as long as the episodes are.  Then the slots are walked in two launches, and the
    // products over the later half run on a second stream beside the earlier half's recurrence.
    const int tiles = (B * N + 15) / 16, t_mid = plan.cut.t_mid;
    const SampleChunks &cut_late = plan.cut.late, &cut_early = plan.cut.early;
    bool split = side && side->stream && net.planes == 1 && T >= kForkSlots && 2 * tiles <= 3 * n_cu / 2;
    Four late{}, early{};
    if (split) {
        late = products_of(t_mid, T); early = products_of(0, t_mid);
        for (int i = 0; i < 4 && split; ++i) split = tn_wide_fits(late.p[i], cut_late.samples) && tn_wide_fits(early.p[i], cut_early.samples);
    }
    // Tiles of eight rows where each has a compute unit of its own; beside products on the second stream, where enough are left for
    // those (three eighths).  Learner iteration, us, tiles of 16 / of 8, 60 slots: fp32 2048 rows 368 / 343, 1536 328 / 301, 35 220 /
    // 192; bf16 in two launches 1920 rows 257 / 262, 1536 245 / 248, 1200 238 / 236, 800 219 / 206, 200 x 200 slots 420 / 330, in
    // one (15 slots) 2048 rows 149 / 144.
    eights = (B * N + 7) / 8 <= (split ? n_cu * 5 / 8 : n_cu);
    if (!split) {
        const SampleChunks &cut = plan.cut.gru_whole;
        const size_t part = (size_t)cut.chunks * kGruRows * kGruColumns;
        if (roles && 2 * part * sizeof(float) > plan.partial_bytes) return hipErrorInvalidValue;
        err = reverse(0, T, stream);
        if (err != hipSuccess) return err;
        const Four all = products_of(0, T);
        int done = 0;
        if (roles) {
            float *const parts[2] = {partial, partial + part};
            err = launch_gru_products(a, 0, T, cut, parts[0], parts[1], stream);
            if (err != hipSuccess) return err;
            TnReduceBatch red{};
            for (; done < 2; ++done) red.r[done] = reduce_args(all.p[done], parts[done], cut.chunks);
            err = launch_reduce(red, 2, stream);
            if (err != hipSuccess) return err;
        }
        return launch_tn_products(net.planes, all.p + done, 4 - done, plan.cut.whole.samples, plan.cut.whole.chunk, partial, plan.partial_bytes, stream);
    }
    // a product's partial sums: the later half's chunks, then the earlier half's, summed in that order
    float *part_late[4], *part_early[4];
    TnReduceBatch red{};
    {
        size_t used = 0;
        for (int i = 0; i < 4; ++i) {
            const TnProduct &t = late.p[i];
            const size_t p_pad = (size_t)partial_rows(t.P), qp = (size_t)(t.Q + t.n_extra + 15) / 16 * 16;
            const int n_late = (roles && i < 2 ? plan.cut.gru_late : cut_late).chunks, n_early = (roles && i < 2 ? plan.cut.gru_early : cut_early).chunks;
            part_late[i] = reinterpret_cast<float *>(reinterpret_cast<char *>(partial) + used);
            part_early[i] = part_late[i] + (size_t)n_late * p_pad * qp;
            used += (size_t)(n_late + n_early) * p_pad * qp * sizeof(float);
            red.r[i] = reduce_args(t, part_late[i], n_late + n_early);
        }
        if (used > plan.partial_bytes) return hipErrorInvalidValue;
    }
    err = reverse(t_mid, T, stream);
    if (err == hipSuccess) err = hipEventRecord(side->fork, stream);
    if (err == hipSuccess) err = hipStreamWaitEvent(side->stream, side->fork, 0);
    if (roles) {
        if (err == hipSuccess) err = launch_gru_products(a, t_mid, T, plan.cut.gru_late, part_late[0], part_late[1], side->stream);
        if (err == hipSuccess) err = launch_tn_gemms_wide(late.p + 2, 2, cut_late.samples, cut_late.chunk, part_late + 2, side->stream);
        if (err == hipSuccess) err = hipEventRecord(side->join, side->stream);
        if (err == hipSuccess) err = reverse(0, t_mid, stream);
        if (err == hipSuccess) err = launch_gru_products(a, 0, t_mid, plan.cut.gru_early, part_early[0], part_early[1], stream);
        if (err == hipSuccess) err = launch_tn_gemms_wide(early.p + 2, 2, cut_early.samples, cut_early.chunk, part_early + 2, stream);
    } else {
        if (err == hipSuccess) err = launch_tn_gemms_wide(late.p, 4, cut_late.samples, cut_late.chunk, part_late, side->stream);
        if (err == hipSuccess) err = reverse(0, t_mid, stream);
        // the earlier half: W_hh's product follows on the second stream (a second fork: it needs the recurrence's end),
        // the other three on the caller's
        if (err == hipSuccess) err = hipEventRecord(side->fork, stream);
        if (err == hipSuccess) err = hipStreamWaitEvent(side->stream, side->fork, 0);
        if (err == hipSuccess) err = launch_tn_gemms_wide(early.p + 1, 1, cut_early.samples, cut_early.chunk, part_early + 1, side->stream);
        if (err == hipSuccess) err = hipEventRecord(side->join, side->stream);
        if (err == hipSuccess) err = launch_tn_gemms_wide(early.p, 1, cut_early.samples, cut_early.chunk, part_early, stream);
        if (err == hipSuccess) err = launch_tn_gemms_wide(early.p + 2, 2, cut_early.samples, cut_early.chunk, part_early + 2, stream);
    }
    if (err == hipSuccess) err = hipStreamWaitEvent(stream, side->join, 0);
    if (err != hipSuccess) return err;
    err = launch_reduce(red, 4, stream);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(bias_from_columns_kernel, dim3((H + 255) / 256), dim3(256), 0, stream, gW1, H, D + N, D, N, gb1);
    return hipGetLastError();
}

}  // namespace marl
