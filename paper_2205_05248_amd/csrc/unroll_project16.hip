// Input projection of the two-kernel unroll for 128 hidden units in fp32: x = ReLU(W1 o + b1[agent]) and the gate inputs
// W_ih x + b of every (episode, slot, agent), into the scratch buffer that the recurrence reads (unroll_recur16.hip).
//
// The rows do not depend on each other; what bounds it is how often the weights (352 KB with 300 observations, two planes)
// travel.  front_kernel (kernels.hip) streams them through LDS once per 128 rows, a barrier per 24 KB: 27 us for the 21,655
// rows of 61 episodes x 70 slots x 5 agents, whatever their width.  Here they stay in registers: eight waves, each with its block of
// 16 units of both layers (80 registers of W1 at most, 96 of W_ih), one workgroup per compute unit, the networks taking
// turns, which takes a run of items (16 rows of one slot).  One LDS-only barrier per item; in the step of item i a wave
//   puts its part of item i+1's observations down as operand fragments and asks for its part of item i+2's,
//   forms its block of x of item i, and its block of the gate inputs of item i-1.
// Every global access is unconditional (the ends load an item again), so that the waits count exactly.
//
// A lane takes eight observations at a time, 32 k + 8 q + 0..7 of its row.  The row's end rarely falls on eight: there the
// lane reads the row's last eight instead, and the weights of that k-step are shifted to match once, in the prologue.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "fused16_roles.h"

namespace marl {

namespace {

constexpr int kProjWaves = 8, kProjThreads = 64 * kProjWaves;

struct ProjectArgs {
    NetFrags net[2];
    char *gi[2];
    int nets, B, T;
    const int32_t *episode_index;        // null, or the pool episode of each batch position
    int pool_episodes;
    const float *obs;
    int items, per_group;                // 16-row tiles times slots; of them per workgroup
    uint32_t magic;                      // ceil(2^32 / N): row / N is a multiplication, exact below 2^26 rows
};

}  // namespace

// KM: k-steps over the observations, the network's own rounded up (weights of the rest zero).
template <int KM>
__global__ __launch_bounds__(kProjThreads, 2) void project16_kernel(const ProjectArgs a)
{
    constexpr int H = 128, P = 2, KS = H / 32, FBK = H / 16;
    constexpr int kGateBytes = (H / 32) * GiLayout<P>::kBlockBytes, kSlotBytes = 3 * kGateBytes;      // of 32 rows
    constexpr int kParts = (KM + kProjWaves - 1) / kProjWaves;      // fragments of the observations a wave fetches
    __shared__ bf16x8 o_lds[2][KM][P][64], x_lds[2][KS][P][64];
    __shared__ __attribute__((aligned(16))) float b_lds[3 * H];      // gate biases r, z, n input side

    const int lane = threadIdx.x & 63, q4 = lane >> 4, c = lane & 15;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int which = (int)(blockIdx.x % (unsigned)a.nets), group = (int)(blockIdx.x / (unsigned)a.nets);
    const NetFrags &net = a.net[which];
    char *const gi = a.gi[which];
    const int N = net.N, D = net.D, S = a.T + 1, rows = a.B * N, ks1 = (D + 31) / 32;
    const int first = group * a.per_group, n = min(a.items - first, a.per_group);
    if (n <= 0) return;

    WFrag<P> w1[KM], wih[3][KS];
#pragma unroll
    for (int ks = 0; ks < KM; ++ks) {
        w1[ks] = load_wfrag<P>(net.w1_16 + ((size_t)(w * ks1 + min(ks, ks1 - 1)) * P) * 64 + lane);
        const int shift = ks < ks1 ? min(max(32 * ks + 8 * q4 - (D - 8), 0), 8) : 8;
        w1[ks].hi = shift_up(w1[ks].hi, shift);
        w1[ks].lo = shift_up(w1[ks].lo, shift);
    }
#pragma unroll
    for (int gate = 0; gate < 3; ++gate)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            wih[gate][ks] = load_wfrag<P>(net.wih_16 + ((size_t)((gate * FBK + w) * KS + ks) * P) * 64 + lane);
    if (threadIdx.x < 3 * H) {
        const int gate = (int)threadIdx.x / H;
        b_lds[threadIdx.x] = (gate == 0 ? net.bias_r : gate == 1 ? net.bias_z : net.bias_in)[threadIdx.x % H];
    }

    // item -> (tile, slot), stepped: at = the next item whose rows are looked up
    int tile = first / S, slot = first - tile * S, left = n;
    const int32_t *const index = a.episode_index ? a.episode_index : reinterpret_cast<const int32_t *>(a.obs);      // read either way
    struct Rows { int b, n, slot; int32_t listed; };
    auto look_up = [&](Rows &r) {                     // the next item's row of this lane, and its entry in the index
        const int row = tile * 16 + c;
        const uint32_t at = row < rows ? (uint32_t)row : 0u;      // rows past the end compute on row 0's inputs
        r.b = (int)__umulhi(at, a.magic);
        if (N == 1) r.b = (int)at;                    // (2^32 does not fit the factor)
        r.n = (int)at - r.b * N;
        r.slot = slot;
        r.listed = index[a.episode_index ? r.b : 0];
        const bool more = left > 1;                   // the run's last item again and again at its end
        left -= more ? 1 : 0;
        slot += more ? 1 : 0;
        const bool wrap = slot == S;
        slot = wrap ? 0 : slot;
        tile += wrap ? 1 : 0;
    };
    struct Obs { f32x4 v[kParts][2], b1; };
    auto fetch = [&](Obs &o, const Rows &r) {
        const int bi = a.episode_index ? min(max(r.listed, 0), a.pool_episodes - 1) : r.b;
        const float *row = a.obs + (((size_t)bi * S + r.slot) * N + r.n) * D;
#pragma unroll
        for (int p = 0; p < kParts; ++p) {
            const int k0 = min(32 * min(w + p * kProjWaves, KM - 1) + 8 * q4, D - 8);
            __builtin_memcpy(&o.v[p][0], row + k0, 16);
            __builtin_memcpy(&o.v[p][1], row + k0 + 4, 16);
        }
        o.b1 = load_feature4(net.bias1 + (size_t)r.n * H, w, q4);
    };
    auto deposit = [&](const Obs &o, int buf) {
#pragma unroll
        for (int p = 0; p < kParts; ++p) {
            const int ks = w + p * kProjWaves;
            if (ks < KM) {
                const float v[8] = {o.v[p][0][0], o.v[p][0][1], o.v[p][0][2], o.v[p][0][3], o.v[p][1][0], o.v[p][1][1], o.v[p][1][2], o.v[p][1][3]};
                const Frag<P> f = to_frag<P>(v);
                o_lds[buf][ks][0][lane] = f.hi;
                o_lds[buf][ks][1][lane] = f.lo;
            }
        }
    };
    // this lane's place in a gate's block of a record (unroll_common.h, GiLayout<2>), without the half that the tile is
    const uint32_t gi_lane = (uint32_t)((w >> 1) * GiLayout<P>::kBlockBytes + (2 * (w & 1) + (q4 >> 1)) * 1024 + ((q4 & 1) * 32 + c) * 16);

    int out_tile = tile, out_slot = slot;             // of the item whose gate inputs are stored next
    f32x4 b1_ready;                                   // of the item whose x is formed next
    auto step = [&](int s, Obs &o, Rows &r, auto has_x, auto has_gates) {
        // observations of item s+1 -> LDS, those of item s+2 asked for, the rows of item s+3 looked up
        const f32x4 b1 = b1_ready;
        b1_ready = o.b1;
        deposit(o, (s + 1) & 1);
        fetch(o, r);
        look_up(r);
        f32x4 x = {0.0f, 0.0f, 0.0f, 0.0f};
        if constexpr (decltype(has_x)::value) {
#pragma unroll
            for (int ks = 0; ks < KM; ++ks) {
                Frag<P> f;
                f.hi = o_lds[s & 1][ks][0][lane];
                f.lo = o_lds[s & 1][ks][1][lane];
                mma16<P>(x, w1[ks], f);
            }
        }
        if constexpr (decltype(has_gates)::value) {
            f32x4 r_in = load_feature4(b_lds, w, q4), z_in = load_feature4(b_lds + H, w, q4), n_in = load_feature4(b_lds + 2 * H, w, q4);
            f32x4 *const acc[3] = {&r_in, &z_in, &n_in};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                Frag<P> f;
                f.hi = x_lds[(s + 1) & 1][ks][0][lane];
                f.lo = x_lds[(s + 1) & 1][ks][1][lane];
                const WFrag<P> *const wf[3] = {&wih[0][ks], &wih[1][ks], &wih[2][ks]};
                mma16_across<P, 3>(acc, wf, f);
            }
            char *at = gi + ((size_t)(out_tile >> 1) * S + out_slot) * kSlotBytes + (out_tile & 1) * 256;
            *reinterpret_cast<f32x4 *>(at + gi_lane) = r_in;
            *reinterpret_cast<f32x4 *>(at + kGateBytes + gi_lane) = z_in;
            *reinterpret_cast<f32x4 *>(at + 2 * kGateBytes + gi_lane) = n_in;
            ++out_slot;
            const bool wrap = out_slot == S;
            out_slot = wrap ? 0 : out_slot;
            out_tile += wrap ? 1 : 0;
        }
        if constexpr (decltype(has_x)::value) {
            typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
            bf16x4 hi, lo;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                x[i] = fmaxf(x[i] + b1[i], 0.0f);
                hi[i] = (__bf16)x[i];
                lo[i] = (__bf16)(x[i] - (float)hi[i]);
            }
            char *at = reinterpret_cast<char *>(&x_lds[s & 1][w / 2][0][lane]) + (w & 1) * 8;
            *reinterpret_cast<bf16x4 *>(at) = hi;
            *reinterpret_cast<bf16x4 *>(at + 1024) = lo;
        }
        lds_barrier();
    };
    using Yes = std::true_type;
    using No = std::false_type;
    Rows r{};
    Obs o;
    look_up(r);
    fetch(o, r);                                      // item 0
    look_up(r);
#pragma unroll
    for (int ks = 0; ks < KM; ++ks) settle(w1[ks]);
#pragma unroll
    for (int gate = 0; gate < 3; ++gate)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) settle(wih[gate][ks]);
    b1_ready = o.b1;
    step(-1, o, r, No{}, No{});
    step(0, o, r, Yes{}, No{});
    for (int s = 1; s < n; ++s) step(s, o, r, Yes{}, Yes{});
    step(n, o, r, No{}, Yes{});
}

bool project16_fits(const NetFrags &net) { return net.H == 128 && net.planes == 2 && net.D >= 8 && net.D <= 320; }

hipError_t launch_project16(const NetFrags &online, const NetFrags &target, bool two_nets, char *gi_online, char *gi_target, int B, int T,
                            const int32_t *episode_index, int pool_episodes, const float *obs, int n_cu, hipStream_t stream)
{
    if (!project16_fits(online)) return hipErrorInvalidValue;
    ProjectArgs a{};
    a.net[0] = online; a.net[1] = target;
    a.gi[0] = gi_online; a.gi[1] = gi_target;
    a.nets = two_nets ? 2 : 1; a.B = B; a.T = T;
    a.episode_index = episode_index; a.pool_episodes = pool_episodes; a.obs = obs;
    a.items = (B * online.N + 15) / 16 * (T + 1);      // below 2^27: the host bounds rows (T + 1) D to 2^30, and D >= 8
    const int groups = n_cu / a.nets > 0 ? n_cu / a.nets : 1;
    a.per_group = (a.items + groups - 1) / groups;
    a.magic = (uint32_t)((0x100000000ull + (unsigned)online.N - 1) / (unsigned)online.N);
    const dim3 grid((unsigned)((a.items + a.per_group - 1) / a.per_group * a.nets)), block(kProjThreads);
    const int ks1 = (online.D + 31) / 32;
    if (ks1 <= 2) hipLaunchKernelGGL((project16_kernel<2>), grid, block, 0, stream, a);
    else if (ks1 <= 4) hipLaunchKernelGGL((project16_kernel<4>), grid, block, 0, stream, a);
    else if (ks1 <= 6) hipLaunchKernelGGL((project16_kernel<6>), grid, block, 0, stream, a);
    else if (ks1 <= 8) hipLaunchKernelGGL((project16_kernel<8>), grid, block, 0, stream, a);
    else hipLaunchKernelGGL((project16_kernel<10>), grid, block, 0, stream, a);
    return hipGetLastError();
}

}  // namespace marl
