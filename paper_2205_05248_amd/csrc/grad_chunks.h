// Which weight-gradient products there are kernels for, and how the backward pass cuts the samples of its products into chunks,
// one workgroup and one set of partial sums each.  Host arithmetic only, in one place for the launches and for the workspace
// that they write to.
#pragma once

#include <algorithm>

namespace marl {

// What a product needs of its kernel: rows 3 (up to 384), 2 (256) or 1 (128).
inline int row_class(int P) { return P > 256 ? 3 : P > 128 ? 2 : 1; }

// Whether there is a kernel for a product of P rows and `columns` columns (appended ones included, padded to 16).  The kernels
// read an operand as the elements that they are compiled for: A (the adjoints) is bf16 in a one-plane network and fp32 in
// one of two planes, B (states, activations) fp32, or bf16 beside bf16 adjoints in the shapes above 128 rows.
inline bool has_product_kernel(int planes, bool a_bf16, bool b_bf16, int P, int columns)
{
    if (a_bf16 != (planes == 1) || (b_bf16 && !(a_bf16 && P > 128))) return false;
    return P > 128 ? P <= 384 && columns <= 144 : columns <= 336;
}

// chunk: samples of every chunk but the last, whole rounds of two steps of 32
struct SampleChunks { long samples; int chunk, chunks; };

inline SampleChunks cut_samples(long samples, long most_chunks, long least_samples)
{
    const long wanted = std::max(1L, std::min(most_chunks, (samples + least_samples - 1) / least_samples));
    const long chunk = ((samples + wanted - 1) / wanted + 63) / 64 * 64;
    return {samples, (int)chunk, (int)((samples + chunk - 1) / chunk)};
}

// The reverse recurrence may walk the slots in two launches from this many on (one-plane networks).
constexpr int kForkSlots = 16;

struct GradChunks {
    SampleChunks whole;            // one launch of the recurrence, products over all slots
    int t_mid;                     // two launches: slots [t_mid, T), then [0, t_mid)
    SampleChunks late, early;
    int room;                      // most chunks whose partial sums lie in the workspace together
};

// rows: episodes times agents.
inline GradChunks grad_chunks(int planes, long rows, int T)
{
    GradChunks g{};
    const long M = rows * T;
    // Every chunk's partial sums are written once and read once more, up to 221 KB each, where 32 samples are 60 KB at
    // most: few chunks for few samples.  Two planes: the products of a launch come in pairs, 128 chunks each, which
    // are the chip's 256 compute units once, where up to 256 each were one wave and a part of another (gradient with up to
    // 256 / 128 chunks, 96 observations: 8400 samples 111 / 100 us, 38400 362 / 341, 102400 405 / 379, 815900 2068 / 2043;
    // the same below 8192).  One plane (a GRU product is alone in its launch): up to 256 chunks.  Of 64 samples
    // for the fewest, where the steps that follow one another in a chunk are what takes time, of 128 or more beyond,
    // where the partial sums are.  Gradient with chunks of 64 / 128, 128 units and 93 observations: 720 samples 95 / 100 us,
    // 1200 104 / 109, 2250 111 / 113, 2400 131 / 132, 3000 139 / 133, 3600 121 / 120, 4000 144 / 133, 4800 284 / 279,
    // 9900 297 / 290; 64 units, and 33 and 301 observations, change over between the same 2400 and 3000.
    g.whole = planes == 2 ? cut_samples(M, 128, 32) : cut_samples(M, 256, M <= 2560 ? 64 : 128);
    g.room = g.whole.chunks;
    if (planes == 1 && T >= kForkSlots) {
        // the later half's products share the chip with the recurrence, whose workgroups hold half the compute units
        // or less: half as many chunks.  The earlier half's too: its two GRU products then run side by side, one on
        // each stream, 128 workgroups each (256 chunks for the first layer's product, which runs last and alone,
        // changed nothing).  Both halves' partial sums wait for one sum.
        g.t_mid = T / 2;
        g.late = cut_samples(rows * (T - g.t_mid), 128, 32);
        g.early = cut_samples(rows * g.t_mid, 128, 32);
        g.room = std::max(g.room, g.late.chunks + g.early.chunks);
    }
    return g;
}

}  // namespace marl
