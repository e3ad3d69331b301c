// How the backward pass cuts the samples of its weight-gradient products into chunks, one workgroup and one set of
// partial sums each.  Host arithmetic only, in one place for the launches and for the workspace that they write to.
#pragma once

#include <algorithm>

namespace marl {

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
    // are the chip's 256 compute units once, where up to 256 each were one wave and a part of another; learner iteration
    // of 64 x 120 x 5 502 -> 481 us.  One plane (a GRU product is alone in its launch): up to 256 chunks, of 64 samples
    // up to 4096 of them, where the steps that follow one another in a chunk are what takes time (gradient at 576 / 720 /
    // 2400 samples 71 / 182 / 201 us, with chunks of 128 75 / 188 / 202), of 128 or more beyond, where the partial sums
    // are (6640 / 15360 samples 274 / 130 us, 271 / 110 with 128; 128 hidden units all).
    g.whole = planes == 2 ? cut_samples(M, 128, 32) : cut_samples(M, 256, M <= 4096 ? 64 : 128);
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
