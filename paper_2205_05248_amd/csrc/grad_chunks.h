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

// A list of products is launched so many at a time, each with a set of chunks.
constexpr int kProductsPerLaunch = 16;

// count things in as few and as equal parts as hold `most` of them at most: part i has size(i), from first(i) on.
struct EvenParts {
    int count, parts;
    int size(int i) const { return count / parts + (i < count % parts ? 1 : 0); }
    int first(int i) const { return count / parts * i + (i < count % parts ? i : count % parts); }
};
inline EvenParts even_parts(int count, int most) { return {count, std::max(1, (count + most - 1) / most)}; }

// The rows of a matrix of more than 128, in blocks of 16: parts of at most 384 rows, as few as there can be with all of one
// row class, whose products then go together in one launch.  1024 rows as 384 + 384 + 256, or 528 as 272 + 256, are two
// launches in a row that share out the compute units among all the products and then use a part of them each.  Mixer gradient, slices
// of 384 and the rest / these: 32 agents x 32, state 256, 6400 transitions fp32 148 / 126 us, 12800 bf16 114 / 100; 33 x 16, state
// 400, 182 / 152 and 127 / 110.
inline EvenParts tall_slices(int rows)
{
    EvenParts s = even_parts((rows + 15) / 16, 24);
    while (row_class(16 * s.size(0)) != row_class(16 * s.size(s.parts - 1))) ++s.parts;
    return s;
}

// The mixer's products: those of its largest matrix, if it is taller than 128 rows (128 state columns each), and those of the
// others (320 columns) and of v2.
constexpr int kTallColumns = 128, kFlatColumns = 320;
struct MixerProducts { int tall, flat; };
inline MixerProducts mixer_products(int largest_rows, int state_dim)
{
    const int per_flat = (state_dim + kFlatColumns - 1) / kFlatColumns, flat = 3 * per_flat + 1;
    if (largest_rows <= 128) return {0, flat + per_flat};
    return {tall_slices(largest_rows).parts * ((state_dim + kTallColumns - 1) / kTallColumns), flat};
}

// The mixer's chunks, for a launch of `products`.  One workgroup per product and chunk, one per compute unit: as many chunks as
// let the launch fill the chip once, of 64 transitions (two steps) at least.  Chunks of 256 transitions whatever the number of
// products left all but 30 compute units idle on 7680 transitions of 160 x 120 weights (31 + 21 us for the products), one chunk
// in all on 240.  What counts is the products of the launch, not of the list: 24 products of ten chunks each, in launches of
// sixteen and eight, were slower than with chunks of 256 (32 agents x 64, state 512, 6400 transitions fp32: chunks of 256 472 us,
// ten chunks 542, two launches of 12 x 21 chunks 432).
inline SampleChunks mixer_chunks(long transitions, int products) { return cut_samples(transitions, 256 / products, 64); }

// The reverse recurrence may walk the slots in two launches from this many on (one-plane networks).
constexpr int kForkSlots = 16;

struct GradChunks {
    SampleChunks whole;            // one launch of the recurrence, products over all slots
    int t_mid;                     // two launches: slots [t_mid, T), then [0, t_mid)
    SampleChunks late, early;
    // the same three for the GRU matrices of 128 units, one plane (gru_products_kernel: four workgroups a chunk)
    SampleChunks gru_whole, gru_late, gru_early;
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
    // 9900 297 / 290; 64 units, and 33 and 301 observations, change over between the same 2400 and 3000.  (Measured with the GRU
    // products of 128 units among them, which have chunks of their own by now.)
    g.whole = planes == 2 ? cut_samples(M, 128, 32) : cut_samples(M, 256, M <= 2560 ? 64 : 128);
    g.room = g.whole.chunks;
    // 64 chunks of four workgroups each are the chip's compute units once.
    auto cut_gru = [](long samples, long most) { return cut_samples(samples, std::min(64L, most), 64); };
    if (planes == 1 && T >= kForkSlots) {
        // the later half's products share the chip with the recurrence, whose workgroups hold three quarters of the compute
        // units at most: half as many chunks.  The earlier half's too: the two GRU products of 64 units then run side by
        // side, one on each stream, 128 workgroups each (256 chunks for the first layer's product, which runs last and
        // alone, changed nothing).  Both halves' partial sums wait for one sum.
        g.t_mid = T / 2;
        g.late = cut_samples(rows * (T - g.t_mid), 128, 32);
        g.early = cut_samples(rows * g.t_mid, 128, 32);
        // 128 units: both GRU products are one launch, the earlier half's on the caller's stream.  (Beside the recurrence half as
        // many chunks, 128 workgroups for the 128 compute units that it leaves on 64 x 200 x 32: with 64 chunks 64 episodes x 200
        // slots x 32 agents 1196 us for the learner iteration, with 32 1191; 64 x 120 x 8 466 / 458, 9 x 200 x 32 698 / 688)
        g.gru_late = cut_samples(rows * (T - g.t_mid), 32, 64);
        g.gru_early = cut_gru(rows * g.t_mid, 64);
        g.room = std::max(g.room, g.late.chunks + g.early.chunks);
    }
    // No more than there is room for, or a workspace that holds the other products' partial sums would not hold these: fewer than
    // kForkSlots slots and 2561 to 4096 samples, half as many chunks, of 128 samples, as the other products have.
    g.gru_whole = cut_gru(M, g.room);
    return g;
}

}  // namespace marl
