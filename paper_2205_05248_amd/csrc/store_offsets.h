// What the gradient's arrays are bounded to, and the byte offsets at which the reverse recurrence's buffer stores are dropped.
// Plain C++, in one place for the host's check and for the kernels.
#pragma once

#include <cstdint>

namespace marl {

// The largest gradient: 4 H numbers of every row and slot, the slot behind the last among them, are fewer than 2^30.  The adjoints
// of the gates are then below 2^32 bytes in fp32 and below 2^31 in bf16; dpre1 and the adjoint of Q are below 2^30 in either.
constexpr bool gradient_in_range(int64_t B, int64_t N, int64_t T, int64_t H) { return B * N * (T + 1) * 4 * H < (int64_t)1 << 30; }

// Every global access inside the loops over the slots is unconditional, so that their bodies are straight-line code and
// the waits for the prefetched inputs count exactly the stores issued after them: rows past the end store through
// buffer descriptors at an offset beyond the descriptor, which the hardware drops.
// kDrop: beyond any of these arrays, as a whole offset; nothing can be added to it.
constexpr uint32_t kDrop = 0xFFFFFFF0u;
constexpr uint32_t store_offset(uint32_t lane_at, uint32_t slot_at, bool exists) { return exists ? lane_at + slot_at : kDrop; }
// A row of a whole wave that does not exist: a descriptor of no bytes.
constexpr uint32_t descriptor_bytes(uint64_t bytes, bool exists) { return exists ? (uint32_t)bytes : 0u; }
// kPast: beyond the arrays of less than 2^31 bytes, in place of a lane's part; a slot's part within such an array may be added.
constexpr uint32_t kPast = 0x80000000u;

}  // namespace marl
