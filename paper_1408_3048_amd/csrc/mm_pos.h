// Positions within a P^T work range: sorted samples counted from a multiple of 64 at or below
// the range's first.
//
// A range holds whole pixels, so its length is bounded by the hits of one pixel alone, which
// can be every sample of the plan (samples that a survey flags share one pixel): positions reach
// 2^31 + 62, and the chunk loop and its prefetch run up to two chunks past the end.  They are
// unsigned 32-bit values, which hold all of these; offsets into the weights (two a sample) and
// byte offsets don't fit 32 bits and are 64-bit.
#pragma once

#include <cstdint>

namespace mm {

typedef uint32_t pos_t;

// start of the first chunk (chunks are aligned to the e samples of a lane)
constexpr pos_t first_chunk(pos_t i0, int e) { return i0 & ~(pos_t)(e - 1); }
// start of the chunk after c: 64 lanes of e samples
constexpr pos_t next_chunk(pos_t c, int e) { return c + 64u * (pos_t)e; }
// first sample of a lane in the chunk at c
constexpr pos_t lane_base(pos_t c, int lane, int e) { return c + (pos_t)(e * lane); }
// index of sample i's first weight
constexpr int64_t weight_index(pos_t i) { return 2 * (int64_t)i; }

}  // namespace mm
