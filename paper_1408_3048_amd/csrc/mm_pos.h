// Positions within a P^T work range: sorted samples counted from a base sample, a multiple of 64.
//
// A range holds whole pixels, so its length is bounded by the hits of one pixel alone, which
// can be every sample of the plan (samples that a survey flags share one pixel): up to 2^31 - 1,
// with the chunk loop and its prefetch running up to two chunks past the end.  Positions are
// signed 32-bit values, from a base at or up to 63 samples below the first sample, or 2^30 further
// up for ranges of more than 2^30 samples, so that none overflows.  (Unsigned ones, whose wrap the
// compiler has to allow for in every address, cost P^T of 2^22 samples in FP64 31.2 us for 29.8.)
// Offsets into the weights (two a sample) and byte offsets don't fit 32 bits and are 64-bit.
#pragma once

#include <cstdint>

namespace mm {

typedef int32_t pos_t;

// the sample that positions in the range [i0, i1) count from
constexpr int64_t range_base(int64_t i0, int64_t i1) {
    return (i0 & ~(int64_t)63) + (i1 - i0 > ((int64_t)1 << 30) ? (int64_t)1 << 30 : 0);
}
// start of the first chunk (chunks are aligned to the e samples of a lane)
constexpr pos_t first_chunk(pos_t i0, int e) { return i0 & ~(pos_t)(e - 1); }
// start of the chunk after c: 64 lanes of e samples
constexpr pos_t next_chunk(pos_t c, int e) { return c + 64 * e; }
// first sample of a lane in the chunk at c
constexpr pos_t lane_base(pos_t c, int lane, int e) { return c + e * lane; }
// index of sample i's first weight
constexpr int64_t weight_index(pos_t i) { return 2 * (int64_t)i; }

}  // namespace mm
