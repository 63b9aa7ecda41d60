// The arithmetic of the point lists that several workgroups write in order
// (track.hip): the words in which the workgroups publish their counts, and
// the list positions that follow from them.  Plain functions, so that the
// host can check every index that they give.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace rose {

// A part is 1024 padded samples or points; its word is the launch that it was
// published in, then two counts of at most 1024 each.
constexpr int kPartPoints = 1024;
constexpr int kCountBits = 11;
constexpr int kTagShift = 2 * kCountBits;
constexpr uint64_t kCountMask = (1u << kCountBits) - 1u;

__host__ __device__ inline uint64_t launch_tag(uint64_t launch) { return (launch + 1) << kTagShift; }

__host__ __device__ inline uint64_t part_word(uint64_t tag, uint32_t first, uint32_t second) {
    return tag | (uint64_t)second << kCountBits | first;
}

__host__ __device__ inline bool part_published(uint64_t word, uint64_t tag) {
    return word >> kTagShift == tag >> kTagShift;
}

// first count in the low word, second in the high word (sums of up to
// kMaxParts of these stay apart)
__host__ __device__ inline uint64_t part_counts(uint64_t word) {
    return (word & kCountMask) | ((word >> kCountBits) & kCountMask) << 32;
}

// "a predecessor never published" in the place of a sum of part_counts
constexpr uint64_t kCountsLost = ~0ull;

// Position of a part's element number `pos` in a list of `cap` elements after
// the `before` elements of its predecessors, or -1: past the list (counts of
// a frame that another stream set up in the same handle) or unknown.
__host__ __device__ inline int list_slot(uint64_t counts, int which, int pos, int cap) {
    if (counts == kCountsLost) return -1;
    const uint32_t at = (uint32_t)(counts >> (32 * which)) + (uint32_t)pos;
    return at < (uint32_t)cap ? (int)at : -1;
}

// number of elements of a list of `cap` elements
__host__ __device__ inline int list_size(uint64_t counts, int which, int cap) {
    if (counts == kCountsLost) return 0;
    const uint32_t n = (uint32_t)(counts >> (32 * which));
    return n < (uint32_t)cap ? (int)n : cap;
}

}  // namespace rose
