// Range arithmetic of the k-th smallest search in select.hip (block_kth): the values left in [lo, hi]
// are counted in at most 1,024 parts of 2^shift values, and the range is cut to the part that holds the
// k-th one. Unsigned 32-bit arithmetic over the whole range, its ends included; plain integer code,
// which a host test runs over those ends.
#pragma once

#include <stdint.h>

namespace elis {

constexpr int kKthBins = 1024;

struct KthRange {
    uint32_t lo, hi;  // lo <= hi

    // log2 of the part size: (v - lo) >> shift() is below kKthBins for every v in [lo, hi].
    __host__ __device__ int shift() const {
        const int bits = hi > lo ? 32 - __builtin_clz(hi - lo) : 0;
        return bits > 10 ? bits - 10 : 0;
    }
    __host__ __device__ uint32_t part(uint32_t v, int shift) const { return (v - lo) >> shift; }
    // Part p, which holds a value: its end is compared by its distance from lo, since lo + width may pass 2^32.
    __host__ __device__ void cut(uint32_t p, int shift) {
        lo += p << shift;
        const uint32_t width = (1u << shift) - 1u;
        if (hi - lo > width) hi = lo + width;
    }
};

}  // namespace elis
