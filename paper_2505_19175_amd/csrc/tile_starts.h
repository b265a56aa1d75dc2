// tile_starts.h -- the tiles' starts in a list of instances.
//
// N triangles over T tiles make up to N T instances, which 32 bits do not hold
// (3M triangles that average 1432 tiles), while a list holds fewer than 2^32.
// Sums saturate at 2^32 - 1, so that past it no start, run or cursor comes back
// to the list's first slots and no two tiles' runs overlap.  (Saturating 32-bit
// sums, not 64-bit ones: those cost the binning's scan a microsecond.)
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ts {

__host__ __device__ __forceinline__ uint32_t add_sat(uint32_t a, uint32_t b)
{
    const uint32_t s = a + b;   // one instruction on the GPU
    return s < a ? 0xffffffffu : s;
}

// Instances of tiles t0 .. t1 - 1, whose counts are in s_t.
__host__ __device__ __forceinline__ uint32_t slice_sum(const uint32_t* s_t, int t0, int t1)
{
    uint32_t s = 0;
    for (int t = t0; t < t1; ++t) s = add_sat(s, s_t[t]);
    return s;
}

// Replaces those counts by the tiles' starts, the first one's being start.
__host__ __device__ __forceinline__ void slice_starts(uint32_t* s_t, int t0, int t1, uint32_t start)
{
    for (int t = t0; t < t1; ++t) {
        const uint32_t c = s_t[t];
        s_t[t] = start;
        start = add_sat(start, c);
    }
}

// The run [x, y) of a tile whose instances start at a and end before b, clamped
// to a list of `capacity` < 2^32 - 1 slots; empty runs are (0, 0).
__host__ __device__ __forceinline__ uint2 clamp_run(uint32_t a, uint32_t b, uint32_t capacity)
{
    const uint32_t x = a < capacity ? a : capacity, y = b < capacity ? b : capacity;
    return x == y ? make_uint2(0u, 0u) : make_uint2(x, y);
}

// First slot of a group's instances in a tile, `before` of which precede them;
// `capacity` where the list has none.
__host__ __device__ __forceinline__ uint32_t first_slot(uint32_t start, uint32_t before,
                                                        uint32_t capacity)
{
    const uint32_t p = add_sat(start, before);
    return p < capacity ? p : capacity;
}

}  // namespace ts
