// Where a split pass on digits (sort.hip) stores a key, as byte offsets in the destination array.  Plain C++: a CPU test
// compiles this file on its own.
//
// A tile's keys lie in order in LDS, those of a digit from place `start` on, `count` of them; `before` keys of the array go
// in front of the first.  The key at place i of the tile goes to byte 4 * (before + i - start): a base per digit plus 4 i.
// The base may be "negative": before < start where a look-back gave up, here or in an earlier tile or pass, so it is taken
// modulo the width of Place, in which adding 4 i brings it back.  (A difference taken in 32 bits and widened afterwards
// would put a 64-bit place 2^34 bytes too high.)
#ifndef TCUSCAN_DIGIT_PLACES_H
#define TCUSCAN_DIGIT_PLACES_H

#include <stdint.h>

#ifdef __HIPCC__
#define DIGIT_PLACES_FN __host__ __device__ __forceinline__
#else
#define DIGIT_PLACES_FN inline
#endif

// Place: uint32_t below 2^30 - 1 keys, uint64_t from there.
template <class Place> DIGIT_PLACES_FN Place digit_base(Place before, uint32_t start) { return (before - (Place)start) * 4u; }
template <class Place> DIGIT_PLACES_FN Place digit_place(Place base, uint32_t i) { return base + 4u * i; }

// The digit's range [before, before + count) lies inside an array of n keys, whatever the look-back returned.
template <class Place> DIGIT_PLACES_FN bool digit_range_fits(Place before, uint32_t count, uint32_t n)
{
    return before <= n && count <= n - (uint32_t)before;
}

#endif
