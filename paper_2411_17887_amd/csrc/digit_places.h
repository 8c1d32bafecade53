// Where a split pass on digits (sort.hip) stores a key, as byte offsets in the destination array, and how large a bucket may be
// that one workgroup sorts.  Plain C++: a CPU test compiles this file on its own.
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

// A pass on the top digit and a workgroup per bucket take the place of the other passes over n keys if no bucket has more keys than
// this.  The workgroup with the largest bucket is what the sort then waits for: it holds 24,576 keys, but takes longer for them
// than the passes do for few keys in all.  (us for n keys / pairs with m of them in one bucket, by passes and by a pass and
// buckets, the bucket's keys in order, which are the slowest: n = 20,000 m = 7000 31, 30.6 / 37, 36.7, m = 9000 31, 34.7 / 37, 42.0; 131,072 8000 38, 36.1 /
// 44, 44.1, 12,000 38, 40.9 / 44, 49.8; 262,144 10,000 43, 39.7 / 50, 48.5, 14,000 43, 45.5 / 50, 56.1; 400,000 12,000 48, 44.2 / 56, 54.4; 600,000 14,000 52,
// 48.2 / 65, 60.5, 20,000 52, 56.2 / 65, 71.8; 10^6 20,000 62, 59.2 / 76, 75.8, 24,000 62, 68.5 / 76, 89.4; 2 x 10^6 24,000 80, 74.9 / 88, 95.2.)
DIGIT_PLACES_FN uint32_t bucket_limit(uint64_t n, uint32_t capacity)
{
    const uint64_t limit = 6144u + n / 80u;
    return limit < capacity ? (uint32_t)limit : capacity;
}

// n keys that differ in so many bits of those that make the bins of a workgroup: are there as many bins as keys?  (Fewer come only from
// few bits, which two passes sort: us by passes / by bins, buckets or a whole sort of 1.14 to 1.9 keys to a bin, 5000 keys on 12 bits 8.4 / 9.4, pairs 11.2 / 11.8; 1.5 million keys on
// 20 40.7 / 42.2, 2.4 million on 21 52.0 / 54.1, 3.5 million 58.9 / 62.5, 5 million pairs on 22 92.7 / 99.5; of 0.7 to 1.07, 7000 on 13 9.8 / 9.6, pairs 13.0 / 12.7; 1.6 million
// on 21 42.0 / 42.1, pairs 53.8 / 52.9, 4.4 million on 22 65.0 / 66.3, pairs 84.2 / 82.1.)
DIGIT_PLACES_FN bool bins_suffice(uint32_t n, uint32_t bits) { return bits >= 32u || n <= 1u << bits; }

#endif
