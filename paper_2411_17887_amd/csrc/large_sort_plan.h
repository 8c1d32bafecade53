// What a sort by two passes and small buckets (sort.hip) decides before its first launch: how many buckets, where in its scratch everything lies, and from which
// sums on a sample and the buckets' counts say that the keys crowd.  Plain C++: a CPU test compiles this file on its own.
#ifndef TCUSCAN_LARGE_SORT_PLAN_H
#define TCUSCAN_LARGE_SORT_PLAN_H

#include <math.h>
#include <stddef.h>
#include <stdint.h>

namespace large_sort {

constexpr int kDigits = 256, kMaxPasses = 4;
constexpr uint32_t kTables = 8;                                             // of counts, added up by several workgroups each
constexpr uint32_t kPassTile = 16384, kHugeTile = 8192;                     // keys of a workgroup in a pass
constexpr uint32_t kBucketMean = 4700;                                      // keys of a bucket on average, at most
constexpr uint32_t kSmallMost = 5120, kLargeMost = 10240;                   // keys of a bucket that a workgroup of four wavefronts sorts, of eight
constexpr uint32_t kHugeMost = 1u << 18;                                    // keys of a bucket that is sorted by two passes of its own
constexpr int kLogLeast = 13, kLogMost = 14;
constexpr uint32_t kSampleQuads = 2048, kSample = 4 * kSampleQuads;
constexpr size_t kFew = (size_t)3 << 23, kMost = (size_t)kBucketMean << kLogMost;

// What the kernels find out, in the scratch.
struct Found {
    uint32_t split;                       // are there buckets?
    uint32_t tried;                       // the sample says so
    uint32_t large;                       // buckets of more than kSmallMost keys, up to kLargeMost
    uint32_t huge;                        // tiles of buckets of more
    uint32_t work;                        // thousands (2^10) of keys that these read
    uint32_t pad[3];
    uint32_t top[kDigits];                // counts of the first pass's digit
    uint32_t start[1u << kLogMost];
    uint32_t large_at[1u << kLogMost];    // which buckets
};
static_assert(sizeof(Found) % 16 == 0, "16-byte boundaries");

struct Plan {
    int log, low;                         // 2^log buckets; the second pass's bits of it
    uint32_t most_tiles;                  // of the second pass: a chain per range
    uint32_t huge_tiles;                  // places in the list of huge buckets' tiles
    uint32_t huge_work;                   // thousands (2^10) of keys that these may read, each tile its whole bucket: as many as half the array's
    size_t found, counts, ranges, huge, status, end;                        // words from the scratch's first 16-byte boundary on
    // a sample in which ... crowds: one bucket has more than huge_most keys, a 256th of all buckets more than wide_most, buckets with more than some_most
    // have work for more than work_most, or fewer than few_most buckets have a first key of a group of four
    uint32_t some_most, huge_most, wide_most, work_most, few_most;
};

inline int buckets_log(size_t n)
{
    int log = kLogLeast;
    while ((n >> log) > kBucketMean) ++log;
    return log;
}
// The bits that are left are enough for bins, and there are four passes to do otherwise (with three, an odd number starts from a copy).
inline bool wanted(size_t n, int bits) { return n >= kFew && n <= kMost && bits > 24 && bits >= buckets_log(n) + 12; }

inline Plan plan(size_t n, bool vals)
{
    Plan p;
    p.log = buckets_log(n);
    p.low = vals ? (p.log + 2) / 2 : p.log / 2;
    const size_t buckets = (size_t)1 << p.log;
    p.most_tiles = (uint32_t)((n + kPassTile - 1) / kPassTile + ((size_t)1 << (p.log - p.low)));
    p.huge_tiles = (uint32_t)(n / kLargeMost + 4) & ~3u;                    // (each reads more than kLargeMost keys)
    p.huge_work = (uint32_t)(n / 2 >> 10);
    p.found = kTables * kMaxPasses * kDigits + kMaxPasses;                  // (behind digit counts and tickets)
    p.counts = p.found + sizeof(Found) / 4;
    p.ranges = p.counts + kTables * buckets;
    p.huge = p.ranges + (size_t)4 * p.most_tiles;
    p.status = p.huge + p.huge_tiles;
    p.end = p.status + (size_t)kMaxPasses * kDigits * p.most_tiles;
    const double sample = (double)kSample, per_key = sample / (double)n;
    p.some_most = (uint32_t)(2.0 * per_key * kLargeMost) + 8u;              // twice the largest that eight wavefronts sort, and eight: even keys do not come to it by chance
    p.huge_most = (uint32_t)(0.8 * per_key * kHugeMost);
    p.wide_most = (uint32_t)(0.9 * per_key * kLargeMost * (double)(buckets / kDigits));           // (keys that crowd gently: bell-shaped)
    p.work_most = kSample / 2;
    // as few buckets with first keys of a group as if they were huge
    const double used = (double)n / (double)kLargeMost;
    p.few_most = (uint32_t)(used * (1.0 - exp(-(double)kSampleQuads / used)));
    return p;
}

// Work for the passes over a huge bucket, in keys read per key of the sample or of the bucket: each of its tiles reads all of it.
constexpr uint32_t tiles_of(uint32_t size) { return (size + kHugeTile - 1) / kHugeTile; }

}  // namespace large_sort

#endif
