// Split passes on digits of up to eight bits: Blelloch's reduction of radix sort to prefix sums with 256 buckets instead
// of two.  A key goes to
//     (keys of the whole array with a smaller digit) + (keys with the same digit in front of it)
// and the second term is a prefix sum of "digit is d" flags taken at four levels, as everywhere in this library:
//     row of 64 keys   lanes with the same digit in front of this one: eight ballots narrow the wavefront down to them
//     wavefront        256 running counters in LDS, one row after the other
//     workgroup        the counters of the wavefronts, added up digit by digit
//     array            one status word per tile and digit, published and looked up as in the scan kernels' carry chain
// (the published scheme of least-significant-digit passes with a decoupled look-back per digit: Merrill and Garland 2016,
// Adinets and Merrill, "Onesweep", 2022).  By passes alone a full sort is
// four of 8 bytes per key (16 with payloads) and one reading of the keys for the first term.
//
// Sorts of up to 6,055,225 keys on more than 16 bits (up to 16384 keys on more than 8) do with one pass on the top eight bits if the 256
// buckets then are small enough for a workgroup each, which sorts its bucket by the other bits in LDS (partition, then local sorts, as in
// Stehle and Jacobsen, "A Memory Bandwidth-Efficient Hybrid Radix Sort on GPUs", 2017): whether they do is seen on the device, and
// where they do not, that first pass is the least significant one and the others follow (random keys, us in four passes / with
// buckets: 100,000 36.6 / 24.4, 10^6 61.6 / 34.4, with payloads 76.0 / 42.6, 2^22 104 / 61, with payloads 120 / 73; keys that do
// not split, 10^6 equal ones 55.8 / 57.6, normally distributed floats 61.5 / 62.5, 2^22 103.7 / 103.4).  Up to kBlockSortFew keys one workgroup does
// everything: one launch, keys and payloads read and written once.  Sorts of 3 * 2^23 to 77,004,800 keys do with two passes in the same way (2^26
// random keys 664 -> 513 us).

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/tcuscan.h"
#include "digit_places.h"
#include "large_sort_plan.h"
#include "wave_ops.h"

// tcuscan.hip: clears `bytes` bytes on the stream; the process-wide chain policy, the look-back's poll limit and the tile
// that a test keeps silent
extern "C" hipError_t tcuscan_internal_fill(void *d, size_t bytes, hipStream_t s);
extern "C" void tcuscan_internal_chain_knobs(unsigned *ticket, unsigned *spin_limit, unsigned *mute_tile);

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
typedef uint64_t CounterQuad __attribute__((may_alias));   // four 16-bit counters in LDS

constexpr int kDigits = large_sort::kDigits;
constexpr int kMaxPasses = large_sort::kMaxPasses;

struct Digit { int shift, width; };                        // digit = (key >> shift) & (2^width - 1), width 1 .. 8
struct Passes { int count; Digit digit[kMaxPasses]; };

__device__ __forceinline__ uint32_t digit_of(uint32_t key, Digit g) { return __builtin_amdgcn_ubfe(key, (uint32_t)g.shift, (uint32_t)g.width); }

constexpr unsigned kAndXnor = 0x90;        // truth table of a & ~(b ^ c)

// The lanes whose digit agrees with this lane's in every bit, from a ballot per bit: eight are 36 vector instructions.
template <int BITS> __device__ __forceinline__ void same_digit_by_ballots(uint32_t d, uint32_t &lo, uint32_t &hi)
{
    uint32_t sign[BITS];
    uint64_t ones[BITS];
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
        sign[b] = (uint32_t)__builtin_amdgcn_sbfe((int)d, b, 1);                           // the bit in all 32 places
        asm("" : "+v"(sign[b]));                           // (kept: else it is taken out of the digit once more for the compare)
        ones[b] = __builtin_amdgcn_ballot_w64(sign[b] != 0u);
    }
    lo = ~((uint32_t)ones[0] ^ sign[0]);
    hi = ~((uint32_t)(ones[0] >> 32) ^ sign[0]);
#pragma unroll
    for (int b = 1; b < BITS; ++b) {
        lo = __builtin_amdgcn_bitop3_b32(lo, (uint32_t)ones[b], sign[b], kAndXnor);
        hi = __builtin_amdgcn_bitop3_b32(hi, (uint32_t)(ones[b] >> 32), sign[b], kAndXnor);
    }
}

// rank[r]: keys of the wavefront with the same digit in front of key r of this lane (rows of 64 keys, lane order inside
// a row); counters[d] (this wavefront's, zero before): its keys with digit d.
// MASKS: every other row learns its lanes of equal digits from LDS instead, a mask of 64 bits per digit (`masks`, zero before and
// after) that the lanes set their bits in: LDS and vector unit take turns at being busy.  A workgroup alone on its compute
// unit, which waits for nothing but its instructions, gains (16,000 keys 32.4 -> 29.1 us; all rows by masks 34.7, two of three
// 30.7); the passes over an array, which wait for their stores, do not.
// `valid`: the lane's keys from row ceil(valid / 64) on are past the end -- with the highest digit, behind everything -- and set
// no bits: lanes that add to one mask go one after the other (16,000 equal keys: 30 us by ballots, 45 with masks, 30 with the lanes
// of the first one's digit left out).
template <int ITEMS, bool MASKS = false, int BITS = 8>
__device__ __forceinline__ void rank_rows(const uint32_t (&key)[ITEMS], Digit g, uint16_t *counters, uint32_t (&rank)[ITEMS], uint64_t *masks = nullptr, int valid = 64 * ITEMS)
{
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const uint32_t d = digit_of(key[r], g);
        const bool by_mask = MASKS && r % 2 == 0;
        uint32_t lo, hi;
        if (by_mask) {
            // (the lanes that agree with the first one need no bits: equal keys)
            const uint32_t d0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)d);
            const uint64_t as_first = __ballot(d == d0);
            if (d != d0 && 64 * r < valid) atomicOr((unsigned long long *)&masks[d], 1ull << (threadIdx.x & 63u));
            wavefront_sync();
            const uint64_t m = d == d0 ? as_first : masks[d];
            lo = (uint32_t)m;
            hi = (uint32_t)(m >> 32);
        } else {
            same_digit_by_ballots<BITS>(d, lo, hi);
        }
        const uint32_t before = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u));
        const uint32_t all = (uint32_t)(__builtin_popcount(lo) + __builtin_popcount(hi));
        const uint32_t prev = counters[d];
        wavefront_sync();                                  // (every lane has read before the first of its group writes)
        if (before == 0u) {
            counters[d] = (uint16_t)(prev + all);
            if (by_mask) masks[d] = 0ull;
        }
        wavefront_sync();
        rank[r] = prev + before;
    }
}

// Offsets in the ordered tile are 16 bits: of bytes up to 16384 keys, of words beyond.
template <int ITEMS, int W> constexpr uint32_t kUnit = ITEMS * 64 * W <= 16384 ? 4u : 1u;

// The counters of W wavefronts -> offset (in kUnit) of the first (wavefront, digit) place in the ordered tile; threads 0 ..
// 255, one digit each, return the tile's keys with their digit (`count`) and the place of the first (`start`).  `early`
// is called with the count as soon as it is known.
template <int W, uint32_t UNIT, class Early>
__device__ __forceinline__ void scan_counters(uint16_t (*counters)[kDigits], uint32_t *s_part, uint32_t &count, uint32_t &start, Early early)
{
    const int d = threadIdx.x, lane = d & 63, wave = d >> 6;
    count = start = 0u;
    uint32_t inc = 0u;
    if (d < kDigits) {
#pragma unroll
        for (int w = 0; w < W; ++w) count += counters[w][d];
        early(count);
        inc = wave_inclusive_scan(count);
        if (lane == 63) s_part[wave] = inc;
    }
    __syncthreads();
    if (d < kDigits) {
        start = inc - count;
        for (int w = 0; w < wave; ++w) start += s_part[w];
        uint32_t at = UNIT * start;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const uint32_t c = counters[w][d];
            counters[w][d] = (uint16_t)at;
            at += UNIT * c;
        }
    }
    __syncthreads();
}

// Key r of this lane to its place in the ordered tile; at[r]: its rank, then the byte offset of the place.
template <int ITEMS, uint32_t UNIT>
__device__ __forceinline__ void put_in_order(const uint32_t (&key)[ITEMS], Digit g, const uint16_t *counters, uint32_t *order, uint32_t (&at)[ITEMS])
{
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        uint32_t k = key[r];
        asm("" : "+v"(k));                                 // (the digit's address is not kept from the ranking on: 16 registers)
        at[r] = UNIT == 4u ? 4u * at[r] + counters[digit_of(k, g)] : 4u * (at[r] + counters[digit_of(k, g)]);
        *(uint32_t *)((char *)order + at[r]) = k;
    }
}

// ------------------------------------------------------------------------- digit histograms

struct HistArgs {
    const uint32_t *keys, *vals;
    uint32_t *keys_copy, *vals_copy;      // null, or where the keys (and payloads) are copied for an odd number of passes
    uint32_t *hist;                       // [table][pass][digit], zero before unless `own`
    uint32_t tables;
    uint32_t *status;                     // status words of all passes, zeroed here (16-byte aligned)
    uint64_t n, status_quads;
    Passes P;
    bool stream;                          // as in PassArgs
    bool own;                             // no more workgroups than tables
    bool from_end;                        // the last key first
};

// All passes' digit counts in one reading of the keys: the counts do not change when keys change places.  A digit has
// 16 counters in LDS, chosen by lane: equal digits in a wavefront (the common case in the high bytes of small keys)
// meet four at a time and not all 64, and random ones meet less often in a bank.  What bounds it is the four LDS
// additions per key.  2^22 keys in all, payloads on top: 8 counters per digit and workgroups of 256 cost 13 us more, 32
// counters (one workgroup per compute unit) 2 us more; 1024 workgroups instead of 512 add as much again in the final
// additions to the same 1024 words.  Large arrays without a copy are read from the last key on: those written last may still be in the memory-side cache (2^26 normally
// distributed floats, which take four passes, 776 -> 762 us, 3 * 2^23 no change; with the copy that an odd number of passes starts from, 2^24 pairs on 24 bits 284 -> 289).
constexpr int kHistCopies = 16, kHistThreads = 1024, kHistGrid = 512;
// The workgroups add up in one of eight tables -- additions to one word from all dies go one after the other, 27 ns each: 2^22
// keys 14.5 -> 7 us -- and up to eight workgroups have one each, which then needs no clearing in front (HistArgs::own).
constexpr uint32_t kTables = large_sort::kTables, kTableWords = kMaxPasses * kDigits;
template <class T> __device__ __forceinline__ T sum_of_tables(const T *hist, uint32_t tables)
{
    T x[kTables], sum = T{};
#pragma unroll
    for (uint32_t t = 0; t < kTables; ++t) x[t] = t < tables ? hist[t * (kTableWords * sizeof(uint32_t) / sizeof(T))] : T{};     // all in flight together
#pragma unroll
    for (uint32_t t = 0; t < kTables; ++t) sum += x[t];
    return sum;
}
constexpr int kHistWords = kMaxPasses * kDigits * kHistCopies;
__device__ __forceinline__ void digit_histograms(const HistArgs &H, uint32_t *s_hist)
{
    for (int i = threadIdx.x; i < kHistWords; i += kHistThreads) s_hist[i] = 0u;
    __syncthreads();
    const uint64_t stride = (uint64_t)gridDim.x * kHistThreads, t0 = (uint64_t)blockIdx.x * kHistThreads + threadIdx.x;
    const uint32_t copy = threadIdx.x & (kHistCopies - 1);
    auto add = [&](uint32_t key) {
#pragma unroll
        for (int p = 0; p < kMaxPasses; ++p)
            if (p < H.P.count) atomicAdd(&s_hist[((uint32_t)p * kDigits + digit_of(key, H.P.digit[p])) * kHistCopies + copy], 1u);
    };
    const uint64_t quads = H.n / 4;
    const u32x4 *keys4 = (const u32x4 *)H.keys;
    const auto at = [=](uint64_t i) { return H.from_end ? quads - 1 - i : i; };
    // the next four keys are on their way while four are counted
    u32x4 next = {0u, 0u, 0u, 0u};
    auto load = [&](uint64_t i) {
        if (i < quads) next = H.stream ? __builtin_nontemporal_load(keys4 + at(i)) : keys4[at(i)];
    };
    load(t0);
    for (uint64_t i = t0; i < quads; i += stride) {
        const u32x4 k = next;
        load(i + stride);
        if (H.keys_copy) ((u32x4 *)H.keys_copy)[at(i)] = k;
        add(k[0]); add(k[1]); add(k[2]); add(k[3]);
    }
    if (t0 < (H.n & 3u)) {
        const uint64_t i = 4 * quads + t0;
        const uint32_t k = H.keys[i];
        if (H.keys_copy) H.keys_copy[i] = k;
        add(k);
    }
    if (H.vals_copy)
        for (uint64_t i = t0; i < H.n; i += stride) H.vals_copy[i] = H.vals[i];
    for (uint64_t i = t0; i < H.status_quads; i += stride) ((u32x4 *)H.status)[i] = u32x4{0u, 0u, 0u, 0u};
    __syncthreads();
    for (int i = threadIdx.x; i < H.P.count * kDigits; i += kHistThreads) {
        uint32_t sum = 0u;
#pragma unroll
        for (int c = 0; c < kHistCopies; ++c) sum += s_hist[i * kHistCopies + c];
        uint32_t *at = &H.hist[(blockIdx.x % H.tables) * kTableWords + i];
        if (H.own) *at = sum;
        else if (sum) atomicAdd(at, sum);
    }
}
__global__ __launch_bounds__(kHistThreads) void digit_histograms_kernel(HistArgs H)
{
    __shared__ uint32_t s_hist[kHistWords];
    digit_histograms(H, s_hist);
}

// ------------------------------------------------------------------------- one pass over the array

// Status words, one per tile and digit: 2 state bits on top (0 = not published), the value below.  The largest value is no
// count: a tile that could not learn what lies in front of it publishes it, and every sum it goes into is one that lies
// in front of nothing (digit_range_fits; a state of its own, looked at word by word, cost 26 us of a sort of 2^26 keys and 7 of
// one of 2^22 pairs).  32-bit words hold the counts of fewer than 2^30 - 1 keys, 64-bit words all there are.
constexpr uint32_t kCountOfTile = 1u, kCountUpToTile = 2u;
template <class Word> struct StatusWord {
    static constexpr int kStateAt = 8 * (int)sizeof(Word) - 2;
    static constexpr Word kUnknown = ((Word)1 << kStateAt) - 1;
    static __device__ __forceinline__ Word make(uint32_t state, Word value) { return ((Word)state << kStateAt) | (value < kUnknown ? value : kUnknown); }
    static __device__ __forceinline__ uint32_t state(Word w) { return (uint32_t)(w >> kStateAt); }
    static __device__ __forceinline__ Word value(Word w) { return w & kUnknown; }
};

constexpr int kBlockWaves = 16, kBlockItems = 24;
constexpr size_t kBlockCapacity = (size_t)64 * kBlockWaves * kBlockItems;      // keys of a bucket that one workgroup sorts
constexpr size_t kBlockSortMax = 16384;                                         // keys of a sort that one workgroup does, if it must

// What the first pass finds out: have the keys gone into buckets by their top digit, and where does each begin.
enum : uint32_t { kNotSplit = 0u, kSplit = 1u };
struct Buckets { uint32_t split; uint32_t start[kDigits]; };

// Keys from `base` on, `keys` of them (0: no tile), of a range; the range's first tile has `head`.
struct TileOfRange { uint32_t base, keys, range, head; };

struct PassArgs {
    const uint32_t *keys, *vals;
    uint32_t *keys_out, *vals_out;
    void *status;                         // this pass's status words (zero before)
    const uint32_t *hist;                 // this pass's digit counts over the whole array, to be summed over the tables
    uint32_t tables;
    uint32_t *ticket;                     // null, or the counter the workgroups draw their tile from (zero before)
    uint32_t *fault;                      // the workspace's fault word
    uint64_t n;
    uint32_t spin_limit;
    uint32_t mute_tile;                   // test hook: the tile with this index publishes nothing
    Digit digit;
    bool stream;                          // the arrays do not fit the memory-side cache: keys are read around it
    // Sorts that may take one pass and buckets (null otherwise).  First pass: the counts of the top digit, which is taken if no
    // bucket has more than bucket_max keys; later passes have nothing to do then.
    const uint32_t *top_hist;
    Buckets *buckets;
    Digit top;
    uint32_t bucket_max;
    // Sorts that may take two passes and small buckets (null otherwise): whether they do, and if so: the first goes by `top` and top_hist, one
    // table; the second goes by `top` in each range of keys that the first has made, whose tiles `ranges` lists and whose buckets begin at
    // range_start; later passes do the huge buckets, if there are any.
    const TileOfRange *ranges;
    const uint32_t *range_start;
    const uint32_t *split;
    // Later passes of those: huge buckets, by `top`.
    const large_sort::Found *found;
    const uint32_t *huge, *sizes;
    uint32_t huge_tiles;
};

// What kernels in front have written, the same for all lanes: one scalar load, which no vector load in front of it delays.
template <class T> __device__ __forceinline__ T uniform_load(const T *p) { return *(const __attribute__((address_space(4))) T *)(uintptr_t)p; }

enum PassRole { kPlainPass, kChoosingPass, kLaterPass, kFirstOfTwo, kSecondOfTwo, kAfterTwo };

template <int ITEMS>
__device__ __forceinline__ void load_rows(const uint32_t *src, uint32_t first, uint32_t valid, bool whole, bool stream, uint32_t fill, uint32_t (&x)[ITEMS])
{
    if (whole && stream) {                                 // straight-line loads
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) x[r] = __builtin_nontemporal_load(src + first + 64u * r);
    } else if (whole) {
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) x[r] = src[first + 64u * r];
    } else {
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) x[r] = first + 64u * r < valid ? src[first + 64u * r] : fill;
    }
}

// Predecessors asked for at a time: 4.  Every word of a window is 1 KiB of traffic over the 256 digits, and words behind
// the nearest prefix are asked for in vain (2^26 keys: 4 819, 2 831, 8 877, 16 1074 us per sort).
constexpr int kWindow = 4;

// The status words of digit `d` in tiles t, t - 1, ... (a tile before the first counts as "nothing up to here").  Offsets
// are 32 bits: the words of 2^32 keys are less than 2^32 bytes.
template <class Word>
__device__ __forceinline__ void request_window(const Word *status, uint32_t d, int32_t t, Word (&w)[kWindow])
{
#pragma unroll
    for (int u = 0; u < kWindow; ++u)
        w[u] = t - u >= 0 ? __hip_atomic_load((const Word *)((const char *)status + ((uint32_t)(t - u) * kDigits + d) * (uint32_t)sizeof(Word)),
                                              __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                          : StatusWord<Word>::make(kCountUpToTile, 0u);
}

// Keys with this thread's digit in front of the tile (those with smaller digits, anywhere, among them: tile 0 starts
// from there); kUnknown or more if this wait or one it depends on gave up.  `w` holds the window that was requested at tile
// t = tile - 1.
template <class Word>
__device__ __forceinline__ Word digit_look_back(const Word *status, uint32_t d, int32_t t, Word (&w)[kWindow], const PassArgs &A)
{
    using S = StatusWord<Word>;
    Word sum = 0u;
    uint32_t spins = 0u;
    for (;;) {
        bool found = false, waiting = false;
#pragma unroll
        for (int u = 0; u < kWindow; ++u) {
            if (!found && !waiting) {
                const uint32_t state = S::state(w[u]);
                if (state == 0u) waiting = true;
                else { sum += S::value(w[u]); --t; found = state == kCountUpToTile; }
            }
        }
        if (found) return sum;
        if (waiting) {
            if (++spins > A.spin_limit) {                  // never in correct operation: give up instead of hanging
                __hip_atomic_store(A.fault, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                return S::kUnknown;
            }
            __builtin_amdgcn_s_sleep(1);
        }
        request_window(status, d, t, w);
    }
}

// What bounds a pass: writing 256 ranges of a tile each in pieces of 64 keys (2^26 keys: 150 us a pass; with the same
// tiles written back in a row 111 us, and without the ranking on top 100 us, which is the device's copy rate; the
// carry chain is 12 us of it).  The tile is therefore as large as two workgroups per compute unit allow: 16 wavefronts
// of 16 rows, 73 KiB of LDS, and the register allocator is held to 64 registers so that all 32 wavefronts are resident
// (at 101 registers one workgroup was, 215 us a pass); 8192 keys per tile: 18 us a pass more, 12288: 15 us more.  The form for
// 2^30 keys and more keeps 64-bit words and places and takes 80 to 82 registers, which is one workgroup: 2^30 + 12345 keys
// 16.4 ms per sort, with payloads 25.1 (two-bit passes took 37.6 and 80.1), where 16 sorts of 2^26 keys take 12.2.
template <int W, int ITEMS, class Place> struct PassLds {
    uint32_t order[64 * W * ITEMS];
    alignas(16) uint16_t cnt[W][kDigits];
    Place dest[kDigits];
    uint32_t part[4], abort;
};
// The tile that a workgroup takes.
__device__ __forceinline__ uint32_t take_tile(const PassArgs &A, uint32_t *slot)
{
    if (!A.ticket) return blockIdx.x;
    if (threadIdx.x == 0) *slot = __hip_atomic_fetch_add(A.ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const uint32_t tile = (uint32_t)__builtin_amdgcn_readfirstlane((int)*slot);
    __syncthreads();
    return tile;
}
template <int W, int ITEMS, bool VALS, class Word, PassRole ROLE>
__device__ __forceinline__ void digit_pass(const PassArgs &A, PassLds<W, ITEMS, Word> &s, uint32_t tile)
{
    using S = StatusWord<Word>;
    using Place = Word;                    // byte offsets in the destination: 32 bits hold those of 2^30 keys
    constexpr int kThreads = 64 * W;
    constexpr uint32_t kTile = kThreads * ITEMS;
    static_assert(W >= 4 && kTile <= 16384u, "one thread per digit; byte offsets inside a tile are 16 bits");
    auto &s_order = s.order;
    auto &s_cnt = s.cnt;
    auto &s_dest = s.dest;
    uint32_t *s_part = s.part;
    static_assert(alignof(PassLds<W, ITEMS, Word>) >= alignof(CounterQuad), "counters cleared four at a time");

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (tid == 0) s.abort = 0u;
    uint64_t base = (uint64_t)tile * kTile;
    bool head = tile == 0u, of_range = false;              // the first of a chain; a chain per range
    uint32_t valid = A.n - base < kTile ? (uint32_t)(A.n - base) : kTile, range = 0u;
    Digit g = A.digit;
    if constexpr (ROLE == kSecondOfTwo) {                  // (as many workgroups as there may be tiles)
        const u32x4 at_range = uniform_load((const u32x4 *)(A.ranges + tile));
        of_range = uniform_load(A.split) != kNotSplit;
        if (of_range) {
            base = at_range[0];
            valid = at_range[1];
            range = at_range[2];
            head = at_range[3] != 0u;
            g = A.top;
        }
        if (of_range ? valid == 0u : base >= A.n) return;
    }
    // ---- the keys, in rows of 64 per wavefront; keys past the end have the highest digit and come last among its keys
    const uint32_t first = (uint32_t)wave * 64u * ITEMS + (uint32_t)lane;
    uint32_t key[ITEMS], at[ITEMS];
    load_rows<ITEMS>(A.keys + base, first, valid, valid == kTile, A.stream, ~0u, key);
    ((CounterQuad *)s_cnt[wave])[lane] = 0u;
    const uint32_t *hist = A.hist;
    if constexpr (ROLE == kChoosingPass) {
        // every wavefront looks at the counts: is the largest bucket small enough?
        const u32x4 c = sum_of_tables((const u32x4 *)A.top_hist + lane, A.tables);
        const bool fits = c[0] <= A.bucket_max && c[1] <= A.bucket_max && c[2] <= A.bucket_max && c[3] <= A.bucket_max;
        const bool split = __ballot(!fits) == 0ull;
        if (tile == 0u && tid == 0) A.buckets->split = split ? kSplit : kNotSplit;
        if (split) { g = A.top; hist = A.top_hist; }
    }
    uint32_t tables = A.tables;
    if constexpr (ROLE == kFirstOfTwo) {
        if (uniform_load(A.split) != kNotSplit) { g = A.top; hist = A.top_hist; tables = 1u; }
    }
    wavefront_sync();
    rank_rows<ITEMS>(key, g, s_cnt[wave], at);
    __syncthreads();

    // ---- counters -> places; the chain sets out (thread d: digit d)
    Word *column = (Word *)A.status + (tid & (kDigits - 1));
    const bool has_digit = tid < 1 << g.width;             // (a digit of seven bits: nobody asks for the other 128 words.  138 -> 132 us a pass over 2^26 keys)
    const bool speaks = tile != A.mute_tile;
    Word win[kWindow];
    uint32_t count, start;
    scan_counters<W, kUnit<ITEMS, W>>(s_cnt, s_part, count, start, [&](uint32_t c) {
        if (!head && has_digit) {
            if (speaks) __hip_atomic_store(column + (size_t)tile * kDigits, S::make(kCountOfTile, c), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            request_window((const Word *)A.status, (uint32_t)tid, (int32_t)tile - 1, win);
        }
    });

    // ---- meanwhile the tile is put in order
    put_in_order<ITEMS, kUnit<ITEMS, W>>(key, g, s_cnt[wave], s_order, at);
    uint32_t val[VALS ? ITEMS : 1];
    if constexpr (VALS) {
        load_rows<ITEMS>(A.vals + base, first, valid, valid == kTile, A.stream, 0u, val);
    }

    // ---- the chain arrives: where the tile's keys of each digit go
    Word before = 0u;                                      // keys in front of the tile's first with this thread's digit
    if (of_range && head) {                                // (uniform over the workgroup)
        if (tid < 1 << g.width) before = A.range_start[(range << g.width) + (uint32_t)tid];
    } else if (head) {
        uint32_t h = 0u, inc = 0u;
        if (tid < kDigits) {
            h = sum_of_tables(hist + tid, tables);
            inc = wave_inclusive_scan(h);
            if (lane == 63) s_part[wave] = inc;
        }
        __syncthreads();
        if (tid < kDigits) {
            before = inc - h;
            for (int w = 0; w < wave; ++w) before += s_part[w];
            if constexpr (ROLE == kChoosingPass) A.buckets->start[tid] = (uint32_t)before;
        }
    } else if (has_digit) {
        before = digit_look_back((const Word *)A.status, (uint32_t)tid, (int32_t)tile - 1, win, A);
    }
    if (has_digit) {
        if (speaks) __hip_atomic_store(column + (size_t)tile * kDigits, S::make(kCountUpToTile, before + count), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_dest[tid] = digit_base<Place>(before, start);
        // Nothing is stored of a tile that does not know its places, nor, in the passes after one that left tiles out, of a
        // tile whose places the counts over the array do not hold.  (The counts of the last tile include its keys past the
        // end; its stores are bounded one by one.)
        if (!digit_range_fits<Place>(before, valid == kTile ? count : 0u, (uint32_t)A.n)) s.abort = 1u;
    }
    __syncthreads();
    if (s.abort) return;

    // ---- out: consecutive threads write consecutive places of a digit's range
    Place dst[VALS ? ITEMS : 1];
    char *kout = (char *)A.keys_out, *vout = (char *)A.vals_out;
    if (valid == kTile) {
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) {
            const uint32_t i = (uint32_t)tid + (uint32_t)r * kThreads, k = s_order[i];
            const Place to = digit_place(s_dest[digit_of(k, g)], i);
            *(uint32_t *)(kout + to) = k;
            if constexpr (VALS) dst[r] = to;
        }
    } else {
        for (int r = 0; r < ITEMS; ++r) {
            const uint32_t i = (uint32_t)tid + (uint32_t)r * kThreads, k = s_order[i];
            const Place to = digit_place(s_dest[digit_of(k, g)], i);
            if (i < valid && to / 4u < A.n) *(uint32_t *)(kout + to) = k;
            if constexpr (VALS) dst[r] = to;
        }
    }
    if constexpr (VALS) {
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) *(uint32_t *)((char *)s_order + at[r]) = val[r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) {
            const uint32_t i = (uint32_t)tid + (uint32_t)r * kThreads;
            if (valid == kTile || (i < valid && dst[r] / 4u < A.n)) *(uint32_t *)(vout + dst[r]) = s_order[i];
        }
    }
}
// Buckets of large sorts with more keys than a workgroup sorts in LDS (one value many times over, say): two stable passes on the nine or ten bits of half a bucket's
// other bits each, in the launches of the third and fourth pass, which have nothing else to do then.  A bucket's tiles know of each other as in spread_kernel: each counts the
// digits of all the others' keys itself, so no tile waits for another.  That is a reading of the whole bucket per tile, which is why there is a limit to their
// sizes (large_sort::kHugeMost) and to what they read in all (Plan::huge_work: all keys of 3 * 2^23 in such buckets, three tiles each, 443 us, four passes 299).  (us per sort, four
// passes alone / four passes after the counts / now: 2^26 keys, one in 2000 the same, 764 / 844 / 640; 3 * 2^23 289 / 335 / 278, pairs 446 / 494 / 380.)
struct HugeLds {
    static constexpr int kWaves = 16, kItems = large_sort::kHugeTile / (64 * kWaves), kBits = 10;
    static constexpr uint32_t kCount = 1u << kBits;
    uint32_t order[large_sort::kHugeTile];
    alignas(16) uint16_t cnt[kWaves][kCount];
    uint32_t other[2][kCount];            // digit counts of the bucket's tiles in front and behind
    uint32_t part[2][kWaves];
};
static_assert(64 * HugeLds::kWaves == HugeLds::kCount, "a thread per digit");

// One key of each lane to the count of its digit or bucket, `one` each.  Where many lanes agree with the first one they are added at
// once: keys in order or equal would be added one after the other (2^24 keys in order: the counting kernel of large sorts 57 -> 16 us, the sample of equal ones 13 -> 8).
__device__ __forceinline__ void add_to_count(uint32_t *counts, uint32_t at, uint32_t one = 1u)
{
    const bool as_first = at == (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
    const uint64_t those = __ballot(as_first);
    const uint32_t all = (uint32_t)__builtin_popcountll(those);
    if (all < 16u) {
        atomicAdd(&counts[at], one);
    } else {
        const bool first = as_first && __builtin_amdgcn_mbcnt_hi((uint32_t)(those >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)those, 0u)) == 0u;
        if (!as_first || first) atomicAdd(&counts[at], first ? all * one : one);
    }
}

template <bool VALS>
__device__ __forceinline__ void huge_pass(const PassArgs &A, uint32_t tiles, HugeLds &s)
{
    constexpr int W = HugeLds::kWaves, ITEMS = HugeLds::kItems;
    constexpr uint32_t kThreads = 64 * W, kTile = large_sort::kHugeTile;
    const Digit g = A.top;
    tiles = tiles < A.huge_tiles ? tiles : A.huge_tiles;
    for (uint32_t t = blockIdx.x; t < tiles; t += gridDim.x) {
        uint32_t tid = threadIdx.x;
        asm volatile("" : "+v"(tid));                      // (no addresses are kept from one round to the next: registers)
        const uint32_t lane = tid & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
        const uint32_t first = wave * 64u * ITEMS + lane;
        const uint32_t entry = uniform_load(A.huge + t), bucket = entry & ((1u << large_sort::kLogMost) - 1u), base = (entry >> large_sort::kLogMost) * kTile;
        const uint32_t begin = uniform_load(&A.found->start[bucket]), size = uniform_load(A.sizes + bucket);
        const uint32_t valid = size - base < kTile ? size - base : kTile;
        const uint32_t *keys = A.keys + begin;
        uint32_t key[ITEMS], at[ITEMS];
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) key[r] = first + 64u * r < valid ? keys[base + first + 64u * r] : ~0u;
        for (uint32_t i = tid; i < sizeof(s.cnt) / 16u; i += kThreads) ((u32x4 *)s.cnt)[i] = u32x4{0u, 0u, 0u, 0u};
        s.other[0][tid] = s.other[1][tid] = 0u;
        __syncthreads();
        for (uint32_t i = tid; i < base; i += kThreads) add_to_count(s.other[0], digit_of(keys[i], g));
        for (uint32_t i = base + valid + tid; i < size; i += kThreads) add_to_count(s.other[1], digit_of(keys[i], g));
        rank_rows<ITEMS, false, HugeLds::kBits>(key, g, s.cnt[wave], at);
        __syncthreads();
        // ---- thread d: digit d, in the tile and in the bucket
        uint32_t count = 0u;
#pragma unroll 4
        for (int w = 0; w < W; ++w) count += s.cnt[w][tid];
        // (keys past the end of the last tile count as the highest digit)
        const uint32_t in_front = s.other[0][tid], all = in_front + s.other[1][tid] + count - (tid == (1u << g.width) - 1u ? kTile - valid : 0u);
        const uint32_t inc = wave_inclusive_scan(count), inc_all = wave_inclusive_scan(all);
        if (lane == 63u) { s.part[0][wave] = inc; s.part[1][wave] = inc_all; }
        __syncthreads();
        uint32_t start = inc - count, to = inc_all - all + in_front;
        for (uint32_t w = 0; w < wave; ++w) { start += s.part[0][w]; to += s.part[1][w]; }
        s.other[0][tid] = digit_base<uint32_t>(to, start);                  // (its own word: no other thread looks at it before the barrier)
#pragma unroll 4
        for (int w = 0; w < W; ++w) {
            const uint32_t c = s.cnt[w][tid];
            s.cnt[w][tid] = (uint16_t)start;
            start += c;
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) {
            at[r] += s.cnt[wave][digit_of(key[r], g)];
            s.order[at[r]] = key[r];
        }
        uint32_t val[VALS ? ITEMS : 1], dst[VALS ? ITEMS : 1];
        if constexpr (VALS) {
            const uint32_t *vals = A.vals + begin + base;
#pragma unroll
            for (int r = 0; r < ITEMS; ++r) val[r] = first + 64u * r < valid ? vals[first + 64u * r] : 0u;
        }
        __syncthreads();
        char *kout = (char *)(A.keys_out + begin), *vout = VALS ? (char *)(A.vals_out + begin) : nullptr;
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) {
            const uint32_t i = tid + (uint32_t)r * kThreads, k = s.order[i], place = digit_place(s.other[0][digit_of(k, g)], i);
            if (i < valid) *(uint32_t *)(kout + place) = k;
            if constexpr (VALS) dst[r] = place;
        }
        __syncthreads();
        if constexpr (VALS) {
#pragma unroll
            for (int r = 0; r < ITEMS; ++r) s.order[at[r]] = val[r];
            __syncthreads();
#pragma unroll
            for (int r = 0; r < ITEMS; ++r) {
                const uint32_t i = tid + (uint32_t)r * kThreads;
                if (i < valid) *(uint32_t *)(vout + dst[r]) = s.order[i];
            }
            __syncthreads();
        }
    }
}
template <int W, int ITEMS, bool VALS, class Word, PassRole ROLE = kPlainPass>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(sizeof(Word) == 4 ? 8 : 4))) void digit_pass_kernel(PassArgs A)
{
    if constexpr (ROLE == kAfterTwo) {
        __shared__ union { PassLds<W, ITEMS, Word> pass; HugeLds huge; } s;
        const u32x4 found = uniform_load((const u32x4 *)A.found);
        static_assert(offsetof(large_sort::Found, split) == 0 && offsetof(large_sort::Found, huge) == 12, "found[0], found[3]");
        if (found[0] != kNotSplit && found[3] == 0u) return;
        if (found[0] != kNotSplit) huge_pass<VALS>(A, found[3], s.huge);
        else digit_pass<W, ITEMS, VALS, Word, ROLE>(A, s.pass, take_tile(A, s.pass.part));
    } else {
        __shared__ PassLds<W, ITEMS, Word> s;
        if constexpr (ROLE == kLaterPass) {
            if (uniform_load(A.split) != kNotSplit) return;
        }
        digit_pass<W, ITEMS, VALS, Word, ROLE>(A, s, take_tile(A, s.part));
    }
}

// ------------------------------------------------------------------------- the pass in front of a small sort's buckets
//
// Up to kBlockSortMax keys are four tiles at most: every workgroup counts the top digit of the others' keys itself, in place of a
// launch in front and a carry chain.  Every bucket fits a workgroup, so there is nothing to choose.  (us, one workgroup / a
// counting launch, a pass and buckets / this and buckets: 9000 random keys 25 / 17.0 / 14.0, 16,000 32 / 17.2 / 14.7, pairs 39 / 20.7 / 17.8; 12,000 and 16,000
// keys below 2^24, all in one bucket, 25.5 / 28.9 / 26.1 and 31.6 / 34.5 / 31.0, half of them 25.9 / 29.8 / 21.0 and 31.9 / 35.4 / 25.0.)

struct SpreadArgs {
    const uint32_t *keys, *vals;
    uint32_t *keys_out, *vals_out;
    Buckets *buckets;
    uint32_t n;
    Digit top;
};
constexpr int kSpreadWaves = 16, kSpreadItems = 4;
constexpr uint32_t kSpreadTile = 64 * kSpreadWaves * kSpreadItems, kSpreadTiles = (uint32_t)(kBlockSortMax / kSpreadTile);
static_assert(kSpreadTiles * kSpreadTile == kBlockSortMax, "tiles of a small sort");

template <bool VALS>
__global__ __launch_bounds__(64 * kSpreadWaves) void spread_kernel(SpreadArgs A)
{
    constexpr int W = kSpreadWaves, ITEMS = kSpreadItems, kThreads = 64 * W;
    __shared__ uint32_t s_order[kSpreadTile];
    __shared__ __attribute__((aligned(16))) uint16_t s_cnt[W][kDigits];
    static_assert(__alignof__(s_cnt) >= alignof(CounterQuad), "cleared four counters at a time");
    __shared__ uint32_t s_other[2][kDigits];               // digit counts of the tiles in front and behind
    __shared__ uint32_t s_dest[kDigits];
    __shared__ uint32_t s_part[4];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t tile = blockIdx.x, first = (uint32_t)wave * 64u * ITEMS + (uint32_t)lane;
    auto keys_of = [&](uint32_t t) { const uint32_t at = t * kSpreadTile; return at >= A.n ? 0u : A.n - at < kSpreadTile ? A.n - at : kSpreadTile; };
    const uint32_t base = tile * kSpreadTile, valid = keys_of(tile);
    uint32_t key[ITEMS], at[ITEMS], other[kSpreadTiles - 1][ITEMS];
    load_rows<ITEMS>(A.keys + base, first, valid, valid == kSpreadTile, false, ~0u, key);
#pragma unroll
    for (uint32_t q = 0; q < kSpreadTiles - 1; ++q) {
        const uint32_t t = q + (q >= tile ? 1u : 0u), left = keys_of(t);
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) other[q][r] = first + 64u * r < left ? A.keys[t * kSpreadTile + first + 64u * r] : 0u;
    }
    ((CounterQuad *)s_cnt[wave])[lane] = 0u;
    if (tid < 2 * kDigits) s_other[tid / kDigits][tid % kDigits] = 0u;
    __syncthreads();
    rank_rows<ITEMS>(key, A.top, s_cnt[wave], at);
#pragma unroll
    for (uint32_t q = 0; q < kSpreadTiles - 1; ++q) {
        const uint32_t left = keys_of(q + (q >= tile ? 1u : 0u));
        uint32_t *counts = s_other[q >= tile ? 1 : 0];
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) {
            // (lanes that agree with the first one are added at once: lanes that add to one word go one after the other)
            const bool in = first + 64u * r < left;
            const uint32_t d = digit_of(other[q][r], A.top), d0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)d);
            const uint64_t as_first = __ballot(in && d == d0);
            if (lane == 0 && in) atomicAdd(&counts[d0], (uint32_t)__builtin_popcountll(as_first));
            if (in && d != d0) atomicAdd(&counts[d], 1u);
        }
    }
    __syncthreads();
    uint32_t count, start;
    scan_counters<W, kUnit<ITEMS, W>>(s_cnt, s_part, count, start, [](uint32_t) {});
    put_in_order<ITEMS, kUnit<ITEMS, W>>(key, A.top, s_cnt[wave], s_order, at);
    uint32_t val[VALS ? ITEMS : 1];
    if constexpr (VALS) load_rows<ITEMS>(A.vals + base, first, valid, valid == kSpreadTile, false, 0u, val);

    // ---- where the digits begin in the whole array, and this tile's part of each
    uint32_t all = 0u, inc = 0u;
    if (tid < kDigits) {
        // (the keys past the end of the last tile count as the highest digit)
        all = s_other[0][tid] + s_other[1][tid] + count - (tid == (1 << A.top.width) - 1 ? kSpreadTile - valid : 0u);
        inc = wave_inclusive_scan(all);
        if (lane == 63) s_part[wave] = inc;
    }
    __syncthreads();
    if (tid < kDigits) {
        uint32_t begin = inc - all;
        for (int w = 0; w < wave; ++w) begin += s_part[w];
        if (tile == 0u) A.buckets->start[tid] = begin;
        s_dest[tid] = digit_base<uint32_t>(begin + s_other[0][tid], start);
    }
    if (tile == 0u && tid == 0) A.buckets->split = kSplit;
    __syncthreads();

    uint32_t dst[ITEMS];
    char *kout = (char *)A.keys_out, *vout = (char *)A.vals_out;
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const uint32_t i = (uint32_t)tid + (uint32_t)r * kThreads, k = s_order[i];
        dst[r] = digit_place(s_dest[digit_of(k, A.top)], i);
        if (i < valid) *(uint32_t *)(kout + dst[r]) = k;
    }
    if constexpr (VALS) {
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) *(uint32_t *)((char *)s_order + at[r]) = val[r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) {
            const uint32_t i = (uint32_t)tid + (uint32_t)r * kThreads;
            if (i < valid) *(uint32_t *)(vout + dst[r]) = s_order[i];
        }
    }
}

// ------------------------------------------------------------------------- keys to their places by one partition in LDS
//
// The keys of a workgroup, n of them, go into bins by the highest of the bits they differ in: twice as many bins as keys or more (32,768 at
// most), so that most keys have a bin of their own.  A bin's keys get their places from counters (additions that return what was
// there: in no particular order), and where each belongs inside its bin is then seen by comparing it with the others there: key bits
// below the bin's, then the key's place among the n, so the result is the stable order.  This takes the place of all passes: some ten
// accesses to LDS and 45 vector instructions per row of 64 keys, where each pass on eight bits takes more than that.  What bounds it
// is both (256 buckets of 16,384 keys 19.8 us, pairs 22.0, by three passes 33.9; in small buckets of large sorts LDS is busy for 68 % of the time, the
// vector unit for 75).  By passes -> now, us per sort: 5000 keys 13.6 -> 8.3, 8192 18.4 -> 9.7, in order 19.3 -> 4.9 (without the copy of new
// ones), 2^22 in buckets 70.1 -> 61.5, pairs 83.4 -> 72.
//   twice as many bins as keys and not as many: most of the comparisons, which were the largest part, fall away.
//   a bin's first place and the next one's from two aligned words: one read across words takes three times as long.
//   four neighbouring counters a thread when they are added up, not a thread's whole share in a row: that was a quarter of what LDS did (below).
//   payloads loaded when the keys have their places, not with them: 256 x 16,320 pairs 23.2 -> 20.4 us, 16,384 (18 rows) 28.9 -> 21.5.
// Keys that crowd in a part of their range are seen before anything is moved, from a sample of pairs, or from the counters, and the passes do the work:
// what that costs is 0.5 to 1.1 us (below).  Fewer than 2049 keys gain nothing, for more than 20,480 (18,432 with payloads: BlockLdsOf) there are too few registers.

constexpr uint32_t kBinMost = 16;                          // keys of a bin, at most
constexpr uint32_t kAlikeMost = 6;                         // pairs of a sample that share a bin: fewer
template <int W> struct BinParts { uint32_t differ[W], one[W], alike[W], sum[64], most[W]; };

// body(r0, rows) for rows r0 .. r0 + rows - 1 of ITEMS, BATCH at a time, each call with constants of its own.
template <int N> struct Constant { constexpr __device__ __forceinline__ operator int() const { return N; } };
template <int ITEMS, int BATCH, int R0 = 0, class Body> __device__ __forceinline__ void in_batches(Body body)
{
    if constexpr (R0 < ITEMS) {
        body(Constant<R0>(), Constant<(R0 + BATCH < ITEMS ? BATCH : ITEMS - R0)>());
        in_batches<ITEMS, BATCH, R0 + BATCH>(body);
    }
}

__device__ __forceinline__ uint32_t bits_below(uint32_t n) { return n <= 1u ? 0u : 32u - (uint32_t)__builtin_clz(n - 1u); }      // 2^result >= n

// Bits in which the keys differ, or more (exchanges with other wavefronts are the caller's: two parts).
template <int ITEMS> __device__ __forceinline__ uint32_t bits_that_differ(const uint32_t (&key)[ITEMS], uint32_t &one)
{
    // (a wavefront's keys are compared with one of its own, and those with each other: key 0 of all would have to be loaded)
    uint32_t own = 0u;
    one = (uint32_t)__builtin_amdgcn_readfirstlane((int)key[0]);
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) own |= key[r] ^ one;
    return wave_or(own);
}
template <int W> __device__ __forceinline__ uint32_t bits_that_differ_in_all(const BinParts<W> &parts)
{
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t one_of = parts.one[lane % W], differ_of = parts.differ[lane % W];
    return row_or(differ_of | (one_of ^ (uint32_t)__builtin_amdgcn_readfirstlane((int)one_of)));
}

// at[r]: byte offset in the ordered keys of this lane's key r, which is key first + 64 r of n (past the end, where
// the caller has repeated a key: its own); false (in all threads, none of which looks at `bins` any more): not by bins.
// `bits`: those that the keys are ordered by; `bins`: 16-bit counters, 2^MAX_LOG of them,
// and `order` 64 W ITEMS + kBinMost words, both free before and (true) after.
template <int W, int ITEMS, uint32_t MAX_LOG>
__device__ __forceinline__ bool places_by_bins(const uint32_t (&key)[ITEMS], uint32_t first, uint32_t n, uint32_t bits, uint32_t *order, uint32_t *bins, BinParts<W> &parts,
                                               uint32_t (&at)[ITEMS], uint32_t &differ)
{
    differ = ~0u >> (32u - bits);
    if (bits < 32u && !bins_suffice(n, bits)) return false;
    constexpr uint32_t kThreads = 64 * W, kBinChunks = (1u << MAX_LOG) / 2u / kThreads / 4u;
    constexpr int kBatch = 4;
    constexpr uint32_t kSlots = kThreads * ITEMS;
    static_assert(W * kBinChunks <= 64, "a lane for each part of the counters");
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    const uint32_t wave_first = (uint32_t)__builtin_amdgcn_readfirstlane((int)first);
    const uint32_t index_bits = bits_below(n);
    uint32_t log_bins = index_bits + 1u < 11u ? 11u : index_bits + 1u;
    log_bins = log_bins < MAX_LOG ? log_bins : MAX_LOG;
    for (uint32_t i = 4u * tid; i < 1u << (log_bins - 1u); i += 4u * kThreads)
        *(u32x4 *)(bins + i) = u32x4{0u, 0u, 0u, 0u};
    uint32_t one;
    const uint32_t own = bits_that_differ(key, one);
    // Keys that crowd in a part of their range are mostly seen in a sample: a lane's first keys, 64 places apart, that fall into one bin.
    // (normally distributed floats, us in a row of sorts with the copy of new keys, by passes alone / with the look: 2049 10.8 / 11.4, 3000 11.3 / 12.0, 5000 14.1 / 14.8, 8192
    // 19.1 / 19.6; pairs, 13.2 / 14.0, 14.2 / 15.1, 17.7 / 18.6, 23.5 / 24.0.  0.1 us of it is the sample, the rest what all wavefronts find out together.  Without the sample
    // the counters would see it, 0.3 us later.  Evenly spread ones 10.6 / 6.3, 11.1 / 6.7, 13.8 / 7.8, 18.8 / 9.6.)
    uint32_t alike = 0u;
    constexpr int kSample = ITEMS < 4 ? ITEMS : 4;
    const uint32_t range_of_wave = own & differ;
    if (wave_first + 64u * kSample <= n && range_of_wave != 0u) {
        const uint32_t top = 32u - (uint32_t)__builtin_clz(range_of_wave);
        const uint32_t window = differ & (top > log_bins ? ~0u << (top - log_bins) : ~0u);
#pragma unroll
        for (int a = 0; a < kSample; ++a)
#pragma unroll
            for (int b = 0; b < a; ++b) alike += (uint32_t)__builtin_popcountll(__ballot(((key[a] ^ key[b]) & window) == 0u));
    }
    if (lane == 0u) { parts.differ[wave] = own; parts.one[wave] = one; parts.alike[wave] = alike; }
    __syncthreads();
    const uint32_t alike_of = parts.alike[lane % W];
    differ &= bits_that_differ_in_all(parts);
    alike = row_sum(lane % 16u < W ? alike_of : 0u);
    if (differ == 0u) {                                    // all equal: in order
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) at[r] = 4u * (first + 64u * r);
        return true;
    }
    const uint32_t high = 32u - (uint32_t)__builtin_clz(differ);
    const uint32_t width = high < log_bins ? high : log_bins, shift = high - width;
    // (bits that never differ, as low ones of numbers with few digits, make no bins)
    if (!bins_suffice(n, (uint32_t)__builtin_popcount(differ >> shift)) || alike >= kAlikeMost) return false;

    // Rows in batches of four, their accesses to LDS on their way together: one after the other, each row waits for its own.  (The
    // scheduler is kept from putting a row's uses back between the next row's accesses.)  Lanes past the end add nothing to
    // their bins and keep the places that they have.
    const auto batches = [=](auto body) {
        in_batches<ITEMS, kBatch>([&](auto r0, auto rows) {
            body((int)r0, (int)rows, wave_first + 64u * (uint32_t)(r0 + rows) > n);
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    // Word i counts bins i and words + i, in its lower and upper half: both halves are added up at once.
    const uint32_t words = 1u << (width - 1u);
    const auto word_of = [=](uint32_t k) {
        asm("" : "+v"(k));                                 // (nothing, here and below, is kept from one use of a key to the next: registers)
        return (uint32_t *)((char *)bins + 4u * __builtin_amdgcn_ubfe(k, shift, width - 1u));
    };
    const auto half_of = [=](uint32_t k) {                 // 0 or 16
        asm("" : "+v"(k));
        return __builtin_amdgcn_ubfe(k, high - 1u, 1u) << 4;
    };
    const auto index_of = [=](int r) {
        uint32_t i = first;
        asm("" : "+v"(i));
        return i + 64u * r;
    };

    // ---- count
    batches([&](int r0, int rows, bool ends) {
        uint32_t half[kBatch], one[kBatch], *word[kBatch];
#pragma unroll
        for (int q = 0; q < kBatch; ++q) if (q < rows) { half[q] = half_of(key[r0 + q]); word[q] = word_of(key[r0 + q]); one[q] = 1u << half[q]; }
        if (ends) {
#pragma unroll
            for (int q = 0; q < kBatch; ++q) if (q < rows) {
                const uint32_t i = index_of(r0 + q);
                if (i >= n) { word[q] = bins + (i & (words - 1u)); one[q] = 0u; }      // (all over the bins: lanes that add to one go one after the other)
            }
        }
#pragma unroll
        for (int q = 0; q < kBatch; ++q) if (q < rows) at[r0 + q] = atomicAdd(word[q], one[q]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < kBatch; ++q) if (q < rows) at[r0 + q] = __builtin_amdgcn_ubfe(at[r0 + q], half[q], 16u);
    });
    __syncthreads();

    // ---- counters -> first places
    // (Four neighbouring words a thread at a time, the workgroup's one after the other.  Sixteen in a row for a thread would mean one sum for it
    // instead of four, but threads 64 bytes apart meet in the banks: a quarter of all that LDS does here.)
    const auto has = [=](uint32_t c) { return 4u * (c * kThreads + tid) < words; };
    u32x4 w[kBinChunks];
    uint32_t inc[kBinChunks], sums[kBinChunks];            // of both halves
    u16x2 mosts = {0, 0};
#pragma unroll
    for (uint32_t c = 0; c < kBinChunks; ++c) {
        w[c] = has(c) ? *(const u32x4 *)(bins + 4u * (c * kThreads + tid)) : u32x4{0u, 0u, 0u, 0u};
        sums[c] = w[c][0] + w[c][1] + w[c][2] + w[c][3];
        inc[c] = wave_inclusive_scan(sums[c]);
        if (lane == 63u) parts.sum[c * W + wave] = inc[c];
#pragma unroll
        for (int i = 0; i < 4; ++i) mosts = __builtin_elementwise_max(mosts, __builtin_bit_cast(u16x2, (uint32_t)w[c][i]));
    }
    uint32_t most = wave_max(mosts[0] > mosts[1] ? mosts[0] : mosts[1]);
    if (lane == 63u) parts.most[wave] = most;
    __syncthreads();
    most = wave_max(parts.most[lane % W]);
    if (most > kBinMost) return false;
    const uint32_t part = lane < W * kBinChunks ? parts.sum[lane % (W * kBinChunks)] : 0u, up_to = wave_inclusive_scan(part);
    const uint32_t all = uniform_from_lane(up_to, 63);
#pragma unroll
    for (uint32_t c = 0; c < kBinChunks; ++c) {
        // (the upper half of the bins comes after all of the lower)
        uint32_t place = uniform_from_lane(up_to - part, (int)(c * W + wave)) + (all << 16) + inc[c] - sums[c];
        if (has(c)) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t size = w[c][i];
                w[c][i] = place;
                place += size;
            }
            *(u32x4 *)(bins + 4u * (c * kThreads + tid)) = w[c];
        }
    }
    if (tid == 0u) {
        bins[words] = (all & 0xFFFFu) | n << 16;           // (as thread 0 has written it if there are fewer than four)
#pragma unroll
        for (int i = 0; i < 4; ++i) order[kSlots + i] = ~0u;
    }
    __syncthreads();

    // ---- into the bins
    const uint32_t below = (1u << shift) - 1u;
    uint32_t mine[ITEMS], count[ITEMS];                    // what keys of a bin are compared by; keys of the bin
    batches([&](int r0, int rows, bool ends) {
        uint32_t w0[kBatch], w1[kBatch], place[kBatch];
#pragma unroll
        for (int q = 0; q < kBatch; ++q) if (q < rows) {
            const uint32_t *word = word_of(key[r0 + q]);
            w0[q] = word[0]; w1[q] = word[1];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < kBatch; ++q) if (q < rows) {
            const int r = r0 + q;
            const uint32_t half = half_of(key[r]), start = __builtin_amdgcn_ubfe(w0[q], half, 16u);
            count[r] = __builtin_amdgcn_ubfe(w1[q], half, 16u) - start;
            place[q] = start + at[r];
            at[r] = start;
            mine[r] = (key[r] & below) << index_bits | index_of(r);
        }
        if (ends) {
#pragma unroll
            for (int q = 0; q < kBatch; ++q) if (q < rows) {
                const uint32_t i = index_of(r0 + q);
                if (i >= n) { count[r0 + q] = 0u; place[q] = at[r0 + q] = i; }
            }
        }
#pragma unroll
        for (int q = 0; q < kBatch; ++q) if (q < rows) order[place[q]] = mine[r0 + q];
    });
    __syncthreads();

    // ---- the keys of its bin that go in front of each
    // (a key alone in its bin, and one of two, reads the words behind all keys from there on: one address, no conflicts)
    batches([&](int r0, int rows, bool) {
        uint32_t x[kBatch][4];
#pragma unroll
        for (int q = 0; q < kBatch; ++q) if (q < rows) {
            const int r = r0 + q;
            const uint32_t *two = order + (count[r] >= 2u ? at[r] : kSlots), *more = order + (count[r] >= 3u ? at[r] : kSlots);
            x[q][0] = two[0]; x[q][1] = two[1]; x[q][2] = more[2]; x[q][3] = more[3];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < kBatch; ++q) if (q < rows) {
            const int r = r0 + q;
            at[r] += (uint32_t)(x[q][0] < mine[r]);
            at[r] += (uint32_t)(x[q][1] < mine[r]);
            at[r] += (uint32_t)(x[q][2] < mine[r]);
            at[r] += (uint32_t)((count[r] >= 4u) & (x[q][3] < mine[r]));
        }
    });
    // (the few that share it with four and more look it up again: `at` is no longer where it starts)
    if (most > 4u) {
        in_batches<ITEMS, 1>([&](auto r, auto) {
            if (__ballot(count[r] > 4u)) {
                const uint32_t *bin = order + __builtin_amdgcn_ubfe(*word_of(key[r]), half_of(key[r]), 16u);
#pragma unroll 1
                for (uint32_t j = 4u; j < most; ++j)
                    if (j < count[r]) at[r] += (uint32_t)(bin[j] < mine[r]);
            }
        });
    }
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) at[r] *= 4u;
    __syncthreads();
    return true;
}

// ------------------------------------------------------------------------- a sort in one workgroup
//
// A whole sort of few keys, or a bucket of the keys that a first pass on the top digit has split.  What bounds it is the ranking's
// instructions, so the rows per lane are counted out (sort_in_block_of) -- each with code of its own: counted out by a loop, the
// instructions of neighbouring rows lose their place between each other (12,000 keys 26 -> 30 us).

struct BlockArgs {
    const uint32_t *keys, *vals;
    uint32_t *keys_out, *vals_out;        // (may be where the keys come from: a workgroup reads all of its own first)
    const Buckets *buckets;               // null: one workgroup sorts all keys; else workgroup b those of bucket b, if there are buckets
    uint32_t n;                           // keys in all
    Passes P;                             // a bucket's digits, or all
    uint32_t bits;                        // the bits they cover, from the lowest on
};
// A workgroup of WAVES wavefronts that sorts up to ROWS rows a lane, FEW to BIN_ROWS of them by bins (PAIR_ROWS with payloads; more would not do with
// the registers), whose counters lie behind as many keys, in part where more rows have theirs.
// 20 rows with payloads by bins spill 13 registers a lane, and a kernel with scratch starts 0.4 us later, whatever it sorts: 1033 to 2048 pairs 11.9 us
// without that form in the kernel and 12.3 with it, 8000 pairs 12.7 and 13.2.  For buckets of 18,433 to 20,480 pairs it is still the faster way (4.8 million pairs 87.8 us, by
// passes 93.4), so they have a kernel of their own (block_sort_pairs20_kernel).
template <int WAVES, int ROWS, int FEW, int BIN_ROWS, uint32_t LOG_BINS, int PAIR_ROWS = 18> struct BlockLdsOf {
    static constexpr int kWaves = WAVES, kRows = ROWS, kBinFew = FEW;
    template <bool VALS> static constexpr int kBinRows = VALS ? PAIR_ROWS : BIN_ROWS;
    static constexpr uint32_t kCapacity = 64u * WAVES * ROWS, kLogBins = LOG_BINS, kBinsAt = 64u * WAVES * BIN_ROWS + kBinMost, kBinWords = (1u << LOG_BINS) / 2u + 4u;
    uint32_t order[kCapacity];
    union {
        struct {
            alignas(16) uint16_t cnt[WAVES][kDigits];
            uint64_t masks[WAVES][kDigits];
        };
        uint32_t bins_end[kBinsAt + kBinWords - kCapacity];
    };
    uint32_t part[4];
    BinParts<WAVES> bin_parts;
};
using BlockLds = BlockLdsOf<kBlockWaves, kBlockItems, 3, 20, 15>;
using BlockLdsPairs20 = BlockLdsOf<kBlockWaves, kBlockItems, 3, 20, 15, 20>;
static_assert(offsetof(BlockLds, bins_end) == 4 * kBlockCapacity && BlockLds::kBinsAt % 4 == 0, "the bins' counters, from order + kBinsAt on, are the struct's own");
static_assert(alignof(BlockLds) >= alignof(CounterQuad), "counters cleared four at a time");
static_assert(sizeof(BlockLds) <= 160 * 1024, "LDS of a compute unit");

template <int ITEMS, bool VALS, class Lds>
__device__ __forceinline__ void sort_in_block(const BlockArgs &B, uint32_t begin, uint32_t n, Lds &s)
{
    constexpr int W = Lds::kWaves;
    constexpr uint32_t kU = kUnit<ITEMS, W>;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t first = (uint32_t)wave * 64u * ITEMS + (uint32_t)lane;
    const uint32_t *keys = B.keys + begin, *vals = VALS ? B.vals + begin : nullptr;
    uint32_t key[ITEMS], val[VALS ? ITEMS : 1], at[ITEMS];
    // (a 32-bit offset from a uniform address: 64-bit ones of every row would be kept from the loads to the stores)
    const uint32_t lane4 = 4u * first;
    auto row = [=](auto *p, int r) { return (decltype(p))((char *)(p + 64 * r) + lane4); };
    // (past the end the last key is read again: no branches, so that all loads are on their way together)
    auto load = [=](const uint32_t *p, int r) {
        uint32_t i = first;
        asm("" : "+v"(i));                                 // (not kept from keys to payloads, nor from loads to stores: registers)
        i += 64u * r;
        return *(const uint32_t *)((const char *)p + 4u * (i < n ? i : n - 1u));
    };
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) key[r] = load(keys, r);
    const auto load_vals = [&] {
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) val[r] = load(vals, r);
    };
    uint32_t *keys_out = B.keys_out + begin, *vals_out = VALS ? B.vals_out + begin : nullptr;
    uint32_t differ = ~0u;                                 // bits that the keys differ in, or more
    const auto by_bins = [&] {
        if constexpr (ITEMS >= Lds::kBinFew && ITEMS <= Lds::template kBinRows<VALS>)
            return places_by_bins<W, ITEMS, Lds::kLogBins>(key, first, n, B.bits, s.order, s.order + Lds::kBinsAt, s.bin_parts, at, differ);
        else if constexpr (ITEMS > Lds::template kBinRows<VALS> && W < kBlockWaves) {
            // (small buckets of large sorts: the passes leave out digits in which no key differs.  3 * 2^23 pairs of 5000 values, buckets of one value: 402 -> 352 us)
            uint32_t one;
            const uint32_t own = bits_that_differ(key, one);
            if (lane == 0) { s.bin_parts.differ[wave] = own; s.bin_parts.one[wave] = one; }
            __syncthreads();
            differ = bits_that_differ_in_all(s.bin_parts);
            return false;
        }
        else return false;
    };
    if (by_bins()) {
        if constexpr (VALS) load_vals();
#pragma unroll
        for (int r = 0; r < ITEMS; ++r)
            *(uint32_t *)((char *)s.order + at[r]) = key[r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ITEMS; ++r)
            if (first + 64u * r < n) *row(keys_out, r) = s.order[first + 64u * r];
        if constexpr (VALS) {
            __syncthreads();
#pragma unroll
            for (int r = 0; r < ITEMS; ++r)
                *(uint32_t *)((char *)s.order + at[r]) = val[r];
            __syncthreads();
#pragma unroll
            for (int r = 0; r < ITEMS; ++r)
                if (first + 64u * r < n) *row(vals_out, r) = s.order[first + 64u * r];
        }
        return;
    }
    if constexpr (VALS) load_vals();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) key[r] = first + 64u * r < n ? key[r] : ~0u;                  // past the end: last in every pass
    for (int i = lane; i < kDigits; i += 64) s.masks[wave][i] = 0ull;
    for (int p = 0; p < B.P.count; ++p) {
        const Digit g = B.P.digit[p];
        if (digit_of(differ, g) == 0u) continue;           // (the keys stay where they are)
        ((CounterQuad *)s.cnt[wave])[lane] = 0u;
        wavefront_sync();
        rank_rows<ITEMS, (ITEMS <= 20)>(key, g, s.cnt[wave], at, s.masks[wave], (int)n - (int)first);       // (24 rows with payloads: registers)
        __syncthreads();
        uint32_t count, start;
        scan_counters<W, kU>(s.cnt, s.part, count, start, [](uint32_t) {});
        put_in_order<ITEMS, kU>(key, g, s.cnt[wave], s.order, at);
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) {
            const uint32_t k = s.order[first + 64u * r];
            key[r] = first + 64u * r < n ? k : ~0u;
        }
        if constexpr (VALS) {
            __syncthreads();
#pragma unroll
            for (int r = 0; r < ITEMS; ++r) *(uint32_t *)((char *)s.order + at[r]) = val[r];
            __syncthreads();
#pragma unroll
            for (int r = 0; r < ITEMS; ++r) val[r] = s.order[first + 64u * r];
        }
        // (the next pass's writes to s.order come after its barriers)
    }
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        if (first + 64u * r < n) {
            *row(keys_out, r) = key[r];
            if constexpr (VALS) *row(vals_out, r) = val[r];
        }
    }
}
// 1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 14, 16, 18, 20 or 24 rows per lane.
template <bool VALS, int ITEMS = 1, class Lds>
__device__ __forceinline__ void sort_in_block_of(const BlockArgs &B, uint32_t begin, uint32_t n, Lds &s)
{
    if constexpr (ITEMS >= Lds::kRows) {
        sort_in_block<Lds::kRows, VALS>(B, begin, n, s);
    } else {
        if (n <= 64u * Lds::kWaves * ITEMS) sort_in_block<ITEMS, VALS>(B, begin, n, s);
        else sort_in_block_of<VALS, ITEMS < 8 ? ITEMS + 1 : ITEMS < 20 ? ITEMS + 2 : ITEMS + 4>(B, begin, n, s);
    }
}

template <bool VALS, class Lds>
__device__ __forceinline__ void sort_block_or_bucket(const BlockArgs &B, Lds &s)
{
    uint32_t begin = 0u, n = B.n;
    if (B.buckets) {
        begin = B.buckets->start[blockIdx.x];
        const uint32_t end = blockIdx.x + 1u < kDigits ? B.buckets->start[blockIdx.x + 1u] : B.n;
        n = end > begin && end <= B.n ? end - begin : 0u;
        n = n < (uint32_t)kBlockCapacity ? n : (uint32_t)kBlockCapacity;
    }
    n = (uint32_t)__builtin_amdgcn_readfirstlane((int)n);
    if (n != 0u) sort_in_block_of<VALS>(B, begin, n, s);
}
template <bool VALS>
__global__ __launch_bounds__(64 * kBlockWaves) void block_sort_kernel(BlockArgs B)
{
    __shared__ BlockLds s;
    if (B.buckets && B.buckets->split == kNotSplit) return;
    sort_block_or_bucket<VALS>(B, s);
}
__global__ __launch_bounds__(64 * kBlockWaves) void block_sort_pairs20_kernel(BlockArgs B)
{
    __shared__ BlockLdsPairs20 s;
    if (B.buckets->split == kNotSplit) return;
    sort_block_or_bucket<true>(B, s);
}

// The buckets, or the second pass where there are none: a launch that returns at once is 1.2 us (two launches / one: 40,000 keys
// below 2^24 34.4 / 33.2 us, four plain passes 32.6, random ones 23.6 / 22.2; 10^6 63.7 / 62.5, 61.5, 39.2 / 38.0).  The pass has one
// workgroup per compute unit here, for the buckets' LDS, so it does for no more tiles than there are units (kTogetherMax).
template <int ITEMS, bool VALS>
__global__ __launch_bounds__(64 * kBlockWaves) void pass_or_buckets_kernel(PassArgs A, BlockArgs B, uint32_t tiles)
{
    constexpr int W = kBlockWaves;
    __shared__ union { PassLds<W, ITEMS, uint32_t> pass; BlockLds block; } s;
    if (A.buckets->split != kNotSplit) {
        sort_block_or_bucket<VALS>(B, s.block);
    } else {
        const uint32_t tile = take_tile(A, s.pass.part);
        if (tile < tiles) digit_pass<W, ITEMS, VALS, uint32_t, kLaterPass>(A, s.pass, tile);
    }
}

// ------------------------------------------------------------------------- two passes and small buckets
//
// Sorts of more keys than one pass splits finely enough: two passes, on the upper and, in each of its ranges, the lower half of the top 13 or 14 bits, leave
// buckets of some 2300 to 4700 keys, which a workgroup of four wavefronts each sorts by the other bits in LDS, in place.  That is three times
// 8 bytes per key (16 with payloads) where four passes move 8 bytes each; and the second pass has a carry chain per range, of some 32 tiles,
// and writes into 2 MiB (135 us for 2^26 keys on seven bits, the first 132; on six bits 125, on eight 145; a second one over the whole array takes 6 more).
// What the buckets' sizes are has to be known before the first pass: one table of all 2^14 counts in LDS, one addition per key,
// in place of four.  Buckets of up to 10,240 keys are sorted by eight wavefronts, a few larger ones by passes of their own (huge_pass).  Keys that crowd would have too
// many of these: a sample of 8192 keys, taken by the kernel that clears the tables, says whether it is worth counting; if the counts then say otherwise, the
// digits of the four passes are counted after all.
// us for 2^26 random keys: sample 8, count 66, sizes and starts 10, passes 132 + 133, buckets 159, launches with nothing to do 15 (four
// passes: 70 + 4 x 144).  What bounds the buckets' kernel is LDS (68 % of its time) and the vector unit (75 %) at 16 wavefronts a compute unit;
// pairs, 2^25 of them 107 us, the memory.  Tried and dropped: tiles of 8192 and 4096 keys in four and eight smaller workgroups a unit (first pass 176
// and 258), seven ballots for the seven bits (no change), buckets from the last one on, whose keys the memory-side cache may hold (157 -> 156.5), eight wavefronts for
// all buckets, which would save a launch (2^26 keys 611 -> 662).
// us per sort with the copy of new keys, four passes alone / now: 3 * 2^23 random keys 290 / 260, pairs 447 / 362, 2^25 378 / 323, pairs 633 / 486, 2^26 764 / 610, pairs 1450 / 1070, 76
// million 935 / 706, 2^26 in order 768 / 577.
// Keys that crowd pay for the sample (6 us; 3 of them because its places are far apart), for four launches with nothing to do (11) and for passes that ask which way the sort goes (4):
// normally distributed floats, 3 * 2^23 287 / 306, pairs 431 / 453, 2^25 375 / 396, pairs 610 / 629, 2^26 750 / 764, pairs 1390 / 1400, 76 million 890 / 897; and so
// do 3 * 2^23 keys of 16,000 values, whose buckets go by passes (281 / 311; pairs 410 / 415; 2^26 of them 720 / 547).  Fewer keys would lose more of what four passes take
// (2^24: 8 to 13 %) than others gain (11 %), so they keep the four passes.

using large_sort::kLogMost;
using large_sort::kSampleQuads;
static_assert((1u << large_sort::kLogLeast) % (4u * kHistThreads) == 0u && large_sort::kLogLeast == 13 && kLogMost == 14 && kDigits == 256, "who looks at what of a sample");
using FineLds = BlockLdsOf<4, 20, 1, 20, 13>;
static_assert(offsetof(FineLds, bins_end) == 4 * FineLds::kCapacity && FineLds::kBinsAt % 4 == 0 && alignof(FineLds) >= alignof(CounterQuad), "as BlockLds");
static_assert(4 * sizeof(FineLds) <= 160 * 1024, "four workgroups on a compute unit");
using FineLargeLds = BlockLdsOf<8, 20, 1, 20, 14>;
static_assert(offsetof(FineLargeLds, bins_end) == 4 * FineLargeLds::kCapacity && FineLargeLds::kBinsAt % 4 == 0 && alignof(FineLargeLds) >= alignof(CounterQuad), "as BlockLds");
static_assert(2 * sizeof(FineLargeLds) <= 160 * 1024, "two workgroups on a compute unit");
static_assert(FineLds::kCapacity == large_sort::kSmallMost && FineLargeLds::kCapacity == large_sort::kLargeMost, "as planned");

struct FineArgs {
    HistArgs H;                           // keys, the four passes' digits, status words to clear
    large_sort::Found *fine;
    uint32_t *counts;                     // [table][bucket], kTables of them
    TileOfRange *ranges;                  // the second pass's tiles
    uint32_t tile_keys;
    uint32_t *clear;                      // words to clear: H.hist and what follows it, up to the status words
    uint32_t clear_quads;
    Digit all, second;                    // a bucket's bits, and the lower half of them
    uint32_t *huge;                       // tiles of huge buckets: bucket in the lower 14 bits, tile above
    large_sort::Plan plan;
    BlockArgs B;                          // buckets in their places
};

// Sample and clear.  (The sample: groups of four keys, one from each of kSampleQuads equal parts of the array, not at the same place of each.)
// Nobody waits for a sum while keys are added; all sums are looked at afterwards.  The upper half of a counter counts first keys of a group: those of a group
// may share a bucket, as they do in an array in order, where the number of buckets with keys would say that there are few.
__global__ __launch_bounds__(kHistThreads) void fine_sample_kernel(FineArgs F)
{
    __shared__ uint32_t s_count[1u << kLogMost];
    const uint32_t tid = threadIdx.x;
    if (blockIdx.x != 0u) {
        const uint32_t found = (uint32_t)((const u32x4 *)F.fine - (const u32x4 *)F.clear);      // what workgroup 0 writes
        for (uint32_t i = (blockIdx.x - 1u) * kHistThreads + tid; i < F.clear_quads; i += (gridDim.x - 1u) * kHistThreads)
            if (i != found && i != found + 1u) ((u32x4 *)F.clear)[i] = u32x4{0u, 0u, 0u, 0u};
        return;
    }
    const uint32_t buckets = 1u << F.all.width;
    const uint32_t part = (uint32_t)(F.H.n / 4u / kSampleQuads);           // quads: at least one
    u32x4 k[kSampleQuads / kHistThreads];
#pragma unroll
    for (uint32_t q = 0; q < kSampleQuads / kHistThreads; ++q) {
        const uint32_t g = q * kHistThreads + tid;
        k[q] = ((const u32x4 *)F.H.keys)[(uint64_t)g * part + (g * 0x9E3779B1u >> 8) % part];
    }
    for (uint32_t i = 4u * tid; i < buckets; i += 4u * kHistThreads) *(u32x4 *)(s_count + i) = u32x4{0u, 0u, 0u, 0u};
    __syncthreads();
#pragma unroll
    for (uint32_t q = 0; q < kSampleQuads / kHistThreads; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) add_to_count(s_count, digit_of(k[q][i], F.all), i == 0 ? 0x10001u : 1u);
    __syncthreads();
    // Four buckets a thread at a time; 16 lanes, or 8 (2^13 buckets), have a 256th of them.
    uint32_t used = 0u, work = 0u;
    bool crowded = false;
    const uint32_t last_of = F.all.width == kLogMost ? 15u : 7u;
    for (uint32_t i = 4u * tid; i < buckets; i += 4u * kHistThreads) {
        const u32x4 c = *(const u32x4 *)(s_count + i);
        uint32_t wide = 0u, most = 0u;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t keys = c[j] & 0xFFFFu;
            wide += keys;
            most = keys > most ? keys : most;
            used += c[j] > 0xFFFFu ? 1u : 0u;
        }
        if (__ballot(most > F.plan.some_most)) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t keys = c[j] & 0xFFFFu;
                if (keys > F.plan.some_most) work += keys * (1u + (uint32_t)((uint64_t)keys * F.H.n / (large_sort::kSample * large_sort::kHugeTile)));
            }
        }
        wide += dpp0<kRowShr + 1>(wide);
        wide += dpp0<kRowShr + 2>(wide);
        wide += dpp0<kRowShr + 4>(wide);
        if (last_of == 15u) wide += dpp0<kRowShr + 8>(wide);
        crowded |= most > F.plan.huge_most || ((tid & last_of) == last_of && wide > F.plan.wide_most);
    }
    __shared__ uint32_t s_work[kHistThreads / 64], s_used[kHistThreads / 64];
    work = wave_sum(work);                                 // (at most 8192 keys and what a bucket of all of them reads: no overflow)
    used = wave_sum(used);
    if ((tid & 63u) == 0u) { s_work[tid >> 6] = work; s_used[tid >> 6] = used; }
    const bool any = __syncthreads_or(crowded);
    if (tid >= 64u) return;
    work = row_sum(s_work[tid & 15u]);
    used = row_sum(s_used[tid & 15u]);
    if (tid < 8u) ((uint32_t *)F.fine)[tid] = tid < 2u && !any && work <= F.plan.work_most && used >= F.plan.few_most ? 1u : 0u;
}

// The buckets' sizes, or the digits' counts.
__global__ __launch_bounds__(kHistThreads) void fine_count_kernel(FineArgs F)
{
    __shared__ uint32_t s_count[kHistWords > (1 << kLogMost) ? kHistWords : 1 << kLogMost];
    if (!F.fine->tried) { digit_histograms(F.H, s_count); return; }
    const HistArgs &H = F.H;
    const uint32_t tid = threadIdx.x, buckets = 1u << F.all.width;
    for (uint32_t i = 4u * tid; i < buckets; i += 4u * kHistThreads) *(u32x4 *)(s_count + i) = u32x4{0u, 0u, 0u, 0u};
    __syncthreads();
    const uint64_t stride = (uint64_t)gridDim.x * kHistThreads, t0 = (uint64_t)blockIdx.x * kHistThreads + tid, quads = H.n / 4;
    // (from the last key on: those written last may still be in the memory-side cache.  2^26 keys that were: 71 -> 63 us)
    const u32x4 *keys4 = (const u32x4 *)H.keys + quads - 1;
    constexpr int kAhead = 4;
    u32x4 k[kAhead];
    uint64_t i = t0;
    for (; i + (kAhead - 1) * stride < quads; i += kAhead * stride) {
#pragma unroll
        for (int a = 0; a < kAhead; ++a) k[a] = H.stream ? __builtin_nontemporal_load(keys4 - (i + a * stride)) : *(keys4 - (i + a * stride));
#pragma unroll
        for (int a = 0; a < kAhead; ++a)
#pragma unroll
            for (int j = 0; j < 4; ++j) add_to_count(s_count, digit_of(k[a][j], F.all));
    }
    for (; i < quads; i += stride) {
        const u32x4 x = *(keys4 - i);
#pragma unroll
        for (int j = 0; j < 4; ++j) add_to_count(s_count, digit_of(x[j], F.all));
    }
    if (t0 < (H.n & 3u)) atomicAdd(&s_count[digit_of(H.keys[4 * quads + t0], F.all)], 1u);
    for (uint64_t q = t0; q < H.status_quads; q += stride) ((u32x4 *)H.status)[q] = u32x4{0u, 0u, 0u, 0u};
    __syncthreads();
    uint32_t *table = F.counts + (size_t)(blockIdx.x % kTables) * buckets;
    for (uint32_t b = tid; b < buckets; b += kHistThreads)
        if (s_count[b]) atomicAdd(&table[b], s_count[b]);
}

// Workgroup t: buckets t * 2^second.width on, one per thread.  Their sizes over all tables go to table 0.
__global__ __launch_bounds__(kDigits) void fine_judge_kernel(FineArgs F)
{
    if (!F.fine->tried) return;
    __shared__ uint32_t s_part[kDigits / 64];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, buckets = 1u << F.all.width, row = 1u << F.second.width;
    uint32_t size = 0u;
    if (tid < row) {
        const uint32_t b = blockIdx.x * row + tid;
#pragma unroll
        for (uint32_t t = 0; t < kTables; ++t) size += F.counts[(size_t)t * buckets + b];
        F.counts[b] = size;
        if (size > large_sort::kHugeMost) {
            F.fine->split = kNotSplit;
        } else if (size > large_sort::kLargeMost) {
            const uint32_t tiles = large_sort::tiles_of(size), at = atomicAdd(&F.fine->huge, tiles);
            atomicAdd(&F.fine->work, (size >> 10) * tiles);
            for (uint32_t i = 0; i < tiles && at + i < F.plan.huge_tiles; ++i) F.huge[at + i] = b | i << kLogMost;
        } else if (size > large_sort::kSmallMost) {
            F.fine->large_at[atomicAdd(&F.fine->large, 1u)] = b;
        }
    }
    const uint32_t sum = wave_sum(size);
    if (lane == 0u) s_part[tid >> 6] = sum;
    __syncthreads();
    if (tid == 0u) F.fine->top[blockIdx.x] = s_part[0] + s_part[1] + s_part[2] + s_part[3];
}

// Where the buckets start, or, where the sample was wrong, the digits' counts.
__global__ __launch_bounds__(kHistThreads) void fine_start_kernel(FineArgs F)
{
    __shared__ uint32_t s_count[kHistWords];
    if (!F.fine->tried) return;
    // (where the huge buckets are too much work, all workgroups find so, whether they see that the first has written it or not)
    const bool over = F.fine->work > F.plan.huge_work || F.fine->huge > F.plan.huge_tiles;
    if (F.fine->split == kNotSplit || over) {
        if (over && blockIdx.x == 0u && threadIdx.x == 0u) F.fine->split = kNotSplit;
        digit_histograms(F.H, s_count);
        return;
    }
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6, row = 1u << F.second.width;
    if (blockIdx.x >= 1u << (F.all.width - F.second.width) || tid >= kDigits) return;        // (the others of the workgroup wait for nobody)
    // every wavefront adds up what lies in front of the row, and the parts of it in front of its own
    uint32_t before = 0u, tiles = 0u;
    for (uint32_t t = lane; t < blockIdx.x; t += 64u) { before += F.fine->top[t]; tiles += (F.fine->top[t] + F.tile_keys - 1u) / F.tile_keys; }
    const uint32_t base = wave_sum(before), first = wave_sum(tiles);
    const uint32_t *sizes = F.counts + blockIdx.x * row;
    before = 0u;
    for (uint32_t s = lane; s < 64u * wave && s < row; s += 64u) before += sizes[s];
    before = base + wave_sum(before);
    const uint32_t size = tid < row ? sizes[tid] : 0u;
    const uint32_t inc = wave_inclusive_scan(size);
    if (tid < row) F.fine->start[blockIdx.x * row + tid] = before + inc - size;
    const uint32_t keys = F.fine->top[blockIdx.x];
    for (uint32_t i = tid; i * F.tile_keys < keys; i += kDigits) {
        const uint32_t left = keys - i * F.tile_keys;
        F.ranges[first + i] = {base + i * F.tile_keys, left < F.tile_keys ? left : F.tile_keys, blockIdx.x, i == 0u ? 1u : 0u};
    }
}

template <bool VALS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void fine_sort_kernel(FineArgs F)
{
    __shared__ FineLds s;
    if (F.fine->split == kNotSplit) return;
    // (one bucket each: as a loop over buckets this takes too many registers, 157 -> 178 us for 2^26 keys, pairs far worse)
    const uint32_t size = (uint32_t)__builtin_amdgcn_readfirstlane((int)F.counts[blockIdx.x]), begin = F.fine->start[blockIdx.x];
    if (size > 1u && size <= FineLds::kCapacity) sort_in_block_of<VALS, 8>(F.B, begin, size, s);
}
template <bool VALS>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4))) void fine_sort_large_kernel(FineArgs F)
{
    __shared__ FineLargeLds s;
    if (F.fine->split == kNotSplit) return;
    for (uint32_t i = blockIdx.x; i < F.fine->large; i += gridDim.x) {
        const uint32_t b = F.fine->large_at[i];
        const uint32_t size = (uint32_t)__builtin_amdgcn_readfirstlane((int)F.counts[b]);
        sort_in_block_of<VALS, 10>(F.B, F.fine->start[b], size < FineLargeLds::kCapacity ? size : FineLargeLds::kCapacity, s);
        __syncthreads();
    }
}

// ------------------------------------------------------------------------- host side

// Up to here one workgroup does everything (us per sort, one workgroup / a pass and buckets: 7169 random keys 18.0 / 14.0, but equal ones 16.5 /
// 19.9).
constexpr size_t kBlockSortFew = 8192;
// Up to here the counting kernel has eight workgroups and no launch that clears tables in front (a quarter where it also copies).
constexpr size_t kOwnTables = (size_t)1 << 17;
hipError_t launch_block_sort(const BlockArgs &args_in, unsigned grid, hipStream_t s)
{
    BlockArgs B = args_in;
    void *args[] = {&B};
    // (evenly spread keys: the largest of 256 buckets has three standard deviations more than the mean, so 18,432 are exceeded from a mean of 18,000 on; where
    // two passes do, they are as fast: 5 million pairs on 24 bits 92.5 us, 95.8 by bins)
    const bool pairs20 = B.buckets && B.n / kDigits > 18000u && B.n / kDigits <= 20480u && B.P.count > 2;
    const void *fn = !B.vals ? (const void *)block_sort_kernel<false> : pairs20 ? (const void *)block_sort_pairs20_kernel : (const void *)block_sort_kernel<true>;
    return hipLaunchKernel(fn, dim3(grid), dim3(64 * kBlockWaves), args, 0, s);
}
// May random keys be expected to have buckets (of 256) that are small enough: mean and six standard deviations?  (Up to 6,055,225 keys.)
bool buckets_fit(size_t n)
{
    const double mean = (double)n / kDigits;
    return mean + 6.0 * __builtin_sqrt(mean) <= (double)bucket_limit(n, (uint32_t)kBlockCapacity);
}

// Keys per lane of a pass.  Few keys: many small tiles, so that all compute units have one and each is done sooner;
// many keys: long ranges to write and fewer status words (us per sort of random keys, 4 / 8 / 16 keys per lane:
// 100,000 38 / 41 / 53; 400,000 50 / 50 / 60; 1,000,003 69 / 66 / 75; 2^22 150 / 116 / 117, with payloads 162 / 126 / 132;
// 2^23 242 / 173 / 145; 2^26 1704 / 1104 / 776).
constexpr int kPassWaves = 16;
int pass_items(size_t n) { return n <= ((size_t)1 << 19) ? 4 : n < ((size_t)5 << 20) ? 8 : 16; }

template <int ITEMS, PassRole ROLE> const void *pass_kernel_of(bool vals)
{
    return vals ? (const void *)digit_pass_kernel<kPassWaves, ITEMS, true, uint32_t, ROLE> : (const void *)digit_pass_kernel<kPassWaves, ITEMS, false, uint32_t, ROLE>;
}
template <PassRole ROLE> const void *pass_kernel(int items, bool vals)
{
    return items == 4 ? pass_kernel_of<4, ROLE>(vals) : items == 8 ? pass_kernel_of<8, ROLE>(vals) : pass_kernel_of<16, ROLE>(vals);
}
const void *wide_pass_kernel(bool vals)
{
    return vals ? (const void *)digit_pass_kernel<kPassWaves, 16, true, uint64_t> : (const void *)digit_pass_kernel<kPassWaves, 16, false, uint64_t>;
}

// Up to here the second pass and the buckets are one launch: 256 tiles at most.
constexpr size_t kTogetherMax = (size_t)1 << 21;
const void *pass_or_buckets_kernel_for(int items, bool vals)
{
    if (items == 4) return vals ? (const void *)pass_or_buckets_kernel<4, true> : (const void *)pass_or_buckets_kernel<4, false>;
    return vals ? (const void *)pass_or_buckets_kernel<8, true> : (const void *)pass_or_buckets_kernel<8, false>;
}

// `bits` low bits in digits as even as possible.
void split_digits(int bits, Passes &P)
{
    P.count = (bits + 7) / 8;
    for (int p = 0, at = 0; p < kMaxPasses; ++p) {
        const int width = p < P.count ? (bits - at + (P.count - p) - 1) / (P.count - p) : 1;
        P.digit[p] = {at < 32 ? at : 0, width};
        at += width;
    }
}

// `hist`: scratch from a 16-byte boundary on.
tcuscan_status_t fine_sort(void *d_keys, void *d_vals, size_t n, int bits, void *d_keys_tmp, void *d_vals_tmp, uint32_t *hist, const Passes &P, size_t tiles,
                           bool around_cache, unsigned use_tickets, unsigned spin_limit, unsigned mute_tile, void *d_fault, hipStream_t s)
{
    const bool v = d_vals != nullptr;
    FineArgs F;
    F.plan = large_sort::plan(n, v);
    const int log = F.plan.log, low = F.plan.low;          // (2^26 keys, the second pass on 7 / 8 / 6 bits of 14: 512 / 516 / 521 us; 2^25 pairs 392 / 387 / 391)
    const uint32_t buckets = 1u << log;
    const size_t most_tiles = F.plan.most_tiles;
    // scratch: digit counts, tickets, what the kernels find out, the buckets' counts, tiles (all cleared), status words
    uint32_t *tickets = hist + kTables * kTableWords;
    F.fine = (large_sort::Found *)(hist + F.plan.found);
    F.counts = hist + F.plan.counts;
    F.ranges = (TileOfRange *)(hist + F.plan.ranges);
    F.huge = hist + F.plan.huge;
    F.tile_keys = large_sort::kPassTile;
    uint32_t *status = hist + F.plan.status;
    static_assert(sizeof(TileOfRange) == 16 && large_sort::kPassTile == 64u * kPassWaves * 16u, "as planned");
    F.clear = hist;
    F.clear_quads = (uint32_t)F.plan.status / 4u;
    F.all = {bits - log, log};
    F.second = {bits - log, low};
    const Digit top = {bits - log + low, log - low};
    const int half = (bits - log + 1) / 2;                 // (at most ten: 2^13 buckets leave 19 bits of 32)
    const size_t pass_words = most_tiles * kDigits;
    HistArgs &H = F.H;
    H.keys = (const uint32_t *)d_keys; H.vals = nullptr; H.keys_copy = H.vals_copy = nullptr;
    H.hist = hist; H.tables = kTables; H.status = status; H.n = n; H.status_quads = pass_words * P.count / 4; H.P = P; H.stream = around_cache; H.own = false; H.from_end = true;
    F.B = {(const uint32_t *)d_keys, (const uint32_t *)d_vals, (uint32_t *)d_keys, (uint32_t *)d_vals, nullptr, (uint32_t)n, {}, (uint32_t)(bits - log)};
    split_digits(bits - log, F.B.P);
    void *fine_args[] = {&F};
    const auto launch = [&](const void *fn, size_t grid, int block, void **args) { return hipLaunchKernel(fn, dim3((unsigned)grid), dim3(block), args, 0, s) == hipSuccess; };
    if (!launch((const void *)fine_sample_kernel, 1 + 64, kHistThreads, fine_args)) return TCUSCAN_ERR_HIP;
    if (!launch((const void *)fine_count_kernel, kHistGrid, kHistThreads, fine_args)) return TCUSCAN_ERR_HIP;
    if (!launch((const void *)fine_judge_kernel, (size_t)1 << (log - low), kDigits, fine_args)) return TCUSCAN_ERR_HIP;
    if (!launch((const void *)fine_start_kernel, 256, kHistThreads, fine_args)) return TCUSCAN_ERR_HIP;
    uint32_t *src_k = (uint32_t *)d_keys, *dst_k = (uint32_t *)d_keys_tmp, *src_v = (uint32_t *)d_vals, *dst_v = (uint32_t *)d_vals_tmp;
    for (int p = 0; p < P.count; ++p) {
        PassArgs A = {};
        A.keys = src_k; A.vals = src_v; A.keys_out = dst_k; A.vals_out = dst_v;
        A.status = status + pass_words * p; A.hist = hist + kDigits * p; A.tables = kTables;
        A.ticket = use_tickets ? tickets + p : nullptr;
        A.fault = (uint32_t *)d_fault;
        A.n = n; A.spin_limit = spin_limit; A.mute_tile = mute_tile; A.digit = P.digit[p]; A.stream = around_cache;
        A.split = &F.fine->split;
        A.top = p == 0 ? top : p == 1 ? F.second : p == 2 ? Digit{0, half} : Digit{half, bits - log - half};
        A.top_hist = F.fine->top; A.ranges = F.ranges; A.range_start = F.fine->start;
        A.found = F.fine; A.huge = F.huge; A.sizes = F.counts; A.huge_tiles = F.plan.huge_tiles;
        void *args[] = {&A};
        const void *fn = p == 0 ? pass_kernel_of<16, kFirstOfTwo>(v) : p == 1 ? pass_kernel_of<16, kSecondOfTwo>(v) : pass_kernel_of<16, kAfterTwo>(v);
        if (!launch(fn, p == 1 ? most_tiles : tiles, 64 * kPassWaves, args)) return TCUSCAN_ERR_HIP;
        uint32_t *t = src_k; src_k = dst_k; dst_k = t;
        t = src_v; src_v = dst_v; dst_v = t;
    }
    if (!launch(v ? (const void *)fine_sort_kernel<true> : (const void *)fine_sort_kernel<false>, buckets, 256, fine_args)) return TCUSCAN_ERR_HIP;
    if (!launch(v ? (const void *)fine_sort_large_kernel<true> : (const void *)fine_sort_large_kernel<false>, 512, 512, fine_args)) return TCUSCAN_ERR_HIP;
    return TCUSCAN_OK;
}

}  // namespace

// Used by tcuscan_split_radix_sort_u32 (apps.hip), which has checked the arguments.  d_scratch: n words (4-byte aligned);
// d_fault: the workspace's fault word (null up to 16384 keys: no tile waits for another).
extern "C" __attribute__((visibility("hidden")))
tcuscan_status_t tcuscan_internal_digit_sort(void *d_keys, void *d_vals, size_t n, int bits, void *d_keys_tmp, void *d_vals_tmp,
                                             void *d_scratch, void *d_fault, tcuscan_stream_t stream)
{
    hipStream_t s = (hipStream_t)stream;
    Passes P;
    split_digits(bits, P);
    unsigned use_tickets, spin_limit, mute_tile;
    tcuscan_internal_chain_knobs(&use_tickets, &spin_limit, &mute_tile);
    const bool wide = n >= StatusWord<uint32_t>::kUnknown;
    if (n <= kBlockSortMax) {
        BlockArgs B = {(const uint32_t *)d_keys, (const uint32_t *)d_vals, (uint32_t *)d_keys, (uint32_t *)d_vals, nullptr, (uint32_t)n, P, (uint32_t)bits};
        if (n <= kBlockSortFew || P.count < 2) return launch_block_sort(B, 1, s) == hipSuccess ? TCUSCAN_OK : TCUSCAN_ERR_HIP;
        B.keys = (const uint32_t *)d_keys_tmp; B.vals = (const uint32_t *)d_vals_tmp; B.buckets = (const Buckets *)d_scratch;
        split_digits(bits - 8, B.P);
        B.bits = (uint32_t)bits - 8u;
        SpreadArgs A = {(const uint32_t *)d_keys, (const uint32_t *)d_vals, (uint32_t *)d_keys_tmp, (uint32_t *)d_vals_tmp, (Buckets *)d_scratch, (uint32_t)n, {bits - 8, 8}};
        void *args[] = {&A};
        const void *fn = d_vals ? (const void *)spread_kernel<true> : (const void *)spread_kernel<false>;
        if (hipLaunchKernel(fn, dim3((unsigned)((n + kSpreadTile - 1) / kSpreadTile)), dim3(64 * kSpreadWaves), args, 0, s) != hipSuccess) return TCUSCAN_ERR_HIP;
        return launch_block_sort(B, kDigits, s) == hipSuccess ? TCUSCAN_OK : TCUSCAN_ERR_HIP;
    }
    // One pass on the top eight bits, if the buckets then are small enough for a workgroup each, which sorts them by the other bits.
    const bool buckets_wanted = !wide && P.count >= 3 && buckets_fit(n);
    Passes rest = P;
    if (buckets_wanted) {
        split_digits(bits - 8, rest);                                    // (also for the passes that run where the buckets do not fit)
        P = rest;
        P.digit[P.count++] = {bits - 8, 8};
    }
    const bool fine_form = !buckets_wanted && !wide && large_sort::wanted(n, bits);
    const int items = pass_items(n);
    auto tiles_of = [n](int per_lane) { const size_t tile = (size_t)64 * kPassWaves * per_lane; return (n + tile - 1) / tile; };
    const size_t tiles = tiles_of(items);
    // Arrays that do not fit the memory-side cache (256 MiB) together are read around it, which leaves it to the pieces
    // that are being written: 2^26 keys 815 -> 776 us, 2^25 407 -> 395, 2^24 with payloads 314 -> 296, 2^25 with payloads 691
    // -> 595; below, what one pass wrote is what the next one finds there (2^24 keys: 224 against 229, 2^23 with payloads
    // 169 against 175).
    const bool around_cache = n * (d_vals ? 16 : 8) > ((size_t)192 << 20);
    const size_t want = (n / 4 + 2 * kHistThreads - 1) / (2 * kHistThreads);
    const bool odd = P.count & 1;                                        // the first pass then starts from a copy, and the last ends at home
    const bool own = n <= (odd ? kOwnTables / 4 : kOwnTables) && !use_tickets;       // (few workgroups are slow copiers)
    const unsigned hist_grid = (unsigned)(want < 1 ? 1 : own && want > kTables ? kTables : want < kHistGrid ? want : kHistGrid);
    // (one table / eight, us: two passes of 131,073 keys 22.6 / 22.7, 524,287 29.7 / 29.3, 10^6 36.4 / 35.0; with buckets, random ones 25.6 /
    // 26.5, 32.4 / 32.2, 38.8 / 37.7, keys below 2^24 39.5 / 40.1, 52.6 / 52.7, 63.8 / 62.3)
    const uint32_t tables = own ? hist_grid : n < ((size_t)1 << 19) ? 1 : kTables;
    // scratch: digit counts of the passes from the next 16-byte boundary on, ticket counters, what the first pass finds out, status words
    uint32_t *hist = (uint32_t *)(((uintptr_t)d_scratch + 15) & ~(uintptr_t)15), *tickets = hist + tables * kTableWords;
    Buckets *buckets = (Buckets *)(tickets + kMaxPasses);
    uint32_t *status = (uint32_t *)(((uintptr_t)(buckets + 1) + 15) & ~(uintptr_t)15);
    const size_t pass_words = tiles * kDigits * (wide ? 2 : 1);
    if (fine_form) return fine_sort(d_keys, d_vals, n, bits, d_keys_tmp, d_vals_tmp, hist, P, tiles, around_cache, use_tickets, spin_limit, mute_tile, d_fault, s);
    if (!own && tcuscan_internal_fill(hist, 4 * (tables * kTableWords + kMaxPasses), s) != hipSuccess) return TCUSCAN_ERR_HIP;

    uint32_t *src_k = (uint32_t *)d_keys, *dst_k = (uint32_t *)d_keys_tmp, *src_v = (uint32_t *)d_vals, *dst_v = (uint32_t *)d_vals_tmp;
    {
        HistArgs H;
        H.keys = src_k; H.vals = src_v;
        H.keys_copy = odd ? dst_k : nullptr; H.vals_copy = odd && src_v ? dst_v : nullptr;
        H.hist = hist; H.tables = tables; H.status = status; H.n = n; H.status_quads = pass_words * P.count / 4; H.P = P; H.stream = around_cache; H.own = own; H.from_end = false;
        void *args[] = {&H};
        if (hipLaunchKernel((const void *)digit_histograms_kernel, dim3(hist_grid), dim3(kHistThreads), args, 0, s) != hipSuccess) return TCUSCAN_ERR_HIP;
    }
    if (odd) {
        uint32_t *t = src_k; src_k = dst_k; dst_k = t;
        t = src_v; src_v = dst_v; dst_v = t;
    }
    BlockArgs B = {dst_k, dst_v, (uint32_t *)d_keys, (uint32_t *)d_vals, buckets, (uint32_t)n, rest, (uint32_t)bits - 8u};       // (the buckets are where the first pass puts them)
    const bool v = d_vals != nullptr, together = buckets_wanted && n <= kTogetherMax;
    // (passes that seldom have anything to do are cheaper with fewer, larger tiles; where they do, 3.2 million pairs take 105.5 us with
    // 8 rows per lane and 110 with 16, 2^22 the same with both)
    const int later_items = n >= ((size_t)1 << 22) ? 16 : items;
    const unsigned later_tiles = (unsigned)tiles_of(later_items);
    for (int p = 0; p < P.count; ++p) {
        PassArgs A;
        A.keys = src_k; A.vals = src_v; A.keys_out = dst_k; A.vals_out = dst_v;
        A.status = status + pass_words * p; A.hist = hist + kDigits * p; A.tables = tables;
        A.ticket = use_tickets ? tickets + p : nullptr;
        A.fault = (uint32_t *)d_fault;
        A.n = n; A.spin_limit = spin_limit; A.mute_tile = mute_tile; A.digit = P.digit[p]; A.stream = around_cache;
        A.top_hist = hist + kDigits * (P.count - 1); A.buckets = buckets; A.top = P.digit[P.count - 1];
        A.bucket_max = bucket_limit(n, (uint32_t)kBlockCapacity);
        A.split = &buckets->split;
        uint32_t pass_tiles = later_tiles;
        void *args[] = {&A, &B, &pass_tiles};                            // (the kernels of a pass alone take the first)
        hipError_t e = hipSuccess;
        if (buckets_wanted && p == 1 && !together) e = launch_block_sort(B, kDigits, s);
        if (e != hipSuccess) return TCUSCAN_ERR_HIP;
        const void *fn = wide ? wide_pass_kernel(v) : !buckets_wanted ? pass_kernel<kPlainPass>(items, v) : p == 0 ? pass_kernel<kChoosingPass>(items, v)
                       : p == 1 && together ? pass_or_buckets_kernel_for(items, v) : pass_kernel<kLaterPass>(later_items, v);
        const unsigned grid = !buckets_wanted || p == 0 ? (unsigned)tiles : p == 1 && together ? (unsigned)kDigits : later_tiles;
        if (hipLaunchKernel(fn, dim3(grid), dim3(64 * kPassWaves), args, 0, s) != hipSuccess) return TCUSCAN_ERR_HIP;
        uint32_t *t = src_k; src_k = dst_k; dst_k = t;
        t = src_v; src_v = dst_v; dst_v = t;
    }
    return TCUSCAN_OK;
}
