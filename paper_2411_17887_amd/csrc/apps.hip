// Two applications built on the scan, the ones the paper's introduction names as its motivation for
// putting prefix sums on the matrix unit: stream compaction (the "split" / "pack" primitive) and, through
// Blelloch's reduction of radix sort to prefix sums, sorting ("can TCU sort?").
//
// This file checks the arguments and picks the form.  Compaction and the fused one-bit split are kernels around the
// int8 -> int32 MFMA scan of a 0/1 byte mask (tcuscan.hip); the default sort is neither (sort.hip: ranks from ballots, no
// matrix products); the three-kernel split is the reduction spelled out, with kernels here that build the mask and move
// the elements.
//
//   compaction : pos = exclusive_scan(mask);  out[pos[i]] = values[i] where mask[i] != 0
//                (the scatter is fused into the scan kernel: tcuscan.hip, compact_kernel)
//   split(b)   : f[i] = (bit b of key[i] == 0);  pos = exclusive_scan(f);  Z = pos[n-1] + f[n-1]
//                key i goes to  pos[i]            if f[i]      (zeros keep their order, in front)
//                          to  Z + (i - pos[i])   otherwise   (ones keep their order, behind)
//   radix sort : split(0), split(1), ..., split(bits-1)   -- least significant bit first, stable
//                (by default with 256 buckets instead of two, eight bits at a time: sort.hip)

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "../../include/tcuscan.h"
#include "chain_layout.h"

extern "C" tcuscan_status_t tcuscan_internal_compact_fused(const void *d_values, const void *d_mask, void *d_out, size_t n, void *d_positions,
                                                           unsigned *d_count, void *d_ws, size_t ws_bytes, tcuscan_stream_t stream);   // tcuscan.hip
extern "C" tcuscan_status_t tcuscan_internal_bit_zero_counts(const void *d_keys, size_t n, unsigned *d_counts32, tcuscan_stream_t stream);
extern "C" tcuscan_status_t tcuscan_internal_split_pass(const void *d_keys, const void *d_vals, void *d_keys_out, void *d_vals_out, size_t n,
                                                        int bit, const unsigned *d_zeros_total, void *d_ws, size_t ws_bytes,
                                                        tcuscan_stream_t stream);

extern "C" tcuscan_status_t tcuscan_internal_digit_sort(void *d_keys, void *d_vals, size_t n, int bits, void *d_keys_tmp, void *d_vals_tmp,
                                                        void *d_scratch, void *d_fault, tcuscan_stream_t stream);              // sort.hip

namespace {

constexpr int kThreads = 256;

__global__ __launch_bounds__(kThreads) void bit_is_zero_kernel(const uint32_t *__restrict__ keys, int8_t *__restrict__ flags,
                                                               size_t n, int bit)
{
    // 16 keys per thread: one 16-byte store of flags
    const size_t g = (size_t)blockIdx.x * kThreads + threadIdx.x;
    const size_t i0 = g * 16;
    if (i0 + 16 <= n) {
        uint32_t w[4];
        for (int q = 0; q < 4; ++q) {
            const uint4 k = ((const uint4 *)keys)[g * 4 + q];
            w[q] = (((k.x >> bit) & 1u) ^ 1u) | ((((k.y >> bit) & 1u) ^ 1u) << 8) | ((((k.z >> bit) & 1u) ^ 1u) << 16) |
                   ((((k.w >> bit) & 1u) ^ 1u) << 24);
        }
        ((uint4 *)flags)[g] = make_uint4(w[0], w[1], w[2], w[3]);
    } else {
        for (size_t i = i0; i < n; ++i) flags[i] = (int8_t)(((keys[i] >> bit) & 1u) ^ 1u);
    }
}

__global__ __launch_bounds__(kThreads) void split_scatter_kernel(const uint32_t *__restrict__ keys, const uint32_t *__restrict__ vals,
                                                                 const int8_t *__restrict__ flags, const int32_t *__restrict__ pos,
                                                                 uint32_t *__restrict__ keys_out, uint32_t *__restrict__ vals_out, size_t n)
{
    const size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= n) return;
    const uint32_t zeros = (uint32_t)pos[n - 1] + (uint32_t)flags[n - 1];       // total number of keys whose bit is 0
    const uint32_t p = (uint32_t)pos[i];
    const uint32_t dst = flags[i] ? p : zeros + ((uint32_t)i - p);
    keys_out[dst] = keys[i];
    if (vals) vals_out[dst] = vals[i];
}

__global__ __launch_bounds__(kThreads) void copy_u32_kernel(const uint32_t *__restrict__ src, uint32_t *__restrict__ dst, size_t n)
{
    const size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

unsigned blocks_for(size_t items) { return (unsigned)((items + kThreads - 1) / kThreads); }

// measurement / test knob, see tcuscan_set_sort_fusion: 1 passes on eight bits, 2 fused passes on one bit, 0 three
// kernels per bit.  One atomic word, read once at the top of a sort, so that a change made by another thread while a
// sort is being enqueued cannot mix the forms (or their count tables) within that sort.
std::atomic<int> g_sort_form{1};

}  // namespace

extern "C" {

tcuscan_status_t tcuscan_compact_u32(const void *d_values, const void *d_mask, void *d_out, size_t n,
                                     void *d_positions, unsigned *d_count,
                                     void *d_ws, size_t ws_bytes, tcuscan_stream_t stream)
{
    if (n == 0) return TCUSCAN_OK;
    if (n > 0xFFFFFFFFull) return TCUSCAN_ERR_UNSUPPORTED;                       // positions are 32-bit
    if (!d_values || !d_mask || !d_out) return TCUSCAN_ERR_INVALID_ARG;
    if (((uintptr_t)d_values % 4) || ((uintptr_t)d_out % 4) || ((uintptr_t)d_positions % 4) || ((uintptr_t)d_count % 4))
        return TCUSCAN_ERR_INVALID_ARG;
    if (d_positions) {
        // what the scan of the mask into the positions asks for, and callers have sized their workspace by
        if (d_positions == d_mask) return TCUSCAN_ERR_INVALID_ARG;
        const size_t need = chain_layout::bytes_for(n, chain_layout::kSmallTile);
        if (need && (!d_ws || ws_bytes < need || ((uintptr_t)d_ws % 8) != 0)) return TCUSCAN_ERR_WORKSPACE;
    }
    return tcuscan_internal_compact_fused(d_values, d_mask, d_out, n, d_positions, d_count, d_ws, ws_bytes, stream);
}

tcuscan_status_t tcuscan_split_radix_sort_u32(void *d_keys, void *d_vals, size_t n, int bits,
                                              void *d_keys_tmp, void *d_vals_tmp, void *d_flags, void *d_positions,
                                              void *d_ws, size_t ws_bytes, tcuscan_stream_t stream)
{
    if (bits < 0 || bits > 32) return TCUSCAN_ERR_INVALID_ARG;
    if (n <= 1 || bits == 0) return TCUSCAN_OK;
    if (n > 0xFFFFFFFFull) return TCUSCAN_ERR_UNSUPPORTED;
    if (!d_keys || !d_keys_tmp || !d_flags || !d_positions || (d_vals && !d_vals_tmp)) return TCUSCAN_ERR_INVALID_ARG;
    if (((uintptr_t)d_keys % 16) || ((uintptr_t)d_keys_tmp % 16) || ((uintptr_t)d_flags % 16) || ((uintptr_t)d_positions % 4) ||
        ((uintptr_t)d_vals % 4) || ((uintptr_t)d_vals_tmp % 4))
        return TCUSCAN_ERR_INVALID_ARG;
    if (!d_vals) d_vals_tmp = nullptr;                       // (below, source and destination change places: neither may look like payloads)
    hipStream_t s = (hipStream_t)stream;
    uint32_t *src_k = (uint32_t *)d_keys, *dst_k = (uint32_t *)d_keys_tmp;
    uint32_t *src_v = (uint32_t *)d_vals, *dst_v = (uint32_t *)d_vals_tmp;
    int8_t *flags = (int8_t *)d_flags;
    int32_t *pos = (int32_t *)d_positions;
    const int form = g_sort_form.load(std::memory_order_relaxed);
    // The default: passes on eight bits, or the whole sort in one workgroup (sort.hip); the first words of d_positions
    // hold the digit counts and the carry chain's status words.  The chain of 16384 keys to a tile (8192 with payloads)
    // that two-bit passes ran through the workspace is what callers have sized it for: a call that needs it is refused
    // without it, although only its fault word is used.
    if (form == 1) {
        const size_t need = chain_layout::bytes_for(n, d_vals && bits >= 2 ? chain_layout::kFlagTile / 2 : chain_layout::kFlagTile);
        if (need && (!d_ws || ws_bytes < need || ((uintptr_t)d_ws % 8) != 0)) return TCUSCAN_ERR_WORKSPACE;
        return tcuscan_internal_digit_sort(d_keys, d_vals, n, bits, d_keys_tmp, d_vals_tmp, d_positions, need ? d_ws : nullptr, stream);
    }
    // Form 2, one bit per pass: the mask and the positions are never written; the split kernel builds the flags from the
    // keys, scans them and scatters in one go.  How many keys have a zero at each bit does not change when the keys are
    // permuted: it is counted once, up front, into the first 32 words of d_positions.  The unfused form below (mask
    // kernel, tcuscan_exclusive, scatter kernel) remains for n < 96 and as the plain statement of the reduction.
    const bool fused = n >= 96 && form == 2;
    if (fused) {
        unsigned *zeros = (unsigned *)d_positions;
        tcuscan_status_t st = tcuscan_internal_bit_zero_counts(d_keys, n, zeros, stream);
        if (st != TCUSCAN_OK) return st;
        for (int bit = 0; bit < bits; ++bit) {
            st = tcuscan_internal_split_pass(src_k, src_v, dst_k, dst_v, n, bit, zeros + bit, d_ws, ws_bytes, stream);
            if (st != TCUSCAN_OK) return st;
            uint32_t *t = src_k; src_k = dst_k; dst_k = t;
            t = src_v; src_v = dst_v; dst_v = t;
        }
    }
    for (int bit = 0; !fused && bit < bits; ++bit) {
        {
            const uint32_t *k = src_k; void *args[] = {&k, &flags, &n, &bit};
            if (hipLaunchKernel((const void *)bit_is_zero_kernel, dim3(blocks_for((n + 15) / 16)), dim3(kThreads), args, 0, s) != hipSuccess)
                return TCUSCAN_ERR_HIP;
        }
        tcuscan_status_t st = tcuscan_exclusive(flags, pos, n, TCUSCAN_I8_I32, d_ws, ws_bytes, stream);
        if (st != TCUSCAN_OK) return st;
        {
            const uint32_t *k = src_k, *v = src_v; const int8_t *f = flags; const int32_t *p = pos;
            void *args[] = {&k, &v, &f, &p, &dst_k, &dst_v, &n};
            if (hipLaunchKernel((const void *)split_scatter_kernel, dim3(blocks_for(n)), dim3(kThreads), args, 0, s) != hipSuccess)
                return TCUSCAN_ERR_HIP;
        }
        uint32_t *t = src_k; src_k = dst_k; dst_k = t;
        t = src_v; src_v = dst_v; dst_v = t;
    }
    if (src_k != (uint32_t *)d_keys) {                                          // odd number of passes: bring the result home
        const uint32_t *a = src_k; uint32_t *b = (uint32_t *)d_keys;
        void *args[] = {&a, &b, &n};
        if (hipLaunchKernel((const void *)copy_u32_kernel, dim3(blocks_for(n)), dim3(kThreads), args, 0, s) != hipSuccess) return TCUSCAN_ERR_HIP;
        if (d_vals) {
            const uint32_t *av = src_v; uint32_t *bv = (uint32_t *)d_vals;
            void *args2[] = {&av, &bv, &n};
            if (hipLaunchKernel((const void *)copy_u32_kernel, dim3(blocks_for(n)), dim3(kThreads), args2, 0, s) != hipSuccess) return TCUSCAN_ERR_HIP;
        }
    }
    return TCUSCAN_OK;
}

}  // extern "C"

extern "C" tcuscan_status_t tcuscan_set_sort_fusion(int fused)
{
    if (fused < 0 || fused > 2) return TCUSCAN_ERR_INVALID_ARG;
    g_sort_form.store(fused, std::memory_order_relaxed);
    return TCUSCAN_OK;
}
