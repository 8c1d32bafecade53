// Sums and scans across the 64 lanes of a wavefront, on DPP lane moves (no LDS), and its lanes' order in LDS.  Shared by the kernels' sources.
#ifndef TCUSCAN_WAVE_OPS_H
#define TCUSCAN_WAVE_OPS_H

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace {

template <class To, class From> __device__ __forceinline__ To bits(From v) { return __builtin_bit_cast(To, v); }

template <int CTRL> __device__ __forceinline__ uint32_t dpp0(uint32_t v)
{   // lanes whose DPP source does not exist receive 0
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, false);
}
constexpr int kRowShr = 0x110;   // DPP control: shift right by n lanes inside each row of 16
constexpr int kQuadPerm1032 = 0xB1, kQuadPerm2301 = 0x4E;      // lanes 0 to 3 of each four from lanes 1, 0, 3, 2 / 2, 3, 0, 1

__device__ __forceinline__ float    acc_add(float a, float b)       { return a + b; }
__device__ __forceinline__ uint32_t acc_add(uint32_t a, uint32_t b) { return a + b; }
__device__ __forceinline__ uint32_t acc_bits(float a)    { return bits<uint32_t>(a); }
__device__ __forceinline__ uint32_t acc_bits(uint32_t a) { return a; }
template <class A> __device__ __forceinline__ A acc_from_bits(uint32_t b);
template <> __device__ __forceinline__ float    acc_from_bits<float>(uint32_t b)    { return bits<float>(b); }
template <> __device__ __forceinline__ uint32_t acc_from_bits<uint32_t>(uint32_t b) { return b; }

template <class A, int CTRL> __device__ __forceinline__ A dpp_shr(A v) { return acc_from_bits<A>(dpp0<CTRL>(acc_bits(v))); }

// What an LDS access of one lane wrote, other lanes of the wavefront see from here on.
__device__ __forceinline__ void wavefront_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Sum over the 64 lanes, returned wave-uniform.  Row-local DPP shifts give every row's total in its
// lane 15; row_bcast15 / row_bcast31 fold the four row totals into lane 63.
constexpr int kRowBcast15 = 0x142, kRowBcast31 = 0x143;
template <class A> __device__ __forceinline__ A wave_inclusive_scan(A v)
{   // lane l receives v[0] + ... + v[l]
    v = acc_add(v, dpp_shr<A, kRowShr + 1>(v));
    v = acc_add(v, dpp_shr<A, kRowShr + 2>(v));
    v = acc_add(v, dpp_shr<A, kRowShr + 4>(v));
    v = acc_add(v, dpp_shr<A, kRowShr + 8>(v));
    v = acc_add(v, acc_from_bits<A>((uint32_t)__builtin_amdgcn_update_dpp(0, (int)acc_bits(v), kRowBcast15, 0xa, 0xf, false)));
    v = acc_add(v, acc_from_bits<A>((uint32_t)__builtin_amdgcn_update_dpp(0, (int)acc_bits(v), kRowBcast31, 0xc, 0xf, false)));
    return v;
}
template <class A> __device__ __forceinline__ A wave_sum(A v)
{
    return acc_from_bits<A>((uint32_t)__builtin_amdgcn_readlane((int)acc_bits(wave_inclusive_scan(v)), 63));
}
// Bits set in any lane / the largest of the 64 lanes' values, wave-uniform.
template <class Fold> __device__ __forceinline__ uint32_t wave_fold(uint32_t v, Fold fold)
{   // (0 is the neutral element)
    v = fold(v, dpp0<kRowShr + 1>(v));
    v = fold(v, dpp0<kRowShr + 2>(v));
    v = fold(v, dpp0<kRowShr + 4>(v));
    v = fold(v, dpp0<kRowShr + 8>(v));
    v = fold(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kRowBcast15, 0xa, 0xf, false));
    v = fold(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kRowBcast31, 0xc, 0xf, false));
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ __forceinline__ uint32_t wave_or(uint32_t v)  { return wave_fold(v, [](uint32_t a, uint32_t b) { return a | b; }); }
__device__ __forceinline__ uint32_t wave_max(uint32_t v) { return wave_fold(v, [](uint32_t a, uint32_t b) { return a > b ? a : b; }); }
// The same and the sum over lanes 0 to 15.
template <class Fold> __device__ __forceinline__ uint32_t row_fold(uint32_t v, Fold fold)
{
    v = fold(v, dpp0<kRowShr + 1>(v));
    v = fold(v, dpp0<kRowShr + 2>(v));
    v = fold(v, dpp0<kRowShr + 4>(v));
    v = fold(v, dpp0<kRowShr + 8>(v));
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 15);
}
__device__ __forceinline__ uint32_t row_or(uint32_t v)  { return row_fold(v, [](uint32_t a, uint32_t b) { return a | b; }); }
__device__ __forceinline__ uint32_t row_sum(uint32_t v) { return row_fold(v, [](uint32_t a, uint32_t b) { return a + b; }); }
constexpr int kWaveShr1 = 0x138;   // DPP control: shift right by one lane across the whole wavefront
template <class A> __device__ __forceinline__ A wave_shift_up(A v)
{   // lane l receives v[l - 1], lane 0 receives 0
    return dpp_shr<A, kWaveShr1>(v);
}

template <class A> __device__ __forceinline__ A uniform_from_lane(A v, int lane)
{   // wave-uniform copy of one lane's value
    return acc_from_bits<A>((uint32_t)__builtin_amdgcn_readlane((int)acc_bits(v), lane));
}

}  // namespace

#endif
