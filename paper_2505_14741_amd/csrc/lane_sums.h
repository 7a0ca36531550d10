// Sums and maxima over lanes on the vector ALU: DPP moves inside rows of 16 lanes, permlane swaps between rows.  A shuffle
// passes through LDS, about 100 cycles of a chain each; these take about 10.  The pairs and their order are those of a
// butterfly over lane ^ 32, 16, 8, 4, 2, 1.
#pragma once
#include "common.h"

namespace ps {

// the values of lanes l and l ^ 32 (16) in some order
struct LanePair { float a, b; };
__device__ __forceinline__ LanePair lanes_xor32(float v) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return LanePair{__uint_as_float(r[0]), __uint_as_float(r[1])};
}
__device__ __forceinline__ LanePair lanes_xor16(float v) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return LanePair{__uint_as_float(r[0]), __uint_as_float(r[1])};
}
__device__ __forceinline__ float sum_xor32(float v) { const LanePair p = lanes_xor32(v); return p.a + p.b; }
__device__ __forceinline__ float sum_xor16(float v) { const LanePair p = lanes_xor16(v); return p.a + p.b; }
__device__ __forceinline__ float max_xor32(float v) { const LanePair p = lanes_xor32(v); return fmaxf(p.a, p.b); }
__device__ __forceinline__ float max_xor16(float v) { const LanePair p = lanes_xor16(v); return fmaxf(p.a, p.b); }

// DPP controls: rotation of a row by 8 is lane ^ 8; of values that repeat every 8 lanes, by 4, lane ^ 4
constexpr int DPP_ROW_ROR_8 = 0x128, DPP_ROW_ROR_4 = 0x124, DPP_QUAD_XOR_2 = 0x4E, DPP_QUAD_XOR_1 = 0xB1;
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
    return __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
    const unsigned long long u = __double_as_longlong(v);
    const unsigned lo = __builtin_amdgcn_update_dpp(0u, (unsigned)u, CTRL, 0xf, 0xf, true);
    const unsigned hi = __builtin_amdgcn_update_dpp(0u, (unsigned)(u >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double((long long)((unsigned long long)hi << 32 | lo));
}
__device__ __forceinline__ double sum_xor32(double v) {
    const unsigned long long u = __double_as_longlong(v);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)u, (unsigned)u, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(u >> 32), (unsigned)(u >> 32), false, false);
    return __longlong_as_double((long long)((unsigned long long)hi[0] << 32 | lo[0])) +
           __longlong_as_double((long long)((unsigned long long)hi[1] << 32 | lo[1]));
}
__device__ __forceinline__ double sum_xor16(double v) {
    const unsigned long long u = __double_as_longlong(v);
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)u, (unsigned)u, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(u >> 32), (unsigned)(u >> 32), false, false);
    return __longlong_as_double((long long)((unsigned long long)hi[0] << 32 | lo[0])) +
           __longlong_as_double((long long)((unsigned long long)hi[1] << 32 | lo[1]));
}

// over the 16 lanes of a row / all 64 lanes, in every lane (all lanes active)
template <typename T>
__device__ __forceinline__ T sum_of_16(T v) {
    v += dpp<DPP_ROW_ROR_8>(v);
    v += dpp<DPP_ROW_ROR_4>(v);
    v += dpp<DPP_QUAD_XOR_2>(v);
    v += dpp<DPP_QUAD_XOR_1>(v);
    return v;
}
template <typename T>
__device__ __forceinline__ T sum_of_64(T v) { return sum_of_16(sum_xor16(sum_xor32(v))); }

}  // namespace ps
