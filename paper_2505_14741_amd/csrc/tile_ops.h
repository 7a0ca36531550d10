// What the matrix kernels share.
#pragma once
#include "common.h"

namespace ps {

typedef __attribute__((ext_vector_type(2))) float f32x2_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4_t;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;

#define PS_LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))

// global->LDS load of 16 bytes per lane, issued from inline asm: lane j's bytes land at lds_addr + 16*j (lds_addr
// wave-uniform, passed through M0).  The compiler does not see the LDS write, so it never orders LDS reads of other stages
// behind loads still in flight; the explicit vmcnt waits and barriers of a kernel make a stage visible before it is read.
__device__ __forceinline__ void lds_dma16(const void* gptr, unsigned lds_addr) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(gptr), "s"(lds_addr)
                 : "memory", "m0");
}

// lds_dma16 from a scalar 64-bit base + per-lane 32-bit byte offset
__device__ __forceinline__ void lds_dma16_base(unsigned voff, const void* sbase, unsigned lds_addr) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(sbase), "s"(lds_addr)
                 : "memory", "m0");
}

// exp(d) for 0 >= d >= EXP_NEAR, where the result is a normal number; NaN stays NaN.  The hardware's exponential of t, which is
// d * log2(e) rounded, times 1 + (d - t * ln 2), what the rounding left out: as exact as the math library's expf in 6
// instructions instead of 13.  (Without the second factor the argument's rounding, |t| * 2^-24, is the result's error: 4.8e-6 at
// d = -80; and log2(e) times a score is not finite from 2.36e38 on, where the difference of two scores is.)
constexpr float EXP_NEAR = -87.0f;
__device__ __forceinline__ float exp_near(float d) {
    constexpr float LN2 = 0.693147182464599609375f, LN2_REST = -1.9046542121259336e-9f;
    const float t = d * 1.4426950408889634f, e = __builtin_amdgcn_exp2f(t);
    return __builtin_fmaf(e, __builtin_fmaf(-t, LN2_REST, __builtin_fmaf(-t, LN2, d)), e);
}

// Consecutive workgroup ids go to different XCDs (8 of them, each with its own L2).
// Give each XCD a contiguous range of tiles so co-resident workgroups share operand panels.
__device__ __forceinline__ int xcd_remap(unsigned id, unsigned total) {
    const unsigned per = total / 8, rem = total % 8, x = id % 8, j = id / 8;
    return (int)(x * per + (x < rem ? x : rem) + j);
}

// ---- Epilogue arithmetic.  Which kernel computes an output depends on the rows of the whole batch, its value must not: the
// kernels share these, with every fused multiply-add written out.

// tanh-form GELU written as x * sigmoid(2u), u = sqrt(2/pi)(x + 0.044715 x^3): two
// transcendentals and four FMAs; used where the result is rounded to bf16.
__device__ __forceinline__ float gelu_fast(float x) {
    constexpr float c0 = -2.0f * 0.7978845608028654f * 1.4426950408889634f, c1 = c0 * 0.044715f;
    const float t = x * __builtin_fmaf(c1 * x, x, c0);
    return x * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(t));
}

// two (even, odd) pairs turned by t = (cos, sin, cos, sin)
__device__ __forceinline__ f32x4_t rotate_quad(f32x4_t x, f32x4_t t) {
    return f32x4_t{__builtin_fmaf(x[0], t[0], -(x[1] * t[1])), __builtin_fmaf(x[1], t[0], x[0] * t[1]),
                   __builtin_fmaf(x[2], t[2], -(x[3] * t[3])), __builtin_fmaf(x[3], t[2], x[2] * t[3])};
}

__device__ __forceinline__ f32x4_t gated_sum(f32x4_t resid, f32x4_t gate, f32x4_t x) {
    return __builtin_elementwise_fma(gate, x, resid);
}

}  // namespace ps
