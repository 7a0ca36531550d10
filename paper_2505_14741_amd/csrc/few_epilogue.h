// Epilogues of the few-token kernels: a lane holds 4 adjacent output columns of one row.
#pragma once
#include "tile_ops.h"

namespace ps {

// GELU where the result stays fp32: x over 1 + 2^t, the quotient refined once, for the sum as it is before its rounding (19
// instructions; with the math library's tanh, whose two branches a wave both takes, 35).  The rounding of the sum counts in full
// where 2^t is small, i.e. for x > 0: left in, the error against 64 bits over N(0, 1) is 4.21e-8 of the result's norm, carried
// 2.72e-8, with the tanh form 3.75e-8.  Where the sum would not be finite (from x = -10 down) the result is a zero,
// NaN for -infinity, as with the tanh; where it is 1 in fp32 the quotient of an infinite x must not be refined.
__device__ __forceinline__ float gelu_of(float x, float) {
    constexpr float c0 = -2.0f * 0.7978845608028654f * 1.4426950408889634f, c1 = c0 * 0.044715f;
    const float t = x * __builtin_fmaf(c1 * x, x, c0);
    const float e = __builtin_amdgcn_exp2f(t), d = 1.0f + e, lost = e - (d - 1.0f);
    const float r = __builtin_amdgcn_rcpf(d), y = x * r;
    const float g = __builtin_fmaf(__builtin_fmaf(-lost, y, __builtin_fmaf(-d, y, x)), r, y);
    return t < -64.0f ? x : t > 126.0f ? x * 0.0f : g;
}
__device__ __forceinline__ float gelu_of(float x, bf16_t) { return gelu_fast(x); }

__device__ __forceinline__ void store_quad(float* p, f32x4_t v) { *reinterpret_cast<f32x4_t*>(p) = v; }
__device__ __forceinline__ void store_quad(bf16_t* p, f32x4_t v) {
    *reinterpret_cast<bf16x4_t*>(p) = __builtin_convertvector(v, bf16x4_t);
}

// A row of the batch's rows: sample and token, and for the rotation the position on the three axes.
struct EpiRow { int sample, n, pos[3]; };
template <int KIND>
__device__ __forceinline__ EpiRow epilogue_row(const Epilogue& ep, int row) {
    EpiRow r;
    r.sample = row / ep.geom.tokens;
    r.n = row - r.sample * ep.geom.tokens;
    if constexpr (KIND == EPI_QKV_ROPE) {
        const int nv = r.n - ep.geom.text_tokens, q1 = nv / ep.rope_Wp, q2 = q1 / ep.rope_Hp;
        r.pos[0] = q2; r.pos[1] = q1 - q2 * ep.rope_Hp; r.pos[2] = nv - q1 * ep.rope_Wp;
    }
    return r;
}

// What the epilogue of 4 adjacent columns of a row reads besides the sum and the bias; aux: the residual, or (cos, sin) of both
// pairs.
struct EpiOperands { f32x4_t gate, aux; };
template <int KIND>
__device__ __forceinline__ EpiOperands epilogue_operands(const Epilogue& ep, int Nn, const EpiRow& r, int row, int col) {
    EpiOperands o;
    o.gate = f32x4_t{0.f, 0.f, 0.f, 0.f};
    o.aux = f32x4_t{0.f, 0.f, 0.f, 0.f};
    if constexpr (KIND == EPI_GATE_RESIDUAL) {
        o.gate = *reinterpret_cast<const f32x4_t*>(ep.mod_layer + r.sample * ep.mod_batch_stride +
                                                   (long)(ep.gate_chunk + (r.n < ep.geom.text_tokens ? 6 : 0)) * ep.D + col);
        o.aux = *reinterpret_cast<const f32x4_t*>(ep.resid + (long)row * Nn + col);
    }
    if constexpr (KIND == EPI_QKV_ROPE) {
        if (r.n >= ep.geom.text_tokens && col < 2 * ep.D) {
            const int pr = (col % ep.head_dim) >> 1;
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const RopeAxis ra = rope_axis_of(pr + c, ep.head_dim, ep.rope_F, ep.rope_Hp);
                const f32x2_t cs = *reinterpret_cast<const f32x2_t*>(
                    ep.rope_cs + ra.base + (ra.axis == 0 ? r.pos[0] : ra.axis == 1 ? r.pos[1] : r.pos[2]) * ra.stride);
                o.aux[2 * c] = cs[0];
                o.aux[2 * c + 1] = cs[1];
            }
        }
    }
    return o;
}

// x is the finished sum.
template <int KIND, typename T>
__device__ __forceinline__ void epilogue_quad(const Epilogue& ep, T* __restrict__ C, int Nn, const EpiRow& r, int row, int col,
                                              f32x4_t x, f32x4_t bias, const EpiOperands& o) {
    x += bias;
    if constexpr (KIND == EPI_BIAS_GELU) {
#pragma unroll
        for (int c = 0; c < 4; ++c) x[c] = gelu_of(x[c], T{});
    }
    if constexpr (KIND == EPI_GATE_RESIDUAL) {
        *reinterpret_cast<f32x4_t*>(ep.resid + (long)row * Nn + col) = gated_sum(o.aux, o.gate, x);
        return;
    }
    if constexpr (KIND == EPI_UNPATCHIFY) {
        const int text = ep.geom.text_tokens;
        if (r.n < text) return;
        const PatchGeom& g = ep.pg;
        const int Hp = g.H / g.patch, Wp = g.W / g.patch, nv = r.n - text;
        const int pj = nv % Wp, pi = (nv / Wp) % Hp, f = nv / (Wp * Hp);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int q = col + c;
            const int dx = q % g.patch, dy = (q / g.patch) % g.patch, ch = q / (g.patch * g.patch);
            ep.resid[((((long)r.sample * g.C + ch) * g.F + f) * g.H + (pi * g.patch + dy)) * g.W + (pj * g.patch + dx)] = x[c];
        }
        return;
    }
    if constexpr (KIND == EPI_QKV_ROPE) {
        if (r.n >= ep.geom.text_tokens && col < 2 * ep.D) x = rotate_quad(x, o.aux);
        if (col < ep.D) x *= ep.q_scale;
    }
    store_quad(C + (long)row * Nn + col, x);
}

// Adds the K pieces ([piece][row][column]) in order and applies the epilogue: one thread per 4 adjacent columns.
template <typename T, int KIND>
__global__ void __launch_bounds__(256)
gemm_few_reduce_kernel(T* __restrict__ C, int Nn, long rows, int nsplit, Epilogue ep) {
    const int quads = Nn / 4;
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= rows * quads) return;
    const long row = idx / quads;
    const int col = (int)(idx - row * quads) * 4;
    f32x4_t s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int p = 0; p < nsplit; ++p) s += *reinterpret_cast<const f32x4_t*>(ep.split_ws + (p * rows + row) * Nn + col);
    const EpiRow r = epilogue_row<KIND>(ep, (int)row);
    epilogue_quad<KIND, T>(ep, C, Nn, r, (int)row, col, s, *reinterpret_cast<const f32x4_t*>(ep.bias + col), epilogue_operands<KIND>(ep, Nn, r, (int)row, col));
}

}  // namespace ps
