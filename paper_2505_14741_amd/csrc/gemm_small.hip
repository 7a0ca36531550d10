// C[M, Nn] = A[M, K] * W[Nn, K]^T on matrix instructions for fp32 operands and for bf16 samples of few tokens.
//
// With few tokens a projection is a stream of weights (22 MB for 5760 x 1920 in bf16, 4 us at the 5.1 TB/s a large copy
// reaches) and is bound by latency: a 128 x 128 tile leaves 15 of 256 compute units busy at 112 tokens x 1920 columns, each
// walking all of K with one stage in flight.  Here a workgroup takes 64 x 64 outputs, K is cut into pieces where the tiles
// do not fill the chip, and an LDS ring of 8 stages of 16 KB (one workgroup per CU; 4 stages and two workgroups, 3 and three
// where there are more of them) keeps up to 112 KB of loads in flight.  112 tokens, weights cold, before and after:
// 5760 x 1920 24.1 -> 15.0 us, 7680 x 1920 31.0 -> 16.0, 1920 x 1920 24.4 -> 11.5, 1920 x 7680 106.6 -> 18.5.
// fp32 (v_mfma_f32_16x16x4_f32: full fp32 products and sums) at 112 tokens against the 64 x 64 fp32-FMA kernel:
// 5760 x 1920 229 -> 43 us, 1920 x 7680 ~900 -> 45 us; at 512 tokens 101 TFLOP/s.
#include "common.h"
#include "plan.h"
#include <type_traits>


namespace ps {

typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4_t;

static constexpr int TILE = FEW_TILE;                    // output rows and columns of a workgroup
static constexpr int ROWB = FEW_ROW_BYTES;               // bytes of an operand row per stage: 64 bf16 or 32 fp32
static constexpr int STAGE = 2 * TILE * ROWB;            // A rows, then W rows

// global->LDS load of 16 bytes per lane; lane j's bytes land at lds_addr + 16*j (lds_addr wave-uniform)
__device__ __forceinline__ void lds_dma16(const void* gptr, unsigned lds_addr) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(gptr), "s"(lds_addr)
                 : "memory", "m0");
}

// the loads of at most `stages` stages (4 instructions each) may stay in flight
__device__ __forceinline__ void wait_stages(int stages) {
    switch (stages) {
        case 0: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
        case 1: asm volatile("s_waitcnt vmcnt(4)" ::: "memory"); break;
        case 2: asm volatile("s_waitcnt vmcnt(8)" ::: "memory"); break;
        case 3: asm volatile("s_waitcnt vmcnt(12)" ::: "memory"); break;
        case 4: asm volatile("s_waitcnt vmcnt(16)" ::: "memory"); break;
        case 5: asm volatile("s_waitcnt vmcnt(20)" ::: "memory"); break;
        default: asm volatile("s_waitcnt vmcnt(24)" ::: "memory"); break;
    }
}

__device__ __forceinline__ float gelu_of(float x, float) { return gelu_tanh_f(x); }
// where the result is rounded to bf16: x * sigmoid(2u), u = sqrt(2/pi)(x + 0.044715 x^3)
__device__ __forceinline__ float gelu_of(float x, bf16_t) {
    const float c0 = -2.0f * 0.7978845608028654f * 1.4426950408889634f;
    const float t = x * (c0 + c0 * 0.044715f * x * x);
    return x * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(t));
}

__device__ __forceinline__ void store_quad(float* p, f32x4_t v) { *reinterpret_cast<f32x4_t*>(p) = v; }
__device__ __forceinline__ void store_quad(bf16_t* p, f32x4_t v) {
    *reinterpret_cast<bf16x4_t*>(p) = __builtin_convertvector(v, bf16x4_t);
}

// What the epilogue of 4 adjacent output columns of row n of a sample reads besides the sum.
struct EpiOperands { f32x4_t bias, gate, resid; };
template <int KIND>
__device__ __forceinline__ EpiOperands epilogue_operands(const Epilogue& ep, int Nn, int sample, int n, int col) {
    EpiOperands o;
    o.bias = *reinterpret_cast<const f32x4_t*>(ep.bias + col);
    o.gate = o.resid = f32x4_t{0.f, 0.f, 0.f, 0.f};
    if constexpr (KIND == EPI_GATE_RESIDUAL) {
        o.gate = *reinterpret_cast<const f32x4_t*>(ep.mod_layer + sample * ep.mod_batch_stride +
                                                   (long)(ep.gate_chunk + (n < ep.geom.text_tokens ? 6 : 0)) * ep.D + col);
        o.resid = *reinterpret_cast<const f32x4_t*>(ep.resid + ((long)sample * ep.geom.tokens + n) * Nn + col);
    }
    return o;
}

// x is the finished sum.
template <int KIND, typename T>
__device__ __forceinline__ void epilogue_quad(const Epilogue& ep, T* __restrict__ C, int Nn, int sample, int n, int col,
                                              f32x4_t x, const EpiOperands& o) {
    const long row = (long)sample * ep.geom.tokens + n;
    const int text = ep.geom.text_tokens;
    x += o.bias;
    if constexpr (KIND == EPI_BIAS_GELU) {
#pragma unroll
        for (int c = 0; c < 4; ++c) x[c] = gelu_of(x[c], T{});
    }
    if constexpr (KIND == EPI_GATE_RESIDUAL) {
        *reinterpret_cast<f32x4_t*>(ep.resid + row * Nn + col) = o.resid + o.gate * x;
        return;
    }
    if constexpr (KIND == EPI_UNPATCHIFY) {
        if (n < text) return;
        const PatchGeom& g = ep.pg;
        const int Hp = g.H / g.patch, Wp = g.W / g.patch, nv = n - text;
        const int pj = nv % Wp, pi = (nv / Wp) % Hp, f = nv / (Wp * Hp);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int o = col + c;
            const int dx = o % g.patch, dy = (o / g.patch) % g.patch, ch = o / (g.patch * g.patch);
            ep.resid[((((long)sample * g.C + ch) * g.F + f) * g.H + (pi * g.patch + dy)) * g.W + (pj * g.patch + dx)] = x[c];
        }
        return;
    }
    if constexpr (KIND == EPI_QKV_ROPE) {
        if (n >= text && col < 2 * ep.D) {
            const int nv = n - text, q1 = nv / ep.rope_Wp, q2 = q1 / ep.rope_Hp;
            const int pos[3] = {q2, q1 - q2 * ep.rope_Hp, nv - q1 * ep.rope_Wp};
            const int pr = (col % ep.head_dim) >> 1;
#pragma unroll
            for (int c = 0; c < 4; c += 2) {
                const RopeAxis ra = rope_axis_of(pr + c / 2, ep.head_dim, ep.rope_F, ep.rope_Hp);
                const float* cs = ep.rope_cs + ra.base + (ra.axis == 0 ? pos[0] : ra.axis == 1 ? pos[1] : pos[2]) * ra.stride;
                const float v0 = x[c], v1 = x[c + 1];
                x[c] = v0 * cs[0] - v1 * cs[1];
                x[c + 1] = v1 * cs[0] + v0 * cs[1];
            }
        }
        if (col < ep.D) x *= ep.q_scale;
    }
    store_quad(C + row * Nn + col, x);
}

// Workgroup -> (sample, tile, K piece).  Ids that share an XCD are contiguous (see the remap in the kernel); the row
// tiles of all samples that read one W panel come first, so the panel is fetched into that XCD's L2 once.  With more
// than 8 row tiles the tiles go in bands of 8 rows instead.
struct SmallGrid { int batch, tiles_m, tiles_n, nsplit; };

// INREG: one workgroup per tile walks all of K and adds the nsplit pieces up in registers, in the order and with the
// roundings of the reduction.
template <typename T, int KIND, int NST, bool INREG>
__global__ void __launch_bounds__(256, NST == 3 ? 3 : NST == 4 ? 2 : 1)
gemm_small_kernel(const T* __restrict__ A, const T* __restrict__ W, T* __restrict__ C, int Nn, int K, SmallGrid g,
                  Epilogue ep) {
    __shared__ __attribute__((aligned(1024))) unsigned char lds[NST * STAGE];
    const int tokens = ep.geom.tokens, pieces = INREG ? 1 : g.nsplit;    // workgroups along K per tile
    int id, sample, piece, m0, n0;
    {
        const int total = gridDim.x, per = total / 8, rem = total % 8, x = blockIdx.x % 8;
        id = x * per + (x < rem ? x : rem) + blockIdx.x / 8;
    }
    if (g.tiles_m <= 8) {
        m0 = id % g.tiles_m * TILE; id /= g.tiles_m;
        sample = id % g.batch;      id /= g.batch;
        piece = id % pieces;      n0 = id / pieces * TILE;
    } else {
        const int tiles = g.tiles_m * g.tiles_n, tile = id % tiles;
        id /= tiles;
        piece = id % pieces; sample = id / pieces;
        const int band = tile / (8 * g.tiles_n), in_band = tile % (8 * g.tiles_n);
        const int rows_here = min(8, g.tiles_m - band * 8);
        m0 = (band * 8 + in_band % rows_here) * TILE;
        n0 = in_band / rows_here * TILE;
    }
    const int nk = K / (ROWB / (int)sizeof(T));
    const int k0 = nk * piece / pieces, nkt = nk * (piece + 1) / pieces - k0;

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1, l16 = lane & 15, kgrp = lane >> 4;

    // load group q = 8 rows of the stage [64 A rows | 64 W rows]; slot p of row r holds 16-byte chunk p ^ ((r >> 1) & 7),
    // so the 16 rows of a fragment read fall into 16 different bank groups; rows past the edge re-read the last one
    const char* gp[4];
    const long row_bytes = (long)K * sizeof(T);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int row = (wave + 4 * i) * 8 + (lane >> 3);
        const int chunk = (lane & 7) ^ ((row >> 1) & 7);
        const char* base = row < TILE
            ? reinterpret_cast<const char*>(A) + ((long)sample * tokens + min(m0 + row, tokens - 1)) * row_bytes
            : reinterpret_cast<const char*>(W) + (long)min(n0 + row - TILE, Nn - 1) * row_bytes;
        gp[i] = base + chunk * 16 + (long)k0 * ROWB;
    }
    const unsigned lds_base = (unsigned)(size_t)((__attribute__((address_space(3))) void*)lds);
    auto issue = [&](int kt) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            lds_dma16(gp[i] + (long)kt * ROWB,
                      __builtin_amdgcn_readfirstlane(lds_base + (kt % NST) * STAGE + (wave + 4 * i) * 1024));
    };

    // W fragments are the first operand, A fragments the second: lane l of a 16 x 16 result then holds 4 adjacent
    // output columns (4 * (l / 16) ..) of row l % 16, and the epilogue works on 16-byte quads without a transpose
    // (fp32: the two k steps of a stage have sums of their own, a shorter chain of roundings: error of the fp32 step on
    // 112 tokens against 64 bits 5.3e-7 with them, 5.5e-7 without, 1.36e-6 on the fp32-FMA kernel)
    constexpr int SETS = sizeof(T) == 4 ? 2 : 1;
    f32x4_t acc[SETS][2][2];                             // [set][16 columns][16 rows]
#pragma unroll
    for (int z = 0; z < SETS; ++z)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int x = 0; x < 2; ++x) acc[z][y][x] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    auto piece_sum = [&](int y, int x) {
        f32x4_t v = acc[0][y][x];
        if constexpr (SETS == 2) v += acc[1][y][x];
        return v;
    };
    f32x4_t total[2][2];                                 // INREG: the pieces before the current one
    int piece_end = INREG ? nk / g.nsplit : 0, piece_no = 1;
    if constexpr (INREG) {
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int x = 0; x < 2; ++x) total[y][x] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
    const int aoff = (wm * 32 + l16) * ROWB, woff = (TILE + wn * 32 + l16) * ROWB, sw = (l16 >> 1) & 7;

    // the epilogue's operands are requested now, with the first stages, and not when the sums are done
    // (rows and columns past the edge: clamped, not stored)
    EpiOperands eo[2][2];
    if (pieces == 1) {
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y)
                eo[x][y] = epilogue_operands<KIND>(ep, Nn, sample, min(m0 + wm * 32 + x * 16 + l16, tokens - 1),
                                                   min(n0 + wn * 32 + y * 16 + kgrp * 4, Nn - 4));
    }
    for (int p = 0; p < NST - 1 && p < nkt; ++p) issue(p);
    for (int kt = 0; kt < nkt; ++kt) {
        wait_stages(min(NST - 2, nkt - 1 - kt));         // own share of stage kt has landed
        __syncthreads();                                 // ... everyone's, and nobody reads stage kt - 1 any more
        if (kt + NST - 1 < nkt) issue(kt + NST - 1);
        const unsigned char* st = lds + (kt % NST) * STAGE;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const int slot = ((ks * 4 + kgrp) ^ sw) << 4;
            if constexpr (sizeof(T) == 2) {
                bf16x8_t a[2], w[2];
#pragma unroll
                for (int x = 0; x < 2; ++x) {
                    a[x] = *reinterpret_cast<const bf16x8_t*>(st + aoff + x * 16 * ROWB + slot);
                    w[x] = *reinterpret_cast<const bf16x8_t*>(st + woff + x * 16 * ROWB + slot);
                }
#pragma unroll
                for (int y = 0; y < 2; ++y)
#pragma unroll
                    for (int x = 0; x < 2; ++x)
                        acc[0][y][x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[y], a[x], acc[0][y][x], 0, 0, 0);
            } else {
                // one 16-byte read gives a lane 4 adjacent k: instruction e multiplies the k = 4 * group + e
                f32x4_t a[2], w[2];
#pragma unroll
                for (int x = 0; x < 2; ++x) {
                    a[x] = *reinterpret_cast<const f32x4_t*>(st + aoff + x * 16 * ROWB + slot);
                    w[x] = *reinterpret_cast<const f32x4_t*>(st + woff + x * 16 * ROWB + slot);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int y = 0; y < 2; ++y)
#pragma unroll
                        for (int x = 0; x < 2; ++x)
                            acc[ks][y][x] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[y][e], a[x][e], acc[ks][y][x], 0, 0, 0);
            }
        }
        if constexpr (INREG) {
            if (kt + 1 == piece_end) {                   // (the last piece ends with the last stage)
#pragma unroll
                for (int y = 0; y < 2; ++y)
#pragma unroll
                    for (int x = 0; x < 2; ++x) {
                        total[y][x] += piece_sum(y, x);
#pragma unroll
                        for (int z = 0; z < SETS; ++z) acc[z][y][x] = f32x4_t{0.f, 0.f, 0.f, 0.f};
                    }
                ++piece_no;
                piece_end = nk * piece_no / g.nsplit;
            }
        }
    }
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        const int n = m0 + wm * 32 + x * 16 + l16;
        if (n >= tokens) continue;
#pragma unroll
        for (int y = 0; y < 2; ++y) {
            const int col = n0 + wn * 32 + y * 16 + kgrp * 4;
            if (col >= Nn) continue;
            const f32x4_t sum = INREG ? total[y][x] : piece_sum(y, x);
            if (pieces > 1)                              // [piece][row][column]
                *reinterpret_cast<f32x4_t*>(ep.split_ws + (((long)piece * g.batch + sample) * tokens + n) * Nn + col) = sum;
            else
                epilogue_quad<KIND, T>(ep, C, Nn, sample, n, col, sum, eo[x][y]);
        }
    }
}

// Adds the K pieces in order and applies the epilogue: one thread per 4 adjacent columns.
template <typename T, int KIND>
__global__ void __launch_bounds__(256)
gemm_small_reduce_kernel(T* __restrict__ C, int Nn, SmallGrid g, Epilogue ep) {
    const int quads = Nn / 4;
    const long rows = (long)g.batch * ep.geom.tokens, idx = (long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= rows * quads) return;
    const long row = idx / quads;
    const int col = (int)(idx - row * quads) * 4;
    f32x4_t s = {0.f, 0.f, 0.f, 0.f};
    for (int p = 0; p < g.nsplit; ++p) s += *reinterpret_cast<const f32x4_t*>(ep.split_ws + (p * rows + row) * Nn + col);
    const int sample = (int)(row / ep.geom.tokens);
    const int n = (int)(row - (long)sample * ep.geom.tokens);
    epilogue_quad<KIND, T>(ep, C, Nn, sample, n, col, s, epilogue_operands<KIND>(ep, Nn, sample, n, col));
}

template <typename T, int KIND>
static hipError_t launch_small_kind(const T* A, const T* W, T* C, int batch, int tokens, int Nn, int K, const FewPlan& p,
                                    bool inreg, const Epilogue& ep, int* deferred, hipStream_t st) {
    const SmallGrid g{batch, p.tiles_m, p.tiles_n, p.nsplit};
    const int pieces = inreg ? 1 : p.nsplit;
    const long blocks = (long)batch * p.tiles_m * p.tiles_n * pieces;
    if (blocks >= (1L << 31)) return hipErrorInvalidValue;
    auto go = [&](auto kernel) { kernel<<<(int)blocks, 256, 0, st>>>(A, W, C, Nn, K, g, ep); };
    // as deep a ring as lets every workgroup start at once (with two per CU, 513 to 768 are a second, nearly empty round:
    // 1920 x 1920 at 1100 rows, 540 tiles, 23.8 -> 20.8 us with three; 5760 x 1920 at 440, 630 tiles, 23.2 -> 20.7, both
    // with the weights in cache)
    const auto ring = [&](auto in_registers) {
        constexpr bool R = decltype(in_registers)::value;
        if (blocks <= 256) go(gemm_small_kernel<T, KIND, 8, R>);
        else if (blocks <= 512) go(gemm_small_kernel<T, KIND, 4, R>);
        else go(gemm_small_kernel<T, KIND, 3, R>);
    };
    if (inreg && p.nsplit > 1) ring(std::true_type{}); else ring(std::false_type{});
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || pieces == 1) return e;
    if (deferred) { *deferred = p.nsplit; return e; }
    const long quads = (long)batch * tokens * (Nn / 4);
    gemm_small_reduce_kernel<T, KIND><<<(int)((quads + 255) / 256), 256, 0, st>>>(C, Nn, g, ep);
    return hipGetLastError();
}

template <typename T>
static hipError_t launch_small(const T* A, const T* W, T* C, int batch, int tokens, int Nn, int K, const FewPlan& p, bool inreg,
                               const Epilogue& ep, int* deferred, hipStream_t st) {
    switch (ep.kind) {
        case EPI_BIAS: return launch_small_kind<T, EPI_BIAS>(A, W, C, batch, tokens, Nn, K, p, inreg, ep, nullptr, st);
        case EPI_BIAS_GELU: return launch_small_kind<T, EPI_BIAS_GELU>(A, W, C, batch, tokens, Nn, K, p, inreg, ep, nullptr, st);
        case EPI_GATE_RESIDUAL: return launch_small_kind<T, EPI_GATE_RESIDUAL>(A, W, C, batch, tokens, Nn, K, p, inreg, ep, deferred, st);
        case EPI_QKV_ROPE: return launch_small_kind<T, EPI_QKV_ROPE>(A, W, C, batch, tokens, Nn, K, p, inreg, ep, nullptr, st);
        case EPI_UNPATCHIFY: return launch_small_kind<T, EPI_UNPATCHIFY>(A, W, C, batch, tokens, Nn, K, p, inreg, ep, nullptr, st);
        default: return hipErrorInvalidValue;
    }
}

// inreg: one workgroup per tile, the plan's pieces added in registers; else one per piece, through epi.split_ws.
hipError_t launch_gemm_small(int dtype, const void* A, const void* W, void* C, int batch, int tokens, int Nn, int K,
                             const Epilogue& epi, const FewPlan& p, bool inreg, int* deferred, hipStream_t st) {
    Epilogue ep = epi;
    ep.geom.tokens = tokens;                             // (the plain kinds leave it unset)
    if (!p.use) return hipErrorInvalidValue;
    if (dtype == PS_BF16)
        return launch_small<bf16_t>((const bf16_t*)A, (const bf16_t*)W, (bf16_t*)C, batch, tokens, Nn, K, p, inreg, ep, deferred, st);
    return launch_small<float>((const float*)A, (const float*)W, (float*)C, batch, tokens, Nn, K, p, inreg, ep, deferred, st);
}

}  // namespace ps
