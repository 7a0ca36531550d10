// HBM-bound kernels of the denoising step: time conditioning, patch embedding,
// LayerNorm + adaLN modulation, final projection, the fused DDIM update with the
// relative-MAE sums of paper Eq. (1), and the stand-alone relative MAE.
#include "lane_sums.h"

#include <mutex>
#include <type_traits>

namespace ps {

static constexpr int WAVE = 64;

// ------------------------------------------------------------------ time conditioning
struct TList { int t[16]; };

// s(t) = [cos(t w_j) | sin(t w_j)], w_j = 10000^(-j/(D/2)); double precision because
// t*w reaches ~1e3 rad and the result feeds an fp32 MLP compared at 1e-4.
__device__ __forceinline__ void sinusoid_entry(const TList& tl, float* __restrict__ out, int D, int b, int j) {
    int half = D / 2;
    if (j >= half) return;
    double w = exp(-(double)j / (double)half * 9.210340371976184);   // ln(10000)
    double ang = (double)tl.t[b] * w;
    out[(long)b * D + j] = (float)cos(ang);
    out[(long)b * D + half + j] = (float)sin(ang);
}

// One wave per GEMV_ROWS consecutive output rows; weights stream once from HBM (16 bytes per lane and load when the row
// length allows, the loads of the wave's rows in flight together), inputs stay in cache and are read once for the wave's
// rows.  Each row's sum is formed as if the wave had that row alone (same lanes, same order).  Few rows in all (a time MLP
// layer: 512) take a wave each, which spreads the loads and the sums over lanes, one per row and vector, over the chip: 512 rows
// of 1920 bf16 weights, one vector 9.0 -> 5.3 us (8 rows per wave), 64 rows of 64 fp32, nine vectors 20 -> 5 (as measured with
// sums of six shuffles).
// blockIdx.y picks one of up to GEMV_SET matrices of the same shape applied to the same input.
template <typename T, int MAXB, int GEMV_ROWS>
__global__ void gemv_kernel(GemvSet set, const float* __restrict__ in, int rows,
                            int cols, int batch, long in_bs, long out_bs, int act) {
    const int wave = (blockIdx.x * blockDim.x + threadIdx.x) / WAVE;
    const int lane = threadIdx.x % WAVE;
    const int row0 = wave * GEMV_ROWS;
    if (row0 >= rows) return;
    const T* __restrict__ W = static_cast<const T*>(set.W[blockIdx.y]);
    const float* __restrict__ bias = set.bias[blockIdx.y];
    float* __restrict__ out = set.out[blockIdx.y];
    const T* w[GEMV_ROWS];
#pragma unroll
    for (int r = 0; r < GEMV_ROWS; ++r) w[r] = W + (long)min(row0 + r, rows - 1) * cols;   // rows past the end: recomputed, not stored
    float acc[GEMV_ROWS][MAXB];
#pragma unroll
    for (int r = 0; r < GEMV_ROWS; ++r)
#pragma unroll
        for (int b = 0; b < MAXB; ++b) acc[r][b] = 0.f;
    constexpr int VEC = 16 / sizeof(T);                      // elements per 16-byte load
    if (cols % VEC == 0 && in_bs % 4 == 0) {
#pragma unroll 4
        for (int c = lane * VEC; c < cols; c += WAVE * VEC) {
            float wv[GEMV_ROWS][VEC];
#pragma unroll
            for (int r = 0; r < GEMV_ROWS; ++r) {
                if constexpr (sizeof(T) == 2) {
                    typedef __attribute__((ext_vector_type(8))) __bf16 b8;
                    const b8 v = *reinterpret_cast<const b8*>(w[r] + c);
#pragma unroll
                    for (int e = 0; e < VEC; ++e) wv[r][e] = (float)v[e];
                } else {
                    const float4 v = *reinterpret_cast<const float4*>(w[r] + c);
                    wv[r][0] = v.x; wv[r][1] = v.y; wv[r][2] = v.z; wv[r][3] = v.w;
                }
            }
#pragma unroll
            for (int b = 0; b < MAXB; ++b) {
                if (b < batch) {
                    const float* ip = in + b * in_bs + c;
#pragma unroll
                    for (int e4 = 0; e4 < VEC; e4 += 4) {
                        const float4 x = *reinterpret_cast<const float4*>(ip + e4);
#pragma unroll
                        for (int r = 0; r < GEMV_ROWS; ++r)
                            acc[r][b] += (wv[r][e4] * x.x + wv[r][e4 + 1] * x.y) + (wv[r][e4 + 2] * x.z + wv[r][e4 + 3] * x.w);
                    }
                }
            }
        }
    } else {
        for (int c = lane; c < cols; c += WAVE) {
#pragma unroll
            for (int r = 0; r < GEMV_ROWS; ++r) {
                const float wv = to_f32(w[r][c]);
#pragma unroll
                for (int b = 0; b < MAXB; ++b)
                    if (b < batch) acc[r][b] += wv * in[b * in_bs + c];
            }
        }
    }
#pragma unroll
    for (int r = 0; r < GEMV_ROWS; ++r) {
        if (row0 + r >= rows) break;
#pragma unroll
        for (int b = 0; b < MAXB; ++b) {
            if (b < batch) {
                float v = sum_of_64(acc[r][b]);
                if (lane == 0) {
                    v += bias[row0 + r];
                    if (act == 1) v = silu_f(v);
                    out[b * out_bs + row0 + r] = v;
                }
            }
        }
    }
}

static constexpr long GEMV_FEW_ROWS = 4096;              // waves, half of what the chip holds

hipError_t launch_gemv_set(int dtype, const GemvSet& set, int count, const float* in, int rows, int cols, int batch,
                           long in_bs, long out_bs, int act, hipStream_t st) {
    if (count < 1 || count > GEMV_SET) return hipErrorInvalidValue;
    int threads = 256;
    auto go = [&](auto kernel, int rows_per_wave) {
        const int per_block = (threads / WAVE) * rows_per_wave;
        dim3 blocks((rows + per_block - 1) / per_block, count);
        kernel<<<blocks, threads, 0, st>>>(set, in, rows, cols, batch, in_bs, out_bs, act);
    };
    if (batch < 1 || batch > 16) return hipErrorInvalidValue;
    if ((long)rows * count <= GEMV_FEW_ROWS) {
        threads = 64;
        if (dtype == PS_BF16) {
            if (batch == 1) go(gemv_kernel<bf16_t, 1, 1>, 1);
            else if (batch <= 4) go(gemv_kernel<bf16_t, 4, 1>, 1);
            else go(gemv_kernel<bf16_t, 16, 1>, 1);
        } else {
            if (batch == 1) go(gemv_kernel<float, 1, 1>, 1);
            else if (batch <= 4) go(gemv_kernel<float, 4, 1>, 1);
            else go(gemv_kernel<float, 16, 1>, 1);
        }
        return hipGetLastError();
    }
    if (dtype == PS_BF16) {
        if (batch == 1) go(gemv_kernel<bf16_t, 1, 8>, 8);
        else if (batch <= 4) go(gemv_kernel<bf16_t, 4, 4>, 4);
        else go(gemv_kernel<bf16_t, 16, 4>, 4);
    } else {
        if (batch == 1) go(gemv_kernel<float, 1, 8>, 8);
        else if (batch <= 4) go(gemv_kernel<float, 4, 4>, 4);
        else go(gemv_kernel<float, 16, 4>, 4);
    }
    return hipGetLastError();
}

hipError_t launch_gemv(int dtype, const void* W, const float* bias, const float* in, float* out,
                       int rows, int cols, int batch, long in_bs, long out_bs, int act,
                       hipStream_t st) {
    GemvSet set{};
    set.W[0] = W; set.bias[0] = bias; set.out[0] = out;
    return launch_gemv_set(dtype, set, 1, in, rows, cols, batch, in_bs, out_bs, act, st);
}

// The modulation matrices as one matrix product in fp32, out[b][row] = W[row] . in[b] + bias[row], on
// v_mfma_f32_16x16x4_f32: 16 rows x up to 16 vectors per instruction, weights widened to fp32, so that one pass over the
// weights (708 MB for 30 layers of 1920) serves every timestep of a run's next steps.  Reading them is the bound, the matrix
// instructions (72 us of those 708 MB) come second.  A wave takes 16 rows at a time; lane l reads 16 adjacent weights of row
// l % 16, whole 128-byte lines (bf16) per row and 64 columns.  512 columns in bf16, 256 in fp32 are in flight per wave, the
// first of them requested before the vectors are staged, each step's registers refilled for what comes next behind its products.
// Four sums per output.  The same kernel serves one vector, so a vector's result does not depend on the batch.
// us, weights from memory, all loads of a pass and then its products / this: 30 layers bf16 162 / 147 (4.85 TB/s; rel_mae_kernel,
// which like this one only reads, reaches 6.8), nine vectors 176 / 160, one layer 12.9 / 12.0; fp32, two layers 31.3 / 25.0, one
// 19.4 / 14.9.
// (The kernel above has a sum over lanes per row and vector and reads the vectors again for every eight or four rows: 30 layers,
// one / four / nine vectors 143 / 259 / 569 us, this 145 / 157 / 161.)
static constexpr int MOD_MAX_COLS = 1000;                // 16 vectors of cols + 4 floats within 64 KB of LDS
template <typename T>
__global__ void __launch_bounds__(256, 4)
modulation_kernel(ModSet set, const float* __restrict__ in, int cols, int batch, long in_bs, int wg_rows) {
    typedef __attribute__((ext_vector_type(4))) float f4;
    extern __shared__ __attribute__((aligned(16))) float xs[];   // [batch][cols + 4]: 4 banks from vector to vector
    const int rows = set.rows[blockIdx.y], ld = cols + 4;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, kgrp = lane >> 4;
    if ((int)blockIdx.x * wg_rows >= rows) return;       // (whole workgroup)
    const int row_end = min(rows, (int)(blockIdx.x + 1) * wg_rows);
    const T* W = static_cast<const T*>(set.g.W[blockIdx.y]);
    constexpr int NQ = sizeof(T);                        // 16-byte loads per 16 weights: 2 (bf16) or 4
    constexpr int CH = 16 / NQ;                          // steps of 64 columns in flight
    uint4 raw[CH][NQ];
    auto row_of = [&](int row0) { return W + (long)min(row0 + l16, rows - 1) * cols + kgrp * 16; };
    auto request = [&](const T* w, int c0, int h) {      // (columns past the end: read again, not multiplied)
#pragma unroll
        for (int i = 0; i < NQ; ++i) raw[h][i] = *reinterpret_cast<const uint4*>(w + min(c0 + 64 * h, cols - 64) + i * (16 / NQ));
    };
    int row0 = blockIdx.x * wg_rows + wave * 16;
    {
        const T* w = row_of(row0);
#pragma unroll
        for (int h = 0; h < CH; ++h) request(w, 0, h);
    }
    for (int e = threadIdx.x * 4; e < batch * cols; e += 1024) {
        const int b = e / cols, c = e - b * cols;
        *reinterpret_cast<f4*>(xs + b * ld + c) = *reinterpret_cast<const f4*>(in + b * in_bs + c);
    }
    __syncthreads();
    const int xoff = (l16 < batch ? l16 : 0) * ld + kgrp * 16;   // columns past the batch repeat vector 0, unused
    f4 acc[4];
    // 64 * CH columns of the 16 rows at row0; NEXT: refill from `w`, column `nc0`, behind the products
    auto columns = [&](int c0, auto next_c, const T* w, int nc0) {
        constexpr bool NEXT = decltype(next_c)::value;
        int xo = xoff + c0;
        asm volatile("" : "+v"(xo));                     // (else the vectors are kept in registers over the passes, which spill)
#pragma unroll
        for (int h = 0; h < CH; ++h) {
            if (c0 + 64 * h < cols) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const f4 xv = *reinterpret_cast<const f4*>(xs + xo + 64 * h + i * 4);
                    f4 wv;
                    if constexpr (sizeof(T) == 2) {
                        const unsigned* u = reinterpret_cast<const unsigned*>(&raw[h][i / 2]) + (i & 1) * 2;
#pragma unroll
                        for (int e = 0; e < 2; ++e) {    // bf16 -> fp32: the upper half of the word
                            wv[2 * e] = __uint_as_float(u[e] << 16);
                            wv[2 * e + 1] = __uint_as_float(u[e] & 0xffff0000u);
                        }
                    } else {
                        wv = __builtin_bit_cast(f4, raw[h][i]);
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[e], xv[e], acc[e], 0, 0, 0);
                }
            }
            if constexpr (NEXT) request(w, nc0, h);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    for (; row0 < row_end; row0 += 64) {
#pragma unroll
        for (int a = 0; a < 4; ++a) acc[a] = f4{0.f, 0.f, 0.f, 0.f};
        const int out_row = row0 + kgrp * 4;             // rows % 4 == 0: inside or outside together
        const f4 bias = *reinterpret_cast<const f4*>(set.g.bias[blockIdx.y] + min(out_row, rows - 4));
        int c0 = 0;
        for (; c0 + 64 * CH < cols; c0 += 64 * CH) columns(c0, std::true_type{}, row_of(row0), c0 + 64 * CH);
        if (row0 + 64 < row_end) columns(c0, std::true_type{}, row_of(row0 + 64), 0);
        else columns(c0, std::false_type{}, nullptr, 0);
        if (l16 < batch && out_row < rows)
            *reinterpret_cast<f4*>(set.g.out[blockIdx.y] + l16 * set.out_bs[blockIdx.y] + out_row) =
                ((acc[0] + acc[1]) + (acc[2] + acc[3])) + bias;
    }
}

hipError_t launch_modulation(int dtype, const ModSet& set, int count, const float* in, int cols, int batch, long in_bs,
                             hipStream_t st) {
    if (count < 1 || count > GEMV_SET || batch < 1 || batch > 16) return hipErrorInvalidValue;
    int most = 0;
    bool ok = cols % 64 == 0 && cols <= MOD_MAX_COLS && in_bs % 4 == 0;   // (never a matter of the batch)
    for (int i = 0; i < count; ++i) {
        if (set.rows[i] > most) most = set.rows[i];
        ok = ok && set.rows[i] % 4 == 0 && set.out_bs[i] % 4 == 0;
    }
    if (!ok) {                                           // matrices of one shape (the layers') share a launch
        for (int i = 0, n; i < count; i += n) {
            GemvSet part{};
            for (n = 0; i + n < count && set.rows[i + n] == set.rows[i] && set.out_bs[i + n] == set.out_bs[i]; ++n) {
                part.W[n] = set.g.W[i + n]; part.bias[n] = set.g.bias[i + n]; part.out[n] = set.g.out[i + n];
            }
            const hipError_t e = launch_gemv_set(dtype, part, n, in, set.rows[i], cols, batch, in_bs, set.out_bs[i], 0, st);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    // Few matrices have to fill the chip: 64 rows per workgroup.  Many: 256, so that the vectors are staged less.  (The values
    // are the same.)  23040 x 512 bf16, 30 layers: 128 rows 146 us, nine vectors 165, 256 rows 147 and 160, 512 rows 155 and 166.
    const bool few = (long)most * count <= 200000;
    const int wg_rows = few ? 64 : 256;
    dim3 grid((most + wg_rows - 1) / wg_rows, count);
    const size_t sh = (size_t)batch * (cols + 4) * sizeof(float);
    if (dtype == PS_BF16) modulation_kernel<bf16_t><<<grid, 256, sh, st>>>(set, in, cols, batch, in_bs, wg_rows);
    else modulation_kernel<float><<<grid, 256, sh, st>>>(set, in, cols, batch, in_bs, wg_rows);
    return hipGetLastError();
}

// ------------------------------------------------------------------------- 3D RoPE table
// (cos, sin) of pos * theta^(-2m/d_A), axis widths d/4, 3d/8, 3d/8 over (frame, row, col), double precision
// angles.  The angle of a pair depends on the token only through its position on the pair's axis, so the table is
// stored per axis -- [F][d/8], [Hp][3d/16], [Wp][3d/16] entries of (cos, sin) -- about 1 KB instead of 256 bytes
// per token: the projection epilogue that rotates q and k finds it in the nearest cache.
__device__ __forceinline__ void rope_entry(float2* __restrict__ table, int F, int Hp, int Wp, int head_dim, float theta, int idx) {
    const int p0 = head_dim / 8, p1 = 3 * head_dim / 16;
    const int total = F * p0 + (Hp + Wp) * p1;
    if (idx >= total) return;
    int pos, m, dA;
    if (idx < F * p0) { pos = idx / p0; m = idx % p0; dA = 2 * p0; }
    else if (idx < F * p0 + Hp * p1) { int r = idx - F * p0; pos = r / p1; m = r % p1; dA = 2 * p1; }
    else { int r = idx - F * p0 - Hp * p1; pos = r / p1; m = r % p1; dA = 2 * p1; }
    double ang = (double)pos * exp(-2.0 * (double)m / (double)dA * log((double)theta));
    table[idx] = make_float2((float)cos(ang), (float)sin(ang));
}

size_t rope_table_floats(int F, int Hp, int Wp, int head_dim) {
    return 2 * ((size_t)F * (head_dim / 8) + (size_t)(Hp + Wp) * (3 * head_dim / 16));
}

// Both tables in one launch (each was a few microseconds of its own): rows 0 .. batch - 1 of the grid are the timesteps,
// the last row the rotary table.
__global__ void __launch_bounds__(128)
tables_kernel(TList tl, float* __restrict__ sinus, int D, int batch, float2* __restrict__ rope, int F, int Hp, int Wp,
              int head_dim, float theta) {
    const int stride = gridDim.x * 128;
    if ((int)blockIdx.y < batch) {
        for (int j = blockIdx.x * 128 + threadIdx.x; j < D / 2; j += stride) sinusoid_entry(tl, sinus, D, blockIdx.y, j);
    } else {
        const int total = F * (head_dim / 8) + (Hp + Wp) * (3 * head_dim / 16);
        for (int i = blockIdx.x * 128 + threadIdx.x; i < total; i += stride) rope_entry(rope, F, Hp, Wp, head_dim, theta, i);
    }
}

hipError_t launch_tables(const int32_t* t_host, float* sinus, int batch, int D, float* rope, int F, int Hp, int Wp,
                         int head_dim, float theta, hipStream_t st) {
    TList tl;
    for (int i = 0; i < 16; ++i) tl.t[i] = i < batch ? t_host[i] : 0;
    const size_t entries = rope ? rope_table_floats(F, Hp, Wp, head_dim) / 2 : 0;
    size_t most = (size_t)(D / 2) > entries ? (size_t)(D / 2) : entries;
    size_t blocks = (most + 127) / 128;
    if (blocks < 1) return hipSuccess;
    if (blocks > 65536) blocks = 65536;                  // (a longer table is walked)
    tables_kernel<<<dim3((unsigned)blocks, batch + (entries ? 1 : 0)), 128, 0, st>>>(
        tl, sinus, D, batch, reinterpret_cast<float2*>(rope), F, Hp, Wp, head_dim, theta);
    return hipGetLastError();
}

// ------------------------------------------------------------------------ patch embedding
// X[b, L_txt + (f,i,j), :] = W_pe . patch(c,dy,dx) + b_pe ; X[b, n < L_txt, :] = ctx[b, n, :].
// A matrix product in fp32 (v_mfma_f32_16x16x4_f32 on the fp32 latent and the widened weights): one workgroup per 64
// tokens x 64 columns, both operands staged in LDS 64 patch values at a time.  The weights are the first operand, so a
// lane ends with 4 adjacent columns of one token: X is written in 16-byte stores, and writing it is the bound for many
// tokens.  (One workgroup per 16 tokens whose threads each walked a whole weight row took 98 us at 112 tokens -- seven
// workgroups, uncoalesced -- and 116 us at 4516; this takes 13 and 33, 17776 tokens 159 -> 100.)
template <typename T>
__global__ void __launch_bounds__(256)
patch_embed_kernel(const float* __restrict__ x, const T* __restrict__ ctx, const T* __restrict__ W_pe,
                   const float* __restrict__ b_pe, float* __restrict__ X, int C, int F, int H, int Wd, int patch,
                   int text_tokens, int D, long ctx_bs) {
    typedef __attribute__((ext_vector_type(4))) float f4;
    constexpr int TILE = 64, KC = 64, LD = KC + 4;       // (rows 16-byte aligned, 4 banks apart)
    __shared__ __attribute__((aligned(16))) float pt[TILE * LD], wt[TILE * LD];
    const int Hp = H / patch, Wp = Wd / patch, N = text_tokens + F * Hp * Wp, P = C * patch * patch;
    const int tiles_d = (D + TILE - 1) / TILE;           // the column tiles of a token tile are neighbours
    const int n0 = blockIdx.x / tiles_d * TILE, d0 = blockIdx.x % tiles_d * TILE, b = blockIdx.y;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1, l16 = lane & 15, kgrp = lane >> 4;
    f4 acc[2][2];                                        // [16 columns][16 tokens]
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
        for (int t = 0; t < 2; ++t) acc[y][t] = f4{0.f, 0.f, 0.f, 0.f};
    if (n0 + TILE > text_tokens) {                       // (a tile of text rows only has nothing to multiply)
        const int n = n0 + lane, nv = n - text_tokens;   // lane = token while staging: neighbours read adjacent pixels
        const bool video = n < N && nv >= 0;
        const int j = nv % Wp, i = (nv / Wp) % Hp, f = nv / (Wp * Hp);
        const float* xp = x + (((long)b * C * F + f) * H + (long)i * patch) * Wd + (long)j * patch;
        for (int k0 = 0; k0 < P; k0 += KC) {
            float pv[KC / 4], wv[TILE / 4];              // all 32 loads of a thread in flight together
            // where patch value k0 + lane lies, one division per lane; read from that lane below (a division per value and
            // wave cost 38 against 33 us at 4516 tokens, 120 against 100 at 17776)
            const int lp = k0 + lane, lc = lp / (patch * patch), lr = lp - lc * patch * patch, ly = lr / patch;
            const int in_plane = ly * Wd + (lr - ly * patch);
#pragma unroll
            for (int u = 0; u < KC / 4; ++u) {           // patch value wave + 4u of every token (uniform per wave)
                const int c = __builtin_amdgcn_readlane(lc, wave + 4 * u);
                const int at = __builtin_amdgcn_readlane(in_plane, wave + 4 * u);
                pv[u] = video && k0 + wave + 4 * u < P ? xp[(long)c * F * H * Wd + at] : 0.f;
            }
#pragma unroll
            for (int u = 0; u < TILE / 4; ++u) {         // weight k0 + lane of row wave + 4u
                const int r = d0 + wave + 4 * u;
                wv[u] = k0 + lane < P && r < D ? to_f32(W_pe[(long)r * P + k0 + lane]) : 0.f;
            }
            if (k0) __syncthreads();
#pragma unroll
            for (int u = 0; u < KC / 4; ++u) pt[lane * LD + wave + 4 * u] = pv[u];
#pragma unroll
            for (int u = 0; u < TILE / 4; ++u) wt[(wave + 4 * u) * LD + lane] = wv[u];
            __syncthreads();
#pragma unroll
            for (int k = 0; k < KC; k += 16) {           // instruction e multiplies the k = 4 * kgrp + e of the 16
                f4 p[2], w[2];
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    p[t] = *reinterpret_cast<const f4*>(pt + (wm * 32 + t * 16 + l16) * LD + k + kgrp * 4);
                    w[t] = *reinterpret_cast<const f4*>(wt + (wn * 32 + t * 16 + l16) * LD + k + kgrp * 4);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int y = 0; y < 2; ++y)
#pragma unroll
                        for (int t = 0; t < 2; ++t)
                            acc[y][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[y][e], p[t][e], acc[y][t], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int n = n0 + wm * 32 + t * 16 + l16;
        if (n >= N) continue;
#pragma unroll
        for (int y = 0; y < 2; ++y) {
            const int col = d0 + wn * 32 + y * 16 + kgrp * 4;    // D % 4 == 0: inside or outside together
            if (col >= D) continue;
            f4 v;
            if (n < text_tokens) {
                const T* cp = ctx + b * ctx_bs + (long)n * D + col;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = to_f32(cp[e]);
            } else {
                v = acc[y][t] + *reinterpret_cast<const f4*>(b_pe + col);
            }
            *reinterpret_cast<f4*>(X + ((long)b * N + n) * D + col) = v;
        }
    }
}

// The same for bf16 weights and patch vectors of up to 64 values, on bf16 matrix instructions: a pixel is split into three
// bf16 numbers whose sum it is exactly (8 of its 24 significand bits each), so products and sums are those of fp32 at a
// fifth of the matrix time (six 16 x 16 x 32 instructions of 16 cycles for sixteen 16 x 16 x 4 of 32).  A wave keeps the
// patches of 64 tokens in registers and walks its columns, 32 at a time (whole lines of X), whose weights come straight from
// global memory in operand layout; writing X is the bound.
// (One workgroup per 64 x 64 outputs gathered the pixels once per 64 columns, in fp32 products: 13.4 us at 112 tokens x 1920,
// 31 at 4516, 100 at 17776; this took 7.4, 20 and 58.  Pixels requested without branches, the first weights and the biases with
// them and not when they have arrived: 8.8 -> 8.0, 20.0 -> 18.4, 58 -> 52.)
__global__ void __launch_bounds__(256)
patch_embed64_kernel(const float* __restrict__ x, const bf16_t* __restrict__ ctx, const bf16_t* __restrict__ W_pe,
                     const float* __restrict__ b_pe, float* __restrict__ X, int C, int F, int H, int Wd, int patch,
                     int text_tokens, int D, long ctx_bs, int cols) {
    typedef __attribute__((ext_vector_type(4))) float f4;
    typedef __attribute__((ext_vector_type(8))) __bf16 b8;
    constexpr int TILE = 64, LD = TILE + 4;              // (rows 16-byte aligned, 4 banks apart)
    __shared__ __attribute__((aligned(16))) float pt[TILE * LD];
    const int Hp = H / patch, Wp = Wd / patch, N = text_tokens + F * Hp * Wp, P = C * patch * patch;
    const int n0 = blockIdx.x * TILE, d0 = blockIdx.y * cols, d1 = min(d0 + cols, D), b = blockIdx.z;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, kgrp = lane >> 4;
    if (n0 < text_tokens) {                              // text rows of the tile: widened copies
        const int rows = min(TILE, text_tokens - n0), quads = (d1 - d0) / 4;
        for (int e = threadIdx.x; e < rows * quads; e += 256) {
            const int r = e / quads, col = d0 + (e - r * quads) * 4;
            const bf16_t* cp = ctx + b * ctx_bs + (long)(n0 + r) * D + col;
            *reinterpret_cast<f4*>(X + ((long)b * N + n0 + r) * D + col) = f4{to_f32(cp[0]), to_f32(cp[1]), to_f32(cp[2]), to_f32(cp[3])};
        }
        if (n0 + TILE <= text_tokens) return;            // (whole workgroup)
    }
    // lane l of step s: k = 16 * (l / 16) + 8s .. + 7, of a token in one operand and of a column in the other
    auto weights = [&](int col0, b8 (&w)[2][2], f4 (&bias)[2]) {
#pragma unroll
        for (int y = 0; y < 2; ++y) {
            bias[y] = *reinterpret_cast<const f4*>(b_pe + min(col0 + y * 16 + kgrp * 4, D - 4));
            const bf16_t* wp = W_pe + (long)min(col0 + y * 16 + l16, D - 1) * P + kgrp * 16;
            if (P == 64) {
#pragma unroll
                for (int s = 0; s < 2; ++s) w[y][s] = reinterpret_cast<const b8*>(wp)[s];
            } else {
#pragma unroll
                for (int e = 0; e < 16; ++e) w[y][e / 8][e % 8] = (__bf16)(kgrp * 16 + e < P ? to_f32(wp[e]) : 0.f);
            }
        }
    };
    b8 w[2][2], wn[2][2];
    f4 bias[2], bias_n[2];
    int c0 = d0 + wave * 32;
    {
        const int n = n0 + lane, nv = n - text_tokens;   // lane = token while staging: neighbours read adjacent pixels
        const bool video = n < N && nv >= 0;
        const int at_video = max(min(nv, N - 1 - text_tokens), 0);   // (of the other lanes: read, not used)
        const int j = at_video % Wp, i = (at_video / Wp) % Hp, f = at_video / (Wp * Hp);
        const float* xp = x + (((long)b * C * F + f) * H + (long)i * patch) * Wd + (long)j * patch;
        // where patch value `lane` lies, one division per lane; read from that lane below
        const int lv = min(lane, P - 1), lc = lv / (patch * patch), lr = lv - lc * patch * patch, ly = lr / patch;
        const int in_plane = ly * Wd + (lr - ly * patch);
        float pv[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {                   // patch value wave + 4u of every token (uniform per wave)
            const int c = __builtin_amdgcn_readlane(lc, wave + 4 * u);
            const int at = __builtin_amdgcn_readlane(in_plane, wave + 4 * u);
            pv[u] = xp[(long)c * F * H * Wd + at];
        }
        weights(min(c0, D - 1), w, bias);                // behind the pixels, not behind their arrival
#pragma unroll
        for (int u = 0; u < 16; ++u) pt[lane * LD + wave + 4 * u] = video && wave + 4 * u < P ? pv[u] : 0.f;
    }
    __syncthreads();
    b8 p[4][2][3];                                       // [16 tokens][step][part]
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float v = pt[(t * 16 + l16) * LD + kgrp * 16 + s * 8 + e];
                // (infinities and NaN: all in the first part)
                const auto top = [](float u) { return __uint_as_float(__float_as_uint(u) & 0xffff0000u); };
                const float hi = v == v ? top(v) : v, rest = fabsf(v) < __builtin_inff() ? v - hi : 0.f, mid = top(rest);
                p[t][s][0][e] = (__bf16)hi; p[t][s][1][e] = (__bf16)mid; p[t][s][2][e] = (__bf16)(rest - mid);
            }
    for (; c0 < d1; c0 += 128) {
        if (c0 + 128 < d1) weights(c0 + 128, wn, bias_n);
        f4 acc[4][2];
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int y = 0; y < 2; ++y) acc[t][y] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int part = 2; part >= 0; --part)            // small parts first
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int y = 0; y < 2; ++y)
                        acc[t][y] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[y][s], p[t][s][part], acc[t][y], 0, 0, 0);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int n = n0 + t * 16 + l16;
            if (n < text_tokens || n >= N) continue;
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                const int col = c0 + y * 16 + kgrp * 4;  // D % 4 == 0: inside or outside together
                if (col < d1) *reinterpret_cast<f4*>(X + ((long)b * N + n) * D + col) = acc[t][y] + bias[y];
            }
        }
#pragma unroll
        for (int y = 0; y < 2; ++y) {
            bias[y] = bias_n[y];
#pragma unroll
            for (int s = 0; s < 2; ++s) w[y][s] = wn[y][s];
        }
    }
}

hipError_t launch_patch_embed(int dtype, const float* x, const void* ctx, const void* W_pe,
                              const float* b_pe, float* X, int batch, int C, int F, int H, int Wd,
                              int patch, int text_tokens, int D, long ctx_bs, hipStream_t st) {
    const long N = text_tokens + (long)F * (H / patch) * (Wd / patch);
    if (dtype == PS_BF16 && C * patch * patch <= 64) {
        // Two workgroups of four waves per compute unit, and four or more per tile of tokens, so that their writes start and
        // end at different times; none with fewer than 128 columns.  4516 tokens in 4 / 8 / 15 pieces: 26 / 20 / 23 us,
        // 17776 tokens in 1 / 2 / 4 / 8 / 15: 98 / 68 / 58 / 59 / 72.
        const long tiles = (N + 63) / 64 * batch, most = (D + 127) / 128;
        long split = (2L * compute_units() + tiles - 1) / tiles;
        if (split < 4) split = 4;
        if (split > most) split = most;
        const int cols = (int)((most + split - 1) / split) * 128;
        const dim3 g((unsigned)((N + 63) / 64), (D + cols - 1) / cols, batch);
        patch_embed64_kernel<<<g, 256, 0, st>>>(x, (const bf16_t*)ctx, (const bf16_t*)W_pe, b_pe, X, C, F, H, Wd, patch, text_tokens,
                                                D, ctx_bs, cols);
        return hipGetLastError();
    }
    dim3 grid((unsigned)((N + 63) / 64 * ((D + 63) / 64)), batch);   // at most 2^18 x 2^5
    if (dtype == PS_BF16)
        patch_embed_kernel<bf16_t><<<grid, 256, 0, st>>>(x, (const bf16_t*)ctx, (const bf16_t*)W_pe,
                                                         b_pe, X, C, F, H, Wd, patch, text_tokens, D, ctx_bs);
    else
        patch_embed_kernel<float><<<grid, 256, 0, st>>>(x, (const float*)ctx, (const float*)W_pe, b_pe,
                                                        X, C, F, H, Wd, patch, text_tokens, D, ctx_bs);
    return hipGetLastError();
}

// ------------------------------------------------------------------- LayerNorm + modulate
// One wave per token row.  fp32 statistics (mean, then centred second moment), biased
// variance, no affine; out = y*(1+scale)+shift with the text or video chunk.
// The row is held in registers between the passes: D <= 64*4*MAXV.
// (Two rows per wave, both loaded before the first reduction, measured 18 % slower at 17776 x 1920: 48 against 41 us.)
template <typename T, int MAXV>
__global__ void ln_modulate_kernel(const float* __restrict__ X, T* __restrict__ out, int M, int D,
                                   float eps, const float* __restrict__ mod_layer, long mod_bs,
                                   int shift_chunk, int scale_chunk, TokenGeom g, float* __restrict__ zero_buf,
                                   int zero_n) {
    // a few words some later kernel sets (the attention kernels' per-head flags) are cleared here
    // instead of by a launch of their own
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < zero_n; i += blockDim.x) zero_buf[i] = 0.f;
    int row = (blockIdx.x * blockDim.x + threadIdx.x) / WAVE;
    int lane = threadIdx.x % WAVE;
    if (row >= M) return;
    const float4* xr = reinterpret_cast<const float4*>(X + (long)row * D);
    int nvec = D / 4;
    float4 v[MAXV];
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < MAXV; ++i) {
        int c = lane + i * WAVE;
        if (c < nvec) {
            v[i] = xr[c];
            s += (v[i].x + v[i].y) + (v[i].z + v[i].w);
        }
    }
    float mean = sum_of_64(s) / (float)D;
    float q = 0.f;
#pragma unroll
    for (int i = 0; i < MAXV; ++i) {
        int c = lane + i * WAVE;
        if (c < nvec) {
            float a = v[i].x - mean, b = v[i].y - mean, cc = v[i].z - mean, d = v[i].w - mean;
            q += (a * a + b * b) + (cc * cc + d * d);
        }
    }
    float rstd = 1.0f / sqrtf(sum_of_64(q) / (float)D + eps);
    int b = row / g.tokens, n = row % g.tokens;
    int off = n < g.text_tokens ? 6 : 0;
    const float4* sh = reinterpret_cast<const float4*>(mod_layer + b * mod_bs + (long)(shift_chunk + off) * D);
    const float4* sc = reinterpret_cast<const float4*>(mod_layer + b * mod_bs + (long)(scale_chunk + off) * D);
    T* orow = out + (long)row * D;
#pragma unroll
    for (int i = 0; i < MAXV; ++i) {
        int c = lane + i * WAVE;
        if (c < nvec) {
            float4 h = sh[c], k = sc[c];
            float y0 = (v[i].x - mean) * rstd * (1.f + k.x) + h.x;
            float y1 = (v[i].y - mean) * rstd * (1.f + k.y) + h.y;
            float y2 = (v[i].z - mean) * rstd * (1.f + k.z) + h.z;
            float y3 = (v[i].w - mean) * rstd * (1.f + k.w) + h.w;
            if constexpr (sizeof(T) == 2) {
                union { bf16_t h4[4]; uint2 u; } pk;
                pk.h4[0] = __float2bfloat16(y0); pk.h4[1] = __float2bfloat16(y1);
                pk.h4[2] = __float2bfloat16(y2); pk.h4[3] = __float2bfloat16(y3);
                *reinterpret_cast<uint2*>(orow + 4 * c) = pk.u;
            } else {
                *reinterpret_cast<float4*>(orow + 4 * c) = make_float4(y0, y1, y2, y3);
            }
        }
    }
}

// Sum over the 256 threads of a workgroup, the same value in every thread.  `sm`: 4 floats, one set per call.
__device__ __forceinline__ float block_sum(float v, float* sm) {
    v = sum_of_64(v);
    if (threadIdx.x % WAVE == 0) sm[threadIdx.x / WAVE] = v;
    __syncthreads();
    return (sm[0] + sm[1]) + (sm[2] + sm[3]);
}

// The same for samples of few tokens: one workgroup per row, so that 112 rows occupy 112 compute units and a thread
// has two 16-byte loads per operand instead of eight.  It also finishes a projection whose K pieces are still apart
// (PendingResidual): the pieces are added in order, X is updated in place and its new row is normalised from registers,
// which saves the launch and the pass over X that a reduction of its own would take.
// CAP: pieces at most (0: none are apart).  All that a row reads is requested at once, without branches: one operand after the
// other, and the pieces four at a time, were up to six trips to memory in a row.  Rows x pieces of 1920, us: bf16 48 x 6 5.8 ->
// 4.4, 48 x 8 4.9 -> 4.2, 112 x 4 4.7 -> 4.4, 112 x 8 5.3 -> 4.2, 448 x 4 7.5 -> 7.1, 448 x 8 8.2 -> 8.0, 560 x 8 9.8 -> 9.6,
// 900 x 3 8.8 -> 8.6, 1100 x 3 10.6 both, 1250 x 3 10.25 -> 10.3 (the piece read for a fourth comes from the same lines); fp32
// 112 x 8 6.0 -> 5.4, 161 x 5 6.2 -> 5.9.
template <typename T, int CAP>
__global__ void __launch_bounds__(256)
ln_modulate_row_kernel(float* __restrict__ X, T* __restrict__ out, int M, int D, float eps,
                       const float* __restrict__ mod_layer, long mod_bs, int shift_chunk, int scale_chunk, TokenGeom g,
                       float* __restrict__ zero_buf, int zero_n, PendingResidual pd, int pd_text, long pd_bs) {
    constexpr int MAXV = 2, ROOM = CAP > 0 ? CAP : 1;
    __shared__ float sm[2][4];
    const int row = blockIdx.x, b = row / g.tokens, n = row - b * g.tokens, nvec = D / 4;
    if (row == 0)
        for (int i = threadIdx.x; i < zero_n; i += 256) zero_buf[i] = 0.f;
    const int off = n < g.text_tokens ? 6 : 0;
    const float4* sh = reinterpret_cast<const float4*>(mod_layer + b * mod_bs + (long)(shift_chunk + off) * D);
    const float4* sc = reinterpret_cast<const float4*>(mod_layer + b * mod_bs + (long)(scale_chunk + off) * D);
    float4* xr = reinterpret_cast<float4*>(X + (long)row * D);
    float4 v[MAXV], h[MAXV], k[MAXV], bi[MAXV], ga[MAXV], part[MAXV][ROOM];
    int at[MAXV];                                        // (threads past the row's end repeat its last quad, unused)
#pragma unroll
    for (int i = 0; i < MAXV; ++i) at[i] = min((int)threadIdx.x + i * 256, nvec - 1);
    if constexpr (CAP > 0) {
        const float4* gate = reinterpret_cast<const float4*>(pd.mod_layer + b * pd_bs +
                                                             (long)(pd.gate_chunk + (n < pd_text ? 6 : 0)) * D);
#pragma unroll
        for (int p = 0; p < CAP; ++p)
#pragma unroll
            for (int i = 0; i < MAXV; ++i)               // (past the last piece: that one again, not added)
                part[i][p] = reinterpret_cast<const float4*>(pd.part + ((long)min(p, pd.pieces - 1) * M + row) * D)[at[i]];
#pragma unroll
        for (int i = 0; i < MAXV; ++i) { bi[i] = reinterpret_cast<const float4*>(pd.bias)[at[i]]; ga[i] = gate[at[i]]; }
    }
#pragma unroll
    for (int i = 0; i < MAXV; ++i) { v[i] = xr[at[i]]; h[i] = sh[at[i]]; k[i] = sc[at[i]]; }
    const auto arrived = [](float4& u) { asm volatile("" : "+v"(u.x), "+v"(u.y), "+v"(u.z), "+v"(u.w) : : "memory"); };
#pragma unroll
    for (int i = 0; i < MAXV; ++i) {                     // (nothing is used before all of it is requested)
#pragma unroll
        for (int p = 0; p < CAP; ++p) arrived(part[i][p]);
        if constexpr (CAP > 0) { arrived(bi[i]); arrived(ga[i]); }
        arrived(v[i]);
        arrived(h[i]);
        arrived(k[i]);
    }
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < MAXV; ++i) {
        const bool live = (int)threadIdx.x + i * 256 < nvec;
        if constexpr (CAP > 0) {
            float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int p = 0; p < CAP; ++p) {
                const float4 u = part[i][p];             // (selects, not a branch, behind which its loads would move)
                const bool in = p < pd.pieces;
                t.x += in ? u.x : 0.f; t.y += in ? u.y : 0.f; t.z += in ? u.z : 0.f; t.w += in ? u.w : 0.f;
            }
            v[i].x += ga[i].x * (t.x + bi[i].x); v[i].y += ga[i].y * (t.y + bi[i].y);
            v[i].z += ga[i].z * (t.z + bi[i].z); v[i].w += ga[i].w * (t.w + bi[i].w);
            if (live) xr[at[i]] = v[i];
        }
        if (live) s += (v[i].x + v[i].y) + (v[i].z + v[i].w);
    }
    const float mean = block_sum(s, sm[0]) / (float)D;
    float q = 0.f;
#pragma unroll
    for (int i = 0; i < MAXV; ++i) {
        if ((int)threadIdx.x + i * 256 >= nvec) continue;
        const float a = v[i].x - mean, bb = v[i].y - mean, cc = v[i].z - mean, d = v[i].w - mean;
        q += (a * a + bb * bb) + (cc * cc + d * d);
    }
    const float rstd = 1.0f / sqrtf(block_sum(q, sm[1]) / (float)D + eps);
    T* orow = out + (long)row * D;
#pragma unroll
    for (int i = 0; i < MAXV; ++i) {
        const int c = threadIdx.x + i * 256;
        if (c >= nvec) continue;
        const float y0 = (v[i].x - mean) * rstd * (1.f + k[i].x) + h[i].x;
        const float y1 = (v[i].y - mean) * rstd * (1.f + k[i].y) + h[i].y;
        const float y2 = (v[i].z - mean) * rstd * (1.f + k[i].z) + h[i].z;
        const float y3 = (v[i].w - mean) * rstd * (1.f + k[i].w) + h[i].w;
        if constexpr (sizeof(T) == 2) {
            union { bf16_t h4[4]; uint2 u; } pk;
            pk.h4[0] = __float2bfloat16(y0); pk.h4[1] = __float2bfloat16(y1);
            pk.h4[2] = __float2bfloat16(y2); pk.h4[3] = __float2bfloat16(y3);
            *reinterpret_cast<uint2*>(orow + 4 * c) = pk.u;
        } else {
            *reinterpret_cast<float4*>(orow + 4 * c) = make_float4(y0, y1, y2, y3);
        }
    }
}

// up to this many tokens per sample a row gets a workgroup: 112 rows 8.4 -> 5.5 us, 2060 rows 9.6 -> 7.3, 4400 rows 13.9 ->
// 11.4, 6200 rows 19.7 -> 14.1; 17776 rows take the wave kernel 40 us, 5.1 TB/s (the choice changes the order of a row's sums, so it must
// not depend on the batch)
static constexpr int LN_ROW_TOKENS = 6144;

hipError_t launch_ln_modulate(int dtype, float* X, void* out, int M, int D, float eps,
                              const float* mod_layer, long mod_bs, int shift_chunk, int scale_chunk,
                              TokenGeom geom, hipStream_t st, float* zero_buf, int zero_n,
                              const PendingResidual* pending, int text_tokens, long pending_bs) {
    if (D % 4 != 0 || D > 64 * 4 * 8) return hipErrorInvalidValue;
    const bool pend = pending && pending->pieces > 0;
    if (pend || geom.tokens <= LN_ROW_TOKENS) {
        const PendingResidual pd = pend ? *pending : PendingResidual{};
        if (pd.pieces > 16) return hipErrorInvalidValue;
        auto go = [&](auto kernel, auto* to) {
            kernel<<<M, 256, 0, st>>>(X, to, M, D, eps, mod_layer, mod_bs, shift_chunk, scale_chunk, geom, zero_buf, zero_n, pd,
                                      text_tokens, pending_bs);
            return hipGetLastError();
        };
        auto as = [&](auto* to) {
            using T = std::remove_pointer_t<decltype(to)>;
            if (pd.pieces == 0) return go(ln_modulate_row_kernel<T, 0>, to);
            if (pd.pieces <= 4) return go(ln_modulate_row_kernel<T, 4>, to);
            if (pd.pieces <= 8) return go(ln_modulate_row_kernel<T, 8>, to);
            return go(ln_modulate_row_kernel<T, 16>, to);
        };
        return dtype == PS_BF16 ? as((bf16_t*)out) : as((float*)out);
    }
    int threads = 256;
    int blocks = (M + 3) / 4;
    if (dtype == PS_BF16)
        ln_modulate_kernel<bf16_t, 8><<<blocks, threads, 0, st>>>(X, (bf16_t*)out, M, D, eps, mod_layer, mod_bs,
                                                                 shift_chunk, scale_chunk, geom, zero_buf, zero_n);
    else
        ln_modulate_kernel<float, 8><<<blocks, threads, 0, st>>>(X, (float*)out, M, D, eps, mod_layer, mod_bs,
                                                                shift_chunk, scale_chunk, geom, zero_buf, zero_n);
    return hipGetLastError();
}

// ------------------------------------------------------------------------ final projection
// Video tokens only: y = LN(X_n)(1+scale)+shift with modf = [shift | scale] (fp32 [B][2D]),
// out = W_out y + b_out (C*ps*ps values in (c,dy,dx) order) scattered into eps[C,F,H,W].
// One workgroup (256 threads) per token; y kept in LDS.
template <typename T>
__global__ void final_proj_kernel(const float* __restrict__ X, const float* __restrict__ modf,
                                  const T* __restrict__ W_out, const float* __restrict__ b_out,
                                  float* __restrict__ eps_out, int C, int F, int H, int Wd, int patch,
                                  int text_tokens, int D, float eps) {
    extern __shared__ float y[];     // [D] + 8 partials
    float* red = y + D;
    int Hp = H / patch, Wp = Wd / patch;
    int Nv = F * Hp * Wp, N = text_tokens + Nv;
    int b = blockIdx.y, nv = blockIdx.x;
    const float* xr = X + ((long)b * N + text_tokens + nv) * D;
    int lane = threadIdx.x % WAVE, wave = threadIdx.x / WAVE, nw = blockDim.x / WAVE;
    float s = 0.f;
    for (int c = threadIdx.x; c < D; c += blockDim.x) { float v = xr[c]; y[c] = v; s += v; }
    s = sum_of_64(s);
    if (lane == 0) red[wave] = s;
    __syncthreads();
    float tot = 0.f;
    for (int w = 0; w < nw; ++w) tot += red[w];
    float mean = tot / (float)D;
    __syncthreads();
    float q = 0.f;
    for (int c = threadIdx.x; c < D; c += blockDim.x) { float dlt = y[c] - mean; q += dlt * dlt; }
    q = sum_of_64(q);
    if (lane == 0) red[wave] = q;
    __syncthreads();
    float qt = 0.f;
    for (int w = 0; w < nw; ++w) qt += red[w];
    float rstd = 1.0f / sqrtf(qt / (float)D + eps);
    const float* shift = modf + (long)b * 2 * D;
    const float* scale = shift + D;
    for (int c = threadIdx.x; c < D; c += blockDim.x)
        y[c] = (y[c] - mean) * rstd * (1.f + scale[c]) + shift[c];
    __syncthreads();
    int P = C * patch * patch;
    int j = nv % Wp, i = (nv / Wp) % Hp, f = nv / (Wp * Hp);
    for (int o = wave; o < P; o += nw) {
        const T* w = W_out + (long)o * D;
        float acc = 0.f;
        for (int c = lane; c < D; c += WAVE) acc += to_f32(w[c]) * y[c];
        acc = sum_of_64(acc);
        if (lane == 0) {
            int dx = o % patch, dy = (o / patch) % patch, c = o / (patch * patch);
            eps_out[((((long)b * C + c) * F + f) * H + (i * patch + dy)) * Wd + (j * patch + dx)] = acc + b_out[o];
        }
    }
}

hipError_t launch_final_proj(int dtype, const float* X, const float* modf, const void* W_out,
                             const float* b_out, float* eps_out, int batch, int C, int F, int H,
                             int Wd, int patch, int text_tokens, int D, float eps, hipStream_t st) {
    int Nv = F * (H / patch) * (Wd / patch);
    dim3 grid(Nv, batch);
    size_t sh = (size_t)(D + 8) * sizeof(float);
    if (dtype == PS_BF16)
        final_proj_kernel<bf16_t><<<grid, 256, sh, st>>>(X, modf, (const bf16_t*)W_out, b_out, eps_out, C, F, H,
                                                        Wd, patch, text_tokens, D, eps);
    else
        final_proj_kernel<float><<<grid, 256, sh, st>>>(X, modf, (const float*)W_out, b_out, eps_out, C, F, H, Wd,
                                                       patch, text_tokens, D, eps);
    return hipGetLastError();
}

// ------------------------------------------------- scheduler update + relative-MAE sums
// Two-stage deterministic reduction.  Stage 1 streams the tensors once with non-temporal
// 16-byte accesses.  A workgroup takes contiguous chunks of 256 x 4 float4 (16 KB of every
// tensor), each thread four float4 per tensor 4 KB apart, all loads of a chunk in flight
// before the first use; the grid has one workgroup per chunk up to 32768 (measured on MI355X
// at 2^28 elements: 6.1 TB/s for the update with sums, against 5.3 for a grid-stride walk with
// two float4 in flight and 4.3-5.0 for grids of 2048-8192 long-running workgroups); each
// workgroup leaves its partial sums in the workspace.  Stage 2 (one workgroup of 1024) adds
// the partials in a fixed order in double.
static constexpr int RED_THREADS = 256;
static constexpr int RED_MAX_BLOCKS = 32768;
static constexpr int RED_UNROLL = 4;
static constexpr size_t RED_CHUNK = (size_t)RED_THREADS * RED_UNROLL;      // float4 per workgroup step

typedef __attribute__((ext_vector_type(4))) float v4f_t;
__device__ __forceinline__ float4 stream_load(const float4* p) {
    v4f_t v = __builtin_nontemporal_load(reinterpret_cast<const v4f_t*>(p));
    return make_float4(v[0], v[1], v[2], v[3]);
}
__device__ __forceinline__ void stream_store(float4 r, float4* p) {
    v4f_t v = {r.x, r.y, r.z, r.w};
    __builtin_nontemporal_store(v, reinterpret_cast<v4f_t*>(p));
}
__device__ __forceinline__ float abs4(float4 v) { return (fabsf(v.x) + fabsf(v.y)) + (fabsf(v.z) + fabsf(v.w)); }
__device__ __forceinline__ float absdiff4(float4 a, float4 b) {
    return (fabsf(a.x - b.x) + fabsf(a.y - b.y)) + (fabsf(a.z - b.z) + fabsf(a.w - b.w));
}

static int red_blocks(size_t n) {
    size_t per_block = RED_CHUNK * 4;
    size_t b = (n + per_block - 1) / per_block;
    if (b < 1) b = 1;
    if (b > RED_MAX_BLOCKS) b = RED_MAX_BLOCKS;
    return (int)b;
}

size_t reduce_workspace_bytes(size_t n) { (void)n; return (size_t)RED_MAX_BLOCKS * 4 * sizeof(double); }

template <int NS>
__device__ __forceinline__ void block_store_partials(double (&acc)[NS], double* __restrict__ part, float* __restrict__ fin) {
    __shared__ double sm[NS][RED_THREADS / WAVE];
    int lane = threadIdx.x % WAVE, wave = threadIdx.x / WAVE;
#pragma unroll
    for (int k = 0; k < NS; ++k) {
        double v = sum_of_64(acc[k]);
        if (lane == 0) sm[k][wave] = v;
    }
    __syncthreads();
    // The only workgroup has the whole sums: it writes the result and stage 2 is not launched (up to 4096 elements, where
    // its 3.6 us were as long as the update itself).
    if (fin != nullptr) {
        if (threadIdx.x == 0) {
            double t[NS];
#pragma unroll
            for (int k = 0; k < NS; ++k) {
                t[k] = 0.0;
                for (int w = 0; w < RED_THREADS / WAVE; ++w) t[k] += sm[k][w];
                fin[k] = (float)t[k];
            }
            if constexpr (NS == 2) fin[2] = (float)(t[0] / t[1]);    // relative MAE; IEEE: inf or nan when the denominator is 0
        }
        return;
    }
    if (threadIdx.x < NS) {
        double t = 0.0;
        for (int w = 0; w < RED_THREADS / WAVE; ++w) t += sm[threadIdx.x][w];
        part[(long)blockIdx.x * NS + threadIdx.x] = t;
    }
}

// stage 2: NS sums over nblocks partials with one workgroup of FIN_THREADS; thread k adds
// partials k, k+FIN_THREADS, ... (four rows in flight, added in index order) and the per-thread
// results are combined in a fixed tree, so the result does not depend on timing
static constexpr int FIN_THREADS = 1024;
template <int NS>
__device__ __forceinline__ void reduce_partials(const double* __restrict__ part, int nblocks, double (&out)[NS]) {
    __shared__ double sm2[NS][FIN_THREADS / WAVE];
    double acc[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k) acc[k] = 0.0;
    int b = threadIdx.x;
    for (; b + 3 * FIN_THREADS < nblocks; b += 4 * FIN_THREADS) {
        double v[4][NS];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int k = 0; k < NS; ++k) v[u][k] = part[(long)(b + u * FIN_THREADS) * NS + k];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int k = 0; k < NS; ++k) acc[k] += v[u][k];
    }
    for (; b < nblocks; b += FIN_THREADS)
#pragma unroll
        for (int k = 0; k < NS; ++k) acc[k] += part[(long)b * NS + k];
    int lane = threadIdx.x % WAVE, wave = threadIdx.x / WAVE;
#pragma unroll
    for (int k = 0; k < NS; ++k) {
        double v = sum_of_64(acc[k]);
        if (lane == 0) sm2[k][wave] = v;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NS; ++k) {
        double t = 0.0;
        for (int w = 0; w < FIN_THREADS / WAVE; ++w) t += sm2[k][w];
        out[k] = t;
    }
}

// increment form: d = (a-1)x + b*eps, x' = x + d (a -> 1 near the end of a run, and the sum
// of |x' - x| must not come from a difference of rounded values)
template <bool SUMS, bool PREV>
__global__ void __launch_bounds__(RED_THREADS)
sampler_step_kernel(const float* x, const float* __restrict__ e, const float* __restrict__ ep, float* xo,
                    float am1, float b, size_t n, double* __restrict__ part, float* __restrict__ fin) {
    float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
    const size_t nvec = n / 4;
    const float4* x4 = reinterpret_cast<const float4*>(x);
    const float4* e4 = reinterpret_cast<const float4*>(e);
    const float4* p4 = reinterpret_cast<const float4*>(ep);
    float4* o4 = reinterpret_cast<float4*>(xo);
    auto one = [&](float4 xv, float4 ev, float4 pv, size_t i) {
        float4 dl, r;
        dl.x = am1 * xv.x + b * ev.x; dl.y = am1 * xv.y + b * ev.y;
        dl.z = am1 * xv.z + b * ev.z; dl.w = am1 * xv.w + b * ev.w;
        r.x = xv.x + dl.x; r.y = xv.y + dl.y; r.z = xv.z + dl.z; r.w = xv.w + dl.w;
        stream_store(r, o4 + i);
        if constexpr (SUMS) {
            s0 += abs4(dl); s1 += abs4(r); s3 += abs4(ev);
            if constexpr (PREV) s2 += absdiff4(ev, pv);
        }
    };
    for (size_t base = (size_t)blockIdx.x * RED_CHUNK; base < nvec; base += (size_t)gridDim.x * RED_CHUNK) {
        const size_t i = base + threadIdx.x;
        if (base + RED_CHUNK <= nvec) {
            float4 xv[RED_UNROLL], ev[RED_UNROLL], pv[RED_UNROLL];
#pragma unroll
            for (int u = 0; u < RED_UNROLL; ++u) {
                xv[u] = stream_load(x4 + i + u * RED_THREADS);
                ev[u] = stream_load(e4 + i + u * RED_THREADS);
                pv[u] = xv[u];
                if constexpr (SUMS && PREV) pv[u] = stream_load(p4 + i + u * RED_THREADS);
            }
#pragma unroll
            for (int u = 0; u < RED_UNROLL; ++u) one(xv[u], ev[u], pv[u], i + u * RED_THREADS);
        } else {
            for (int u = 0; u < RED_UNROLL; ++u) {
                const size_t j = i + u * RED_THREADS;
                if (j < nvec) {
                    float4 xa = stream_load(x4 + j), ea = stream_load(e4 + j), pa = xa;
                    if constexpr (SUMS && PREV) pa = stream_load(p4 + j);
                    one(xa, ea, pa, j);
                }
            }
        }
    }
    // ragged tail (n % 4 elements) handled by the first threads of block 0
    if (blockIdx.x == 0 && threadIdx.x < (n & 3)) {
        size_t t = nvec * 4 + threadIdx.x;
        float xv = x[t], ev = e[t];
        float dl = am1 * xv + b * ev;
        float r = xv + dl;
        xo[t] = r;
        if constexpr (SUMS) {
            s0 += fabsf(dl); s1 += fabsf(r); s3 += fabsf(ev);
            if constexpr (PREV) s2 += fabsf(ev - ep[t]);
        }
    }
    if constexpr (SUMS) {
        // a thread adds at most n / (4 * grid * 256) + 1 float4 per sum in fp32 (a few dozen
        // terms at any size the grid cap allows below 2^32 elements), then everything is double
        double acc[4] = {(double)s0, (double)s1, (double)s2, (double)s3};
        block_store_partials<4>(acc, part, fin);
    }
}

__global__ void __launch_bounds__(FIN_THREADS)
finish_sums4_kernel(const double* __restrict__ part, int nblocks, float* __restrict__ out) {
    double t[4];
    reduce_partials<4>(part, nblocks, t);
    if (threadIdx.x < 4) out[threadIdx.x] = (float)t[threadIdx.x];
}

hipError_t launch_sampler_step(const float* x, const float* e, const float* e_prev, float* x_out,
                               double a, double b, size_t n, float* sums4, void* ws, hipStream_t st) {
    if (n == 0) {
        if (sums4) finish_sums4_kernel<<<1, FIN_THREADS, 0, st>>>((const double*)ws, 0, sums4);   // four zeros
        return hipGetLastError();
    }
    int blocks = red_blocks(n);
    double* part = (double*)ws;
    const float am1 = (float)(a - 1.0), bf = (float)b;
    float* fin = blocks == 1 ? sums4 : nullptr;
    if (!sums4)
        sampler_step_kernel<false, false><<<blocks, RED_THREADS, 0, st>>>(x, e, nullptr, x_out, am1, bf, n, nullptr, nullptr);
    else if (e_prev)
        sampler_step_kernel<true, true><<<blocks, RED_THREADS, 0, st>>>(x, e, e_prev, x_out, am1, bf, n, part, fin);
    else
        sampler_step_kernel<true, false><<<blocks, RED_THREADS, 0, st>>>(x, e, nullptr, x_out, am1, bf, n, part, fin);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    if (sums4 && !fin) finish_sums4_kernel<<<1, FIN_THREADS, 0, st>>>(part, blocks, sums4);
    return hipGetLastError();
}

// Partial sums of sampler_step for callers that may not allocate: a file-scope device array (1 MiB, held by
// every GPU the library runs on until the process ends) instead of a caller-supplied workspace.  In host code the
// array's name is only a stand-in; its device address is looked up once per device, with that device current, and
// kept.  Nothing in it has to start at zero: stage 1 writes the partial sums of every workgroup it launches and
// stage 2 reads exactly those.  Calls that overlap on one GPU share the array and race.
static __device__ __align__(256) double scratch[(size_t)RED_MAX_BLOCKS * 4];
static constexpr int SCRATCH_MAX_DEVICES = 64;
static double* scratch_ptr[SCRATCH_MAX_DEVICES];     // device address of `scratch` on each device (nullptr: not yet asked)
static std::mutex scratch_mutex;

hipError_t launch_sampler_step_static(const float* x, const float* e, const float* e_prev, float* x_out,
                                      double a, double b, size_t n, float* sums4, hipStream_t st) {
    double* ptr = nullptr;
    if (sums4) {
        int dev = -1;
        hipError_t err = hipGetDevice(&dev);
        if (err != hipSuccess) return err;
        if (dev < 0 || dev >= SCRATCH_MAX_DEVICES) return hipErrorInvalidDevice;
        std::lock_guard<std::mutex> lock(scratch_mutex);
        if (scratch_ptr[dev] == nullptr) {
            void* p = nullptr;
            err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
            if (err != hipSuccess) return err;
            if (p == nullptr) return hipErrorInvalidSymbol;
            scratch_ptr[dev] = static_cast<double*>(p);
        }
        ptr = scratch_ptr[dev];
    }
    return launch_sampler_step(x, e, e_prev, x_out, a, b, n, sums4, ptr, st);
}

__global__ void __launch_bounds__(RED_THREADS)
rel_mae_kernel(const float* __restrict__ a, const float* __restrict__ b, size_t n, double* __restrict__ part,
               float* __restrict__ fin) {
    float s0 = 0.f, s1 = 0.f;
    const size_t nvec = n / 4;
    const float4* a4 = reinterpret_cast<const float4*>(a);
    const float4* b4 = reinterpret_cast<const float4*>(b);
    for (size_t base = (size_t)blockIdx.x * RED_CHUNK; base < nvec; base += (size_t)gridDim.x * RED_CHUNK) {
        const size_t i = base + threadIdx.x;
        if (base + RED_CHUNK <= nvec) {
            float4 av[RED_UNROLL], bv[RED_UNROLL];
#pragma unroll
            for (int u = 0; u < RED_UNROLL; ++u) {
                av[u] = stream_load(a4 + i + u * RED_THREADS);
                bv[u] = stream_load(b4 + i + u * RED_THREADS);
            }
#pragma unroll
            for (int u = 0; u < RED_UNROLL; ++u) { s0 += absdiff4(av[u], bv[u]); s1 += abs4(av[u]); }
        } else {
            for (int u = 0; u < RED_UNROLL; ++u) {
                const size_t j = i + u * RED_THREADS;
                if (j < nvec) {
                    float4 a0 = stream_load(a4 + j), b0 = stream_load(b4 + j);
                    s0 += absdiff4(a0, b0);
                    s1 += abs4(a0);
                }
            }
        }
    }
    if (blockIdx.x == 0 && threadIdx.x < (n & 3)) {
        size_t t = nvec * 4 + threadIdx.x;
        s0 += fabsf(a[t] - b[t]); s1 += fabsf(a[t]);
    }
    double acc[2] = {(double)s0, (double)s1};
    block_store_partials<2>(acc, part, fin);
}

__global__ void __launch_bounds__(FIN_THREADS)
finish_rel_mae_kernel(const double* __restrict__ part, int nblocks, float* __restrict__ out3) {
    double t[2];
    reduce_partials<2>(part, nblocks, t);
    if (threadIdx.x == 0) {
        out3[0] = (float)t[0];
        out3[1] = (float)t[1];
        out3[2] = (float)(t[0] / t[1]);     // IEEE: inf or nan when the denominator is 0
    }
}

hipError_t launch_rel_mae(const float* a, const float* b, size_t n, float* out3, void* ws, hipStream_t st) {
    int blocks = n ? red_blocks(n) : 0;
    double* part = (double*)ws;
    if (blocks) {
        rel_mae_kernel<<<blocks, RED_THREADS, 0, st>>>(a, b, n, part, blocks == 1 ? out3 : nullptr);
        hipError_t err = hipGetLastError();
        if (err != hipSuccess || blocks == 1) return err;
    }
    finish_rel_mae_kernel<<<1, FIN_THREADS, 0, st>>>(part, blocks, out3);
    return hipGetLastError();
}

}  // namespace ps
