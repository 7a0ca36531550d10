// A whole forward of a narrow fp32 network (see slim_network) in layers + 1 launches.
//
// In such a network every operation of a layer is a few microseconds of latency: a launch, the loads of its operands, a
// short chain of products (2 layers of 64 on 32 tokens: 17 launches of 3.3 to 6.5 us).  Everything but attention's keys and
// values belongs to one token, and 16 tokens' rows fit LDS many times over, so a workgroup of four waves takes 16 tokens
// through all that lies between two attentions: attention itself (a wave per head, keys and values straight from memory
// into operand layout), output projection, LayerNorm, MLP, and the next layer's LayerNorm and q, k, v -- or, after the last
// layer, the final projection.  The first launch embeds and does the first layer's q, k, v.  Weights come from L2 in operand
// layout, requested a phase ahead, across the barrier in front of their use.
// fp32 products and sums on v_mfma_f32_16x16x4_f32 throughout; instruction e of a 16-deep step multiplies k = 4 * (lane / 16)
// + e, even and odd steps have sums of their own.
// us per forward of 2 layers of hidden 64 with the launches of the conditioning, a launch per operation and this: 32 tokens
// 94 and 42, 128 tokens 98 and 42, 416 tokens 112 and 55.
#include "few_epilogue.h"
#include "lane_sums.h"
#include "slim.h"

namespace ps {

namespace {

constexpr int ROWS = 16;                                 // tokens of a workgroup
__device__ __forceinline__ f32x4_t quad(const float* p) { return *reinterpret_cast<const f32x4_t*>(p); }

// One wave's share of out = in * W^T: 16-column blocks wave, wave + 4, ... (NF of them, `blocks` in all), K = 16 * KB.
// The weights of the first blocks are requested by request(), the others when their turn comes.
template <int KB, int NF>
struct Project {
    static constexpr int G = KB >= 16 ? 1 : NF * KB <= 16 ? NF : 16 / KB;
    static constexpr int LOADS = G * KB, STEPS = NF * KB;
    f32x4_t pre[G][KB];
    const float* W;
    int wave, blocks;
    __device__ __forceinline__ void load(int j, f32x4_t (&w)[KB]) const {
        const int lane = threadIdx.x & 63, col = min(wave + 4 * j, blocks - 1) * 16 + (lane & 15);
        const float* p = W + (long)col * (16 * KB) + (lane >> 4) * 4;
#pragma unroll
        for (int i = 0; i < KB; ++i) w[i] = quad(p + i * 16);
    }
    __device__ __forceinline__ void prepare(const float* weights, int w, int n) { W = weights; wave = w; blocks = n; }
    __device__ __forceinline__ void request(const float* weights, int w, int n) {
        prepare(weights, w, n);
#pragma unroll
        for (int j = 0; j < G; ++j) load(j, pre[j]);
    }
    // its share of step s of `steps`
    __device__ __forceinline__ void request_step(int s, int steps) {
        const int lane = threadIdx.x & 63, per = (LOADS + steps - 1) / steps;
#pragma unroll
        for (int u = s * per; u < (s + 1) * per && u < LOADS; ++u) {
            const int col = min(wave + 4 * (u / KB), blocks - 1) * 16 + (lane & 15);
            pre[u / KB][u % KB] = quad(W + col * (16 * KB) + (lane >> 4) * 4 + u % KB * 16);
        }
    }
    // in: LDS, this lane's row (lane % 16); epi(j, first of the lane's 4 columns, sums) for its j-th block.  between(s): what
    // goes behind the s-th four products, the loads of another projection: issued in one go they held the products up for as
    // long as a compute unit takes to accept them, about 160 cycles for one of each wave.
    template <class Epi, class Between>
    __device__ __forceinline__ void run(const float* in, Epi epi, Between between) const {
        const int kgrp = (threadIdx.x & 63) >> 4;
        f32x4_t a[KB];
#pragma unroll
        for (int i = 0; i < KB; ++i) a[i] = quad(in + i * 16 + kgrp * 4);
#pragma unroll
        for (int j = 0; j < NF; ++j) {
            if (wave + 4 * j >= blocks) {                // (whole wave)
#pragma unroll
                for (int i = 0; i < KB; ++i) between(j * KB + i);
                continue;
            }
            f32x4_t later[KB], s[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
            if (j >= G) load(j, later);
#pragma unroll
            for (int i = 0; i < KB; ++i) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    s[i & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(j < G ? pre[j < G ? j : 0][i][e] : later[i][e], a[i][e], s[i & 1], 0, 0, 0);
                between(j * KB + i);
            }
            epi(j, (wave + 4 * j) * 16 + kgrp * 4, s[0] + s[1]);
        }
    }
    template <class Epi>
    __device__ __forceinline__ void run(const float* in, Epi epi) const { run(in, epi, [](int) {}); }
};

// What the phases read besides activations and weights -- biases, gates, modulation, rotary table -- is requested with the
// first loads of a launch, or behind its attention: asked for when its turn came, each of the six was a trip to L2 in the middle
// of the chain (8 steps of 2 layers of 64 on 128 tokens: 386 -> 352 us).
// BlockVec: 4 columns of each of a wave's blocks of 16.
template <int NF>
struct BlockVec {
    f32x4_t v[NF];
    __device__ __forceinline__ void request(const float* p, int wave, int blocks) {
        const int kgrp = (threadIdx.x & 63) >> 4;
#pragma unroll
        for (int j = 0; j < NF; ++j) v[j] = quad(p + min(wave + 4 * j, blocks - 1) * 16 + kgrp * 4);
    }
};

// out = LN(in) * (1 + scale) + shift for rows 4 * wave + lane / 16; shift, scale: of that row
template <int D>
struct SlimNorm {
    static constexpr int V = D / 16;                     // adjacent values of a lane
    typedef __attribute__((ext_vector_type(V))) float vec;
    vec h, k;
    static __device__ __forceinline__ vec at(const float* p) { return *reinterpret_cast<const vec*>(p + (threadIdx.x & 15) * V); }
    __device__ __forceinline__ void request(const float* shift, const float* scale) { h = at(shift); k = at(scale); }
    __device__ __forceinline__ void run(const float* in, float* out, float eps) const {
        vec v = at(in), o;
        float s = 0.f, q = 0.f;
#pragma unroll
        for (int i = 0; i < V; ++i) s += v[i];
        const float mean = sum_of_16(s) / (float)D;
#pragma unroll
        for (int i = 0; i < V; ++i) q += (v[i] - mean) * (v[i] - mean);
        const float rstd = 1.0f / sqrtf(sum_of_16(q) / (float)D + eps);
#pragma unroll
        for (int i = 0; i < V; ++i) o[i] = (v[i] - mean) * rstd * (1.f + k[i]) + h[i];
        *reinterpret_cast<vec*>(out + (threadIdx.x & 15) * V) = o;
    }
};

// q, k, v of a row block: bias, rotation, store
template <int D>
struct SlimQkv {
    static constexpr int NF = (3 * D / 16 + 3) / 4, BLOCKS = 3 * D / 16;
    Epilogue ep;
    EpiRow r;
    int row;
    BlockVec<NF> bias;
    EpiOperands o[NF];
    __device__ __forceinline__ void request(const SlimArgs& g, const SlimLayer& w, int wave, int b, int n) {
        ep = Epilogue{};
        ep.kind = EPI_QKV_ROPE; ep.bias = w.b_qkv; ep.D = D; ep.geom = TokenGeom{g.tokens, g.text_tokens};
        ep.rope_cs = g.rope; ep.rope_F = g.pg.F; ep.rope_Hp = g.pg.H / g.pg.patch; ep.rope_Wp = g.pg.W / g.pg.patch;
        ep.head_dim = g.head_dim; ep.q_scale = 1.0f;
        row = b * g.tokens + min(n, g.tokens - 1);
        r = epilogue_row<EPI_QKV_ROPE>(ep, row);
        bias.request(w.b_qkv, wave, BLOCKS);
        const int kgrp = (threadIdx.x & 63) >> 4;
#pragma unroll
        for (int j = 0; j < NF; ++j)
            o[j] = epilogue_operands<EPI_QKV_ROPE>(ep, 3 * D, r, row, min(wave + 4 * j, BLOCKS - 1) * 16 + kgrp * 4);
    }
    __device__ __forceinline__ void run(const SlimArgs& g, const Project<D / 16, NF>& pj, const float* in, int n) const {
        pj.run(in, [&](int j, int col, f32x4_t x) {
            if (n < g.tokens) epilogue_quad<EPI_QKV_ROPE, float>(ep, g.qkv_out, 3 * D, r, row, col, x, bias.v[j], o[j]);
        });
    }
};

// Embedding, first LayerNorm and q, k, v.  P = 16 * PB values per patch.
template <int D, int PB>
__global__ void __launch_bounds__(256, 1) slim_begin_kernel(SlimArgs g, SlimLayer w) {
    constexpr int LD = D + 4, P = 16 * PB, LP = P + 4;   // rows 16-byte aligned, 4 banks apart
    __shared__ __attribute__((aligned(16))) float pt[ROWS * LP], xt[ROWS * LD], ht[ROWS * LD];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15;
    const int n0 = blockIdx.x * ROWS, b = blockIdx.y, N = g.tokens, L = g.text_tokens;
    const int n = n0 + l16;                              // this lane's row in the projections
    Project<PB, (D / 16 + 3) / 4> embed;
    embed.request(g.W_pe, wave, D / 16);
    Project<D / 16, (3 * D / 16 + 3) / 4> qkv;
    qkv.request(w.W_qkv, wave, 3 * D / 16);
    BlockVec<(D / 16 + 3) / 4> b_pe;
    b_pe.request(g.b_pe, wave, D / 16);
    const int nr = wave * 4 + (lane >> 4);               // this lane's row in the LayerNorm
    SlimNorm<D> norm;
    {
        const float* m = g.mod + b * g.mod_bs + (n0 + nr < L ? 6 * D : 0);
        norm.request(m, m + D);
    }
    SlimQkv<D> out;
    out.request(g, w, wave, b, n);
    const PatchGeom& pg = g.pg;
    const int Hp = pg.H / pg.patch, Wp = pg.W / pg.patch, ps2 = pg.patch * pg.patch;
    for (int e = threadIdx.x; e < ROWS * P; e += 256) {
        const int r = e & 15, p = e >> 4, nv = n0 + r - L;
        float v = 0.f;
        if (nv >= 0 && n0 + r < N) {
            const int j = nv % Wp, i = (nv / Wp) % Hp, f = nv / (Wp * Hp), c = p / ps2, dy = p % ps2 / pg.patch, dx = p % pg.patch;
            v = g.x[(((long)b * pg.C + c) * pg.F + f) * pg.H * pg.W + (long)(i * pg.patch + dy) * pg.W + j * pg.patch + dx];
        }
        pt[r * LP + p] = v;
    }
    __syncthreads();
    embed.run(pt + l16 * LP, [&](int j, int col, f32x4_t x) {
        x += b_pe.v[j];
        if (n < L) x = quad(g.ctx + b * g.ctx_bs + (long)n * D + col);
        *reinterpret_cast<f32x4_t*>(xt + l16 * LD + col) = x;
        if (n < N) *reinterpret_cast<f32x4_t*>(g.X + ((long)b * N + n) * D + col) = x;
    });
    __syncthreads();
    norm.run(xt + nr * LD, ht + nr * LD, g.eps);
    __syncthreads();
    out.run(g, qkv, ht + l16 * LD, n);
}

// One layer from its attention on; `next`: the following layer's q, k, v, or after the last layer the final projection.
// A wave's code runs once, on one wave per SIMD: every instruction counts, and so does every line of it that comes from L2.
// So the first keys and values are requested first of all and everything else in their shadow, divisions of positions
// included, and exponentials and GELU take six and 19 instructions (in the math library an exponential is 13, a tanh 35).  What a
// compute unit accepts of loads, 112 to 196 KB of weights per layer, is the other bound: they are issued between products, not
// ahead of them.  Cycles of a layer of 64 on 128 tokens, one after the other / the requests in attention's shadow / and between
// products: 34700 / 29800 / 26000, the last layer 42500 / 25300 / 23400; 8 steps of 2 such layers 352 / 301 / 285 us, with W_1
// behind the attention and LayerNorm's vectors in one load each 272.  Of this, exponentials and GELU had lost digits; as exact
// as the math library's 282, with its expf 287.  (Slower: values stored [column][token] for 16-byte loads, 285 -> 287; W_1
// between W_o's products, 270 -> 278.)
// Workgroups per compute unit, four waves each: 16 samples of 800 tokens of hidden 32 take 158 us in heads of 16 with two and 219
// in heads of 32 with one, 137 and 166 with three and two (three at the price of 12 to 20 spilled registers).
template <int D, int HD, bool LAST>
__global__ void __launch_bounds__(256, (D == 32) + (HD == 16) + 1) slim_layer_kernel(SlimArgs g, SlimLayer w, SlimLayer next) {
    constexpr int LD = D + 4, F = 4 * D, LF = F + 4, NB = HD / 16, HEADS = D / HD;
    static_assert(HEADS <= 4, "a wave per head");
    __shared__ __attribute__((aligned(16))) float xt[ROWS * LD], ht[ROWS * LD], ut[ROWS * LF];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, kgrp = lane >> 4;
    const int n0 = blockIdx.x * ROWS, b = blockIdx.y, N = g.tokens, L = g.text_tokens;
    const int n = n0 + l16, row = b * N + min(n, N - 1);
    // attention: a wave per head, its 16 queries in lane % 16.  S^T = K Q^T leaves keys 4 * (lane / 16) + i of every 16-key
    // block, the layout the second operand of O^T = V^T P^T wants: the probabilities stay in their registers, in fp32.
    const int head = min(wave, HEADS - 1);
    const float* base = g.qkv + (long)b * N * 3 * D + head * HD;
    f32x4_t qf[NB];
#pragma unroll
    for (int d = 0; d < NB; ++d) qf[d] = quad(base + (row - b * N) * 3 * D + d * 16 + kgrp * 4);
    f32x4_t kn[4][NB];                                   // the next 64 keys (past the end: the last one again, masked)
    float vn[4][4][NB];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int d = 0; d < NB; ++d) {
                kn[t][d] = quad(base + min(k0 + t * 16 + l16, N - 1) * 3 * D + D + d * 16 + kgrp * 4);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    vn[t][e][d] = base[min(k0 + t * 16 + kgrp * 4 + e, N - 1) * 3 * D + 2 * D + d * 16 + l16];
            }
    };
    fetch(0);
    __builtin_amdgcn_sched_barrier(0);

    const float* mod = g.mod + b * g.mod_bs + (long)g.layer * 12 * D;
    const float* gates = mod + (n < L ? 6 * D : 0);      // of this lane's row
    Project<D / 16, (D / 16 + 3) / 4> po;
    po.request(w.W_o, wave, D / 16);
    constexpr int XV = ROWS * (D / 4) / 256 > 0 ? ROWS * (D / 4) / 256 : 1;
    f32x4_t x_in[XV];
#pragma unroll
    for (int i = 0; i < XV; ++i) {
        const int e = min((int)threadIdx.x + 256 * i, ROWS * (D / 4) - 1);
        x_in[i] = quad(g.X + ((long)b * N + min(n0 + e / (D / 4), N - 1)) * D + e % (D / 4) * 4);
    }
    constexpr int NO = (D / 16 + 3) / 4;
    const int nr = wave * 4 + kgrp;                      // this lane's row in the LayerNorms
    BlockVec<NO> b_o, gate_a;
    b_o.request(w.b_o, wave, D / 16);
    gate_a.request(gates + 2 * D, wave, D / 16);
    SlimNorm<D> mid;
    {
        const float* m = mod + (n0 + nr < L ? 6 * D : 0);
        mid.request(m + 3 * D, m + 4 * D);
    }
    BlockVec<D / 16> b_1;
    b_1.request(w.b_1, wave, F / 16);
    BlockVec<NO> b_2, gate_m;
    b_2.request(w.b_2, wave, D / 16);
    gate_m.request(gates + 5 * D, wave, D / 16);
    SlimNorm<D> end;
    {
        const float* m = LAST ? g.modf + b * 2 * D : mod + 12 * D + (n0 + nr < L ? 6 * D : 0);
        end.request(m, m + D);
    }
    const int P = g.pg.C * g.pg.patch * g.pg.patch;
    BlockVec<1> b_out;
    SlimQkv<D> out;
    int at[4];                                           // where this lane's four values of a patch lie in the latent
    if constexpr (LAST) {
        b_out.request(g.b_out, wave, P / 16);
        const PatchGeom& pg = g.pg;
        const int Hp = pg.H / pg.patch, Wp = pg.W / pg.patch, ps2 = pg.patch * pg.patch, nv = max(min(n, N - 1) - L, 0);
        const int q1 = nv / Wp, pj = nv - q1 * Wp, f = q1 / Hp, pi = q1 - f * Hp;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int q = wave * 16 + kgrp * 4 + c, ch = q / ps2, in = q - ch * ps2, dy = in / pg.patch, dx = in - dy * pg.patch;
            at[c] = (((b * pg.C + ch) * pg.F + f) * pg.H + pi * pg.patch + dy) * pg.W + pj * pg.patch + dx;
        }
    } else {
        out.request(g, next, wave, b, n);
    }
    __builtin_amdgcn_sched_barrier(0);

    if (wave < HEADS) {
        f32x4_t acc[NB];
#pragma unroll
        for (int d = 0; d < NB; ++d) { qf[d] *= g.scale; acc[d] = f32x4_t{0.f, 0.f, 0.f, 0.f}; }
        float m = -INFINITY, l = 0.f;                    // l: over this lane's keys only
        for (int k0 = 0; k0 < N; k0 += 64) {
            f32x4_t kf[4][NB], sc[4];
            float vf[4][4][NB];
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int d = 0; d < NB; ++d) {
                    kf[t][d] = kn[t][d];
#pragma unroll
                    for (int e = 0; e < 4; ++e) vf[t][e][d] = vn[t][e][d];
                }
            if (k0 + 64 < N) fetch(k0 + 64);
#pragma unroll
            for (int t = 0; t < 4; ++t) sc[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int d = 0; d < NB; ++d)
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int t = 0; t < 4; ++t) sc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[t][d][e], qf[d][e], sc[t], 0, 0, 0);
            float tmax = -INFINITY, tmin = INFINITY;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                tmax = fmaxf(tmax, fmaxf(fmaxf(sc[t][0], sc[t][1]), fmaxf(sc[t][2], sc[t][3])));
                tmin = fminf(tmin, fminf(fminf(sc[t][0], sc[t][1]), fminf(sc[t][2], sc[t][3])));
            }
            tmax = max_xor32(max_xor16(tmax));
            const float mn = fmaxf(m, tmax), alpha = expf(m - mn);   // exp(-inf) = 0 on the first keys
            m = mn;
            l *= alpha;
#pragma unroll
            for (int d = 0; d < NB; ++d) acc[d] *= alpha;
            const bool near = __ballot(tmin - mn < EXP_NEAR) == 0;       // (of the whole wave)
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) sc[t][i] -= mn;
            if (near) {
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int i = 0; i < 4; ++i) sc[t][i] = exp_near(sc[t][i]);
            } else {
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int i = 0; i < 4; ++i) sc[t][i] = expf(sc[t][i]);
            }
            if (k0 + 64 > N) {                           // keys past the end (the last one again): no weight, and no value
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (k0 + t * 16 + kgrp * 4 + i >= N) {
                            sc[t][i] = 0.f;
#pragma unroll
                            for (int d = 0; d < NB; ++d) vf[t][i][d] = 0.f;
                        }
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) {
#pragma unroll
                for (int i = 0; i < 4; ++i) l += sc[t][i];
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int d = 0; d < NB; ++d) acc[d] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[t][e][d], sc[t][e], acc[d], 0, 0, 0);
            }
        }
        l = sum_xor32(sum_xor16(l));
#pragma unroll
        for (int d = 0; d < NB; ++d) *reinterpret_cast<f32x4_t*>(ht + l16 * LD + head * HD + d * 16 + kgrp * 4) = acc[d] / l;
    }
    Project<D / 16, D / 16> p1;
    p1.request(w.W_1, wave, F / 16);
#pragma unroll
    for (int i = 0; i < XV; ++i) {
        const int e = threadIdx.x + 256 * i;
        if (e < ROWS * (D / 4)) *reinterpret_cast<f32x4_t*>(xt + e / (D / 4) * LD + e % (D / 4) * 4) = x_in[i];
    }
    __syncthreads();
    auto residual = [&](const BlockVec<NO>& bias, const BlockVec<NO>& gate) {
        return [=](int j, int col, f32x4_t x) {
            float* at = xt + l16 * LD + col;
            *reinterpret_cast<f32x4_t*>(at) = quad(at) + gate.v[j] * (x + bias.v[j]);
        };
    };
    po.run(ht + l16 * LD, residual(b_o, gate_a));
    __syncthreads();
    mid.run(xt + nr * LD, ht + nr * LD, g.eps);
    __syncthreads();
    Project<F / 16, NO> p2;
    p2.prepare(w.W_2, wave, D / 16);
    Project<D / 16, LAST ? 1 : (3 * D / 16 + 3) / 4> pn;
    pn.prepare(LAST ? g.W_out : next.W_qkv, wave, LAST ? P / 16 : 3 * D / 16);
    p1.run(ht + l16 * LD, [&](int j, int col, f32x4_t x) {
        x += b_1.v[j];
#pragma unroll
        for (int c = 0; c < 4; ++c) x[c] = gelu_of(x[c], 0.f);
        *reinterpret_cast<f32x4_t*>(ut + l16 * LF + col) = x;
    }, [&](int s) {
        p2.request_step(s, p1.STEPS);
        __builtin_amdgcn_sched_barrier(0);
    });
    __syncthreads();
    p2.run(ut + l16 * LF, residual(b_2, gate_m), [&](int s) {
        pn.request_step(s, p2.STEPS);
        __builtin_amdgcn_sched_barrier(0);
    });
    __syncthreads();
    if constexpr (LAST) {
        end.run(xt + nr * LD, ht + nr * LD, g.eps);
        __syncthreads();
        pn.run(ht + l16 * LD, [&](int j, int col, f32x4_t x) {
            x += b_out.v[j];
            if (n < N && n >= L)
#pragma unroll
                for (int c = 0; c < 4; ++c) g.eps_out[at[c]] = x[c];
        });
    } else {
        for (int e = threadIdx.x; e < ROWS * (D / 4); e += 256) {
            const int r = e / (D / 4), c = e % (D / 4) * 4;
            if (n0 + r < N) *reinterpret_cast<f32x4_t*>(g.X + ((long)b * N + n0 + r) * D + c) = quad(xt + r * LD + c);
        }
        end.run(xt + nr * LD, ht + nr * LD, g.eps);
        __syncthreads();
        out.run(g, pn, ht + l16 * LD, n);
    }
}

template <int D>
hipError_t launch_begin_as(const SlimArgs& g, const SlimLayer& w, int batch, hipStream_t st) {
    const dim3 grid((g.tokens + ROWS - 1) / ROWS, batch);
    switch (g.pg.C * g.pg.patch * g.pg.patch / 16) {
        case 1: slim_begin_kernel<D, 1><<<grid, 256, 0, st>>>(g, w); break;
        case 2: slim_begin_kernel<D, 2><<<grid, 256, 0, st>>>(g, w); break;
        case 3: slim_begin_kernel<D, 3><<<grid, 256, 0, st>>>(g, w); break;
        case 4: slim_begin_kernel<D, 4><<<grid, 256, 0, st>>>(g, w); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int D, int HD>
hipError_t launch_layer_as(const SlimArgs& g, const SlimLayer& w, const SlimLayer* next, int batch, hipStream_t st) {
    const dim3 grid((g.tokens + ROWS - 1) / ROWS, batch);
    if (next) slim_layer_kernel<D, HD, false><<<grid, 256, 0, st>>>(g, w, *next);
    else slim_layer_kernel<D, HD, true><<<grid, 256, 0, st>>>(g, w, w);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_slim_begin(const SlimArgs& g, int hidden, const SlimLayer& first, int batch, hipStream_t st) {
    switch (hidden) {
        case 32: return launch_begin_as<32>(g, first, batch, st);
        case 64: return launch_begin_as<64>(g, first, batch, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_slim_layer(const SlimArgs& g, int hidden, const SlimLayer& layer, const SlimLayer* next, int batch, hipStream_t st) {
    switch (hidden * 100 + g.head_dim) {
        case 3216: return launch_layer_as<32, 16>(g, layer, next, batch, st);
        case 3232: return launch_layer_as<32, 32>(g, layer, next, batch, st);
        case 6416: return launch_layer_as<64, 16>(g, layer, next, batch, st);
        case 6432: return launch_layer_as<64, 32>(g, layer, next, batch, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace ps
