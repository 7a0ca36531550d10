// C[M, Nn] = A[M, K] * W[Nn, K]^T on matrix instructions, bf16 for few and for some thousand rows, fp32 for all: M = all
// rows of the batch, one matrix.
//
// An output's sum depends on its own row of A and column of W only, so a tile may hold rows of several samples; which
// sample a row belongs to matters in the epilogue alone.
//
// With few rows a projection is a stream of weights and is bound by what a compute unit takes from its L2: about 50 bytes
// per ns and CU with the weights coming from memory (56 to 75 from L2; the same through registers and straight into LDS,
// with and without barriers).  So the tile is the widest that still gives every CU one: per output a 64 x 64 tile reads
// twice what a 128 x 128 tile does.  8 waves, two per SIMD, so that one's LDS reads and barrier waits are covered by the other
// (4 waves of 32 x 32 on the 64 x 64 tile: 5760 x 1920 at 112 rows 14.8 us, 8 waves 12.3), an LDS ring of 4 (3 on the widest)
// 64-deep stages filled by direct global->LDS loads, one barrier per stage in front of its last step, whose operands are
// already in registers, the loads of the stage's slot spread over that step.
// us, weights cold, before (64 x 64 tiles of 4 waves without this pipelining; 128 x 128 of 4 waves from 640 tiles of 64 x 64
// on) and after: 7680 x 1920 at 112 / 224 / 448 / 640 rows 14.6 / 19.5 / 30.5 / 30.9 -> 12.8 / 16.3 / 22.4 / 27.7; 1920 x
// 7680 in K pieces (without the reduction) 13.5 / 18.6 / 38.6 / 60.7 -> 11.7 / 16.8 / 22.9 / 28.3; 1920 x 1920 at 4516 rows
// 48.3 -> 37.5.  Then stages without branches and epilogues that request what they read for all their blocks at once: 448 rows x
// 7680 22.4 -> 21.1, 640 rows 27.6 -> 24.8, 1306 rows x 1920 19.1 -> 17.1, 4516 rows 37.5 -> 33.9, K = 7680 at 1306 rows 58.2 ->
// 55.4.  (Not faster: rings of 5 to 8 stages; fragments read a whole stage ahead, 2 to 9 % slower.)
// fp32 (v_mfma_f32_16x16x4_f32: full fp32 products and sums) is bound by the matrix instructions and takes 64 x 64 tiles at
// every size: 5760 x 1920 at 112 tokens 40 us, at 400 101 us (88 TFLOP/s).
#include "few_epilogue.h"
#include "plan.h"
#include <type_traits>

namespace ps {

static constexpr int ROWB = FEW_ROW_BYTES;               // bytes of an operand row per stage: 64 bf16 or 32 fp32

// at most N direct loads may stay in flight
template <int N>
__device__ __forceinline__ void wait_loads() {
    static_assert(N >= 0 && N <= 63, "vmcnt range");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// nsplit: K pieces per output, a workgroup each (INREG: one workgroup per tile adds them up in registers, in the order and with
// the roundings of the reduction).
struct FewGrid { int rows, tiles_m, tiles_n, nsplit; };

// WR x WC waves; a wave computes TM x TN blocks of 16 x 16 outputs.  NST: stages in the LDS ring.
template <typename T, int TM, int TN, int WR, int WC, int NST, int OCC, int KIND, bool INREG>
__global__ void __launch_bounds__(WR * WC * 64, OCC)
gemm_few_kernel(const T* __restrict__ A, const T* __restrict__ W, T* __restrict__ C, int Nn, int K, FewGrid g, Epilogue ep) {
    constexpr int NW = WR * WC, BM = WR * TM * 16, BN = WC * TN * 16;
    // load groups of 8 rows, the same number for every wave: the A rows are filled up (and not multiplied)
    constexpr int GPW = ((BM + BN) / 8 + NW - 1) / NW, AROWS = GPW * NW * 8 - BN, STAGE = (AROWS + BN) * ROWB;
    static_assert(NST >= 2 && NST <= 4, "the stages behind the steady state are written out for rings of up to 4");
    __shared__ __attribute__((aligned(1024))) unsigned char lds[NST * STAGE];
    const int M = g.rows, pieces = INREG ? 1 : g.nsplit;
    int id = xcd_remap(blockIdx.x, gridDim.x), piece, m0, n0;
    // (ids that share an XCD are contiguous, so that the row tiles of one W panel fetch it into that XCD's L2 once)
    if (g.tiles_m <= 8) {
        m0 = id % g.tiles_m * BM; id /= g.tiles_m;
        piece = id % pieces;    n0 = id / pieces * BN;
    } else {                                             // bands of 8 row tiles
        const int tiles = g.tiles_m * g.tiles_n, tile = id % tiles;
        piece = id / tiles;
        const int band = tile / (8 * g.tiles_n), in_band = tile % (8 * g.tiles_n);
        const int rows_here = min(8, g.tiles_m - band * 8);
        m0 = (band * 8 + in_band % rows_here) * BM;
        n0 = in_band / rows_here * BN;
    }
    const int nk = K / (ROWB / (int)sizeof(T));
    const int k0 = nk * piece / pieces, nkt = nk * (piece + 1) / pieces - k0;

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave / WC, wn = wave % WC, l16 = lane & 15, kgrp = lane >> 4;

    // Waves take neighbouring load groups, so that one's loads are all of A, which is in the caches, or all of W, which may come
    // from memory (alternate groups, 7680 x 1920 at 448 rows, weights from memory: 22.1 -> 21.1 us).
    // A load group = 8 rows of the stage [A rows | W rows]; slot p of row r holds 16-byte chunk p ^ ((r >> 1) & 7),
    // so the 16 rows of a fragment read fall into 16 different bank groups; rows past the edge re-read the last one
    // (a group's rows are all of A or all of W: scalar base of the tile, 32-bit offsets inside it)
    const char* base[GPW];
    unsigned off[GPW];
    const long row_bytes = (long)K * sizeof(T);
#pragma unroll
    for (int i = 0; i < GPW; ++i) {
        const int group = wave * GPW + i, row = group * 8 + (lane >> 3);
        const int chunk = (lane & 7) ^ ((row >> 1) & 7);
        const bool of_a = group * 8 < AROWS;
        base[i] = (of_a ? reinterpret_cast<const char*>(A) + (long)m0 * row_bytes : reinterpret_cast<const char*>(W) + (long)n0 * row_bytes) +
                  (long)k0 * ROWB;
        off[i] = (unsigned)(of_a ? min(row, M - 1 - m0) : min(row - AROWS, Nn - 1 - n0)) * (unsigned)row_bytes + chunk * 16;
    }
    const unsigned lds_base = (unsigned)(size_t)PS_LDS_PTR(lds);
    auto issue_one = [&](int kt, int slot, int i) {
        lds_dma16_base(off[i], base[i] + (long)kt * ROWB, __builtin_amdgcn_readfirstlane(lds_base + slot * STAGE + (wave * GPW + i) * 1024));
    };
    auto issue = [&](int kt) {                           // (prologue: stage kt goes to slot kt)
#pragma unroll
        for (int i = 0; i < GPW; ++i) issue_one(kt, kt, i);
    };

    // W fragments are the first operand, A fragments the second: lane l of a 16 x 16 result then holds 4 adjacent
    // output columns (4 * (l / 16) ..) of row l % 16, and the epilogue works on 16-byte quads without a transpose
    // (fp32: the two k steps of a stage have sums of their own, a shorter chain of roundings: error of the fp32 step on
    // 112 tokens against 64 bits 5.3e-7 with them, 5.5e-7 without, 1.36e-6 on the fp32-FMA kernel)
    constexpr int SETS = sizeof(T) == 4 ? 2 : 1;
    f32x4_t acc[SETS][TN][TM], total[INREG ? TN : 1][INREG ? TM : 1];      // total: the pieces before the current one
#pragma unroll
    for (int z = 0; z < SETS; ++z)
#pragma unroll
        for (int y = 0; y < TN; ++y)
#pragma unroll
            for (int x = 0; x < TM; ++x) acc[z][y][x] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    auto piece_sum = [&](int y, int x) {
        f32x4_t v = acc[0][y][x];
        if constexpr (SETS == 2) v += acc[1][y][x];
        return v;
    };
    int piece_end = INREG ? nk / g.nsplit : 0, piece_no = 1;
    if constexpr (INREG) {
#pragma unroll
        for (int y = 0; y < TN; ++y)
#pragma unroll
            for (int x = 0; x < TM; ++x) total[y][x] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }

    // The bias, and on small tiles all that the epilogue reads besides the sums, is requested now, with the first stages, and
    // not when the sums are done (rows and columns past the edge: clamped, not stored).
    // (On 192 x 192 tiles the sums of the pieces before the current one leave no room for it: 12 to 32 registers spilled.  Two
    // layers, four samples of 1100 tokens 972 -> 964 us, eight of 545 942 -> 933.)
    constexpr bool EARLY = TM * TN <= 4, TIGHT = INREG && TM * TN > 12;
    auto col_of = [&](int y) { return n0 + (wn * TN + y) * 16 + kgrp * 4; };
    auto row_of = [&](int x) { return m0 + (wm * TM + x) * 16 + l16; };
    f32x4_t bias[TN];
    EpiOperands eo[EARLY ? TM : 1][EARLY ? TN : 1];
    auto request_bias = [&]() {
#pragma unroll
        for (int y = 0; y < TN; ++y) bias[y] = *reinterpret_cast<const f32x4_t*>(ep.bias + min(col_of(y), Nn - 4));
    };
    if (pieces == 1) {
        if constexpr (!TIGHT) request_bias();
        if constexpr (EARLY) {
#pragma unroll
            for (int x = 0; x < TM; ++x) {
                const int row = min(row_of(x), M - 1);
                const EpiRow r = epilogue_row<KIND>(ep, row);
#pragma unroll
                for (int y = 0; y < TN; ++y) eo[x][y] = epilogue_operands<KIND>(ep, Nn, r, row, min(col_of(y), Nn - 4));
            }
        }
    }

#pragma unroll
    for (int p = 0; p < NST - 1; ++p)
        if (p < nkt) issue(p);
    if (nkt >= NST - 1) wait_loads<(NST - 2) * GPW>();   // own share of stage 0
    else wait_loads<0>();
    __syncthreads();
    if (NST - 1 < nkt) issue(NST - 1);
    const int aoff = (wm * TM * 16 + l16) * ROWB, woff = (AROWS + wn * TN * 16 + l16) * ROWB, sw = (l16 >> 1) & 7;
    auto slot_of = [&](int ks) { return ((ks * 4 + kgrp) ^ sw) << 4; };
    // A fragment x is read again, for the next step, right after the MFMAs that consume it; W fragments are used by
    // every round of a step and are double-buffered
    // (fp32: one 16-byte read gives a lane 4 adjacent k; instruction e multiplies the k = 4 * group + e)
    typedef typename std::conditional<sizeof(T) == 4, f32x4_t, bf16x8_t>::type frag_t;
    frag_t fa[TM], fw[2][TN];
    {
        const int slot = slot_of(0);
#pragma unroll
        for (int y = 0; y < TN; ++y) fw[0][y] = *reinterpret_cast<const frag_t*>(lds + woff + y * 16 * ROWB + slot);
#pragma unroll
        for (int x = 0; x < TM; ++x) fa[x] = *reinterpret_cast<const frag_t*>(lds + aoff + x * 16 * ROWB + slot);
    }
    constexpr int LPR = (GPW + TM - 1) / TM, WPR = (TN + TM - 1) / TM;     // direct loads and W reads per fragment round
    int cur = 0;                                         // ring slot of stage kt
    // One stage.  LEFT: stages after it, NST or more: any number, which is the steady state and has no branch inside.  (Waits and
    // loads behind run-time conditions, seven branches per stage, cost 250 of its cycles: barriers and matrix instructions
    // alone, 128 x 128 tile 0.34 -> 0.24 us per stage, 64 x 64 0.148 -> 0.055, i.e. the matrix rate.)
    auto stage = [&](int kt, auto left_c) {
        constexpr int LEFT = decltype(left_c)::value;
        const int nxt = cur + 1 == NST ? 0 : cur + 1;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const unsigned char* src = lds + cur * STAGE;            // where the next step's fragments come from
            if (ks == 1) {
                if constexpr (LEFT > 0) {
                    wait_loads<(LEFT - 1 < NST - 2 ? LEFT - 1 : NST - 2) * GPW>();   // own share of stage kt + 1 has landed
                    __syncthreads();                     // ... everyone's; and nobody reads stage kt any more
                }
                src = lds + nxt * STAGE;                 // (after the last stage: stale, unused)
                __builtin_amdgcn_sched_barrier(0);
            }
            const int slot = slot_of(ks ^ 1);
#pragma unroll
            for (int x = 0; x < TM; ++x) {
#pragma unroll
                for (int y = 0; y < TN; ++y) {
                    if constexpr (sizeof(T) == 2) {
                        acc[0][y][x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[ks][y], fa[x], acc[0][y][x], 0, 0, 0);
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            acc[ks][y][x] = __builtin_amdgcn_mfma_f32_16x16x4f32(fw[ks][y][e], fa[x][e], acc[ks][y][x], 0, 0, 0);
                    }
                }
#pragma unroll
                for (int y = x * WPR; y < (x + 1) * WPR && y < TN; ++y)
                    fw[ks ^ 1][y] = *reinterpret_cast<const frag_t*>(src + woff + y * 16 * ROWB + slot);
                fa[x] = *reinterpret_cast<const frag_t*>(src + aoff + x * 16 * ROWB + slot);
                if constexpr (LEFT >= NST) {             // into the slot stage kt occupied
                    if (ks == 1) {
#pragma unroll
                        for (int i = x * LPR; i < (x + 1) * LPR && i < GPW; ++i) issue_one(kt + NST, cur, i);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        cur = nxt;
        if constexpr (INREG) {
            if (kt + 1 == piece_end) {                   // (the last piece ends with the last stage)
#pragma unroll
                for (int y = 0; y < TN; ++y)
#pragma unroll
                    for (int x = 0; x < TM; ++x) {
                        total[y][x] += piece_sum(y, x);
#pragma unroll
                        for (int z = 0; z < SETS; ++z) acc[z][y][x] = f32x4_t{0.f, 0.f, 0.f, 0.f};
                    }
                ++piece_no;
                piece_end = nk * piece_no / g.nsplit;
            }
        }
    };
    int kt = 0;
    for (; kt + NST < nkt; ++kt) stage(kt, std::integral_constant<int, NST>{});
    if (NST > 3 && kt + 3 < nkt) stage(kt++, std::integral_constant<int, 3>{});
    if (kt + 2 < nkt) stage(kt++, std::integral_constant<int, 2>{});
    if (kt + 1 < nkt) stage(kt++, std::integral_constant<int, 1>{});
    stage(kt, std::integral_constant<int, 0>{});

    auto sum_of = [&](int y, int x) {
        if constexpr (INREG) return total[y][x]; else return piece_sum(y, x);
    };
    if (pieces > 1) {                                    // [piece][row][column]
#pragma unroll
        for (int x = 0; x < TM; ++x)
#pragma unroll
            for (int y = 0; y < TN; ++y)
                if (row_of(x) < M && col_of(y) < Nn)     // Nn % 4 == 0: a quad is inside or outside
                    *reinterpret_cast<f32x4_t*>(ep.split_ws + ((long)piece * M + row_of(x)) * Nn + col_of(y)) = sum_of(y, x);
        return;
    }
    // Larger tiles: what the epilogue reads is requested for several rows at once (one 16 x 16 block after the other, each
    // waiting for its own: 2 us on 8 blocks per wave, 4 on 16).
    constexpr int CHUNK = EARLY ? TM : TM * TN <= 12 ? TM : 2;
    if constexpr (TIGHT) request_bias();
#pragma unroll
    for (int x0 = 0; x0 < TM; x0 += CHUNK) {
        EpiRow rows[CHUNK];
        EpiOperands late[EARLY ? 1 : CHUNK][EARLY ? 1 : TN];
#pragma unroll
        for (int c = 0; c < CHUNK; ++c) {
            if (x0 + c >= TM) break;
            const int row = min(row_of(x0 + c), M - 1);
            rows[c] = epilogue_row<KIND>(ep, row);
            if constexpr (!EARLY) {
#pragma unroll
                for (int y = 0; y < TN; ++y) late[c][y] = epilogue_operands<KIND>(ep, Nn, rows[c], row, min(col_of(y), Nn - 4));
            }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < CHUNK; ++c) {
            if (x0 + c >= TM) break;
#pragma unroll
            for (int y = 0; y < TN; ++y)
                if (row_of(x0 + c) < M && col_of(y) < Nn)
                    epilogue_quad<KIND, T>(ep, C, Nn, rows[c], row_of(x0 + c), col_of(y), sum_of(y, x0 + c), bias[y],
                                           EARLY ? eo[EARLY ? x0 + c : 0][EARLY ? y : 0] : late[EARLY ? 0 : c][EARLY ? 0 : y]);
        }
    }
}

template <typename T, int KIND, bool INREG>
static hipError_t launch_few_tile(int tile, const T* A, const T* W, T* C, int Nn, int K, const FewGrid& g, const Epilogue& ep,
                                  hipStream_t st) {
    const long blocks = (long)g.tiles_m * g.tiles_n * (INREG ? 1 : g.nsplit);
    if (blocks >= (1L << 31)) return hipErrorInvalidValue;
    auto go = [&](auto kernel) {
        kernel<<<(int)blocks, 512, 0, st>>>(A, W, C, Nn, K, g, ep);
        return hipGetLastError();
    };
    if (tile == FEW_64x64) return go(gemm_few_kernel<T, 1, 2, 4, 2, 4, 2, KIND, INREG>);
    if constexpr (sizeof(T) == 2) {
        switch (tile) {
            case FEW_128x64: return go(gemm_few_kernel<T, 2, 2, 4, 2, 4, 1, KIND, INREG>);
            case FEW_128x128: return go(gemm_few_kernel<T, 2, 4, 4, 2, 4, 1, KIND, INREG>);
            case FEW_192x128: return go(gemm_few_kernel<T, 3, 4, 4, 2, 3, 1, KIND, INREG>);
            case FEW_256x128: return go(gemm_few_kernel<T, 4, 4, 4, 2, 3, 1, KIND, INREG>);
            case FEW_192x192: return go(gemm_few_kernel<T, 3, 6, 4, 2, 3, 1, KIND, INREG>);
        }
    }
    return hipErrorInvalidValue;
}

template <typename T, int KIND>
static hipError_t launch_few_kind(int tile, const T* A, const T* W, T* C, int rows, int Nn, int K, int nsplit, bool inreg,
                                  const Epilogue& ep, int* deferred, hipStream_t st) {
    const Tile& t = kTiles[tile];
    const FewGrid g{rows, (rows + t.bm - 1) / t.bm, (Nn + t.bn - 1) / t.bn, nsplit};
    if (inreg && nsplit > 1) return launch_few_tile<T, KIND, true>(tile, A, W, C, Nn, K, g, ep, st);
    hipError_t e = launch_few_tile<T, KIND, false>(tile, A, W, C, Nn, K, g, ep, st);
    if (e != hipSuccess || nsplit == 1) return e;
    if (deferred && KIND == EPI_GATE_RESIDUAL) { *deferred = nsplit; return e; }
    const long quads = (long)rows * (Nn / 4);
    gemm_few_reduce_kernel<T, KIND><<<(int)((quads + 255) / 256), 256, 0, st>>>(C, Nn, rows, nsplit, ep);
    return hipGetLastError();
}

template <typename T>
static hipError_t launch_few(const T* A, const T* W, T* C, int rows, int Nn, int K, int tile, int nsplit, bool inreg,
                             const Epilogue& ep, int* deferred, hipStream_t st) {
    switch (ep.kind) {
        case EPI_BIAS: return launch_few_kind<T, EPI_BIAS>(tile, A, W, C, rows, Nn, K, nsplit, inreg, ep, deferred, st);
        case EPI_BIAS_GELU: return launch_few_kind<T, EPI_BIAS_GELU>(tile, A, W, C, rows, Nn, K, nsplit, inreg, ep, deferred, st);
        case EPI_GATE_RESIDUAL: return launch_few_kind<T, EPI_GATE_RESIDUAL>(tile, A, W, C, rows, Nn, K, nsplit, inreg, ep, deferred, st);
        case EPI_QKV_ROPE: return launch_few_kind<T, EPI_QKV_ROPE>(tile, A, W, C, rows, Nn, K, nsplit, inreg, ep, deferred, st);
        case EPI_UNPATCHIFY: return launch_few_kind<T, EPI_UNPATCHIFY>(tile, A, W, C, rows, Nn, K, nsplit, inreg, ep, deferred, st);
        default: return hipErrorInvalidValue;
    }
}

// nsplit pieces per output, added up in registers (inreg) or through epi.split_ws.
hipError_t launch_gemm_few(int dtype, const void* A, const void* W, void* C, int batch, int tokens, int Nn, int K, int tile,
                           int nsplit, bool inreg, const Epilogue& epi, int* deferred, hipStream_t st) {
    Epilogue ep = epi;
    ep.geom.tokens = tokens;                             // (the plain kinds leave it unset)
    const int rows = batch * tokens;
    if (dtype == PS_BF16)
        return launch_few<bf16_t>((const bf16_t*)A, (const bf16_t*)W, (bf16_t*)C, rows, Nn, K, tile, nsplit, inreg, ep, deferred, st);
    return launch_few<float>((const float*)A, (const float*)W, (float*)C, rows, Nn, K, tile, nsplit, inreg, ep, deferred, st);
}

}  // namespace ps
