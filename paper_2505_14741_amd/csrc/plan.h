// Rules that say which thread or workgroup computes what: plain arithmetic on sizes, without device code, so that a host
// program can evaluate them at sizes no test can run.  (constexpr functions are callable from kernels as they are.)
#pragma once

#include <stddef.h>

namespace ps {

// ---- merge of attention's key pieces: 16 threads per query row, 16 rows per workgroup of 256
struct MergeRow { int item, row, d4; };              // split item (over all samples), its row, group of 4 outputs
// Counted in rows: a launch holds fewer than 2^32 threads, i.e. fewer than 2^28 rows, so a row index fits 32 bits where a
// thread index does not (524800 items of 256 rows are 2^31 + 2 * 10^6 threads).
constexpr MergeRow merge_row(int block, int thread, int bq) {
    const int rowid = block * 16 + (thread >> 4);
    return MergeRow{rowid / bq, rowid % bq, thread & 15};
}

// ---- projections of few tokens and of fp32 operands (gemm_small.hip): C[tokens, Nn] = A[tokens, K] * W[Nn, K]^T per sample
constexpr int FEW_TILE = 64;                             // output rows and columns of a workgroup
constexpr int FEW_ROW_BYTES = 128;                       // bytes of an operand row per stage: 64 bf16 or 32 fp32

// A sample's plan: a function of the sample's shape alone, so that its result does not depend on the batch.
//   bf16: up to 640 tiles of 64 x 64; beyond that the 128-wide tiles of the other kernel win by reading less per output.
//     Weights cold / in cache, against 128 x 128 tiles: 5760 x 1920 weights at 440 tokens (630 tiles) 27.4 / 20.7 against
//     29.9 / 22.7 us; 7680 x 1920 at 300 (600) 27.5 / 20.5 against 29.5 / 22.1; 1920 x 1920 at 1340 (630) 21.2 / 21.1
//     against 23.0 / 23.0, at 1500 (720) 26.4 against 24.3 cold.
//     K >= 4096: up to 512.  Beyond, no tile has a second K piece here, while 128 x 128 tiles are cut: 1920 x 7680 at 1100
//     tokens (540 tiles) 78.9 / 76.8 whole here, 58.5 / 54.6 in 3 pieces there; at 1000 (480) 61.1 / 49.0 here.
//   fp32: every size (the matrix instructions bind, 32 cycles per 2048 operations, not the LDS reads).
// K pieces: as many as bring the workgroups to 256 (one per compute unit) where K is short, 512 where it is long (60
// stages and more), 8 at most (fp32 16) and each at least 5 stages.  1920 x 1920 bf16 at 112 tokens (60 tiles): 1 piece 14.2 us,
// 4 pieces 11.5, 6 pieces 12.2 with the reduction launch; 1920 x 7680: 42.8, 19.0 (4 pieces), 18.5 (8).
// path: kernel path (low byte 1: generic kernels, 4: no K pieces).
struct FewPlan { bool use; int tiles_m, tiles_n, nsplit; };
constexpr FewPlan few_plan(bool bf16, int tokens, int Nn, int K, int path) {
    FewPlan p{false, 0, 0, 1};
    const long row_bytes = (long)K * (bf16 ? 2 : 4);
    if ((path & 0xff) == 1 || row_bytes % FEW_ROW_BYTES != 0 || Nn % 4 != 0 || tokens < 1) return p;
    p.tiles_m = (tokens + FEW_TILE - 1) / FEW_TILE;
    p.tiles_n = (Nn + FEW_TILE - 1) / FEW_TILE;
    const long tiles = (long)p.tiles_m * p.tiles_n, nk = row_bytes / FEW_ROW_BYTES;
    if (bf16 && (Nn < 64 || tiles > (K >= 4096 ? 512 : 640))) return p;
    p.use = true;
    if ((path & 0xff) == 4) return p;
    const long most = bf16 ? 8 : 16;
    long ns = (nk >= 60 ? 512 : 256) / tiles;
    ns = ns < most ? ns : most;
    ns = ns < nk / 5 ? ns : nk / 5;
    p.nsplit = ns > 1 ? (int)ns : 1;
    return p;
}

// What runs a batch of samples of one plan.  It counts the tiles of the whole batch; the values are the same either way (same
// instruction, same order of k, pieces added in the same order, same epilogue).
//   FEW_PIECES  a workgroup per 64 x 64 tile and K piece; the pieces pass through memory
//   FEW_INREG   a workgroup per 64 x 64 tile, which adds its pieces in registers
//   FEW_TILES   128-wide tiles of the other kernel, pieces in registers (bf16)
// Pieces of their own pay until the tiles alone occupy the chip.  Layer with cold weights, us, pieces apart / in registers:
// 1920 x 1920 and the LayerNorm that adds the pieces, 112 tokens: 3 samples (180 tiles) 19.3 / 21.5, 4 (240) 23.1 / 22.0,
// 8 (480) 37.1 / 26.3; 1920 x 7680, 4 samples (240) 42.1 / 50.2, 6 (360) 57.5 / 62.4, 8 (480) 74.1 / 62.2.  fp32 is bound by
// the matrix instructions and takes finer pieces longer: 1920 x 7680 at 320 tokens, 4 samples (600 tiles) 358 / 393, 8 (1200)
// 674 / 654.
// 128-wide tiles need 512 of themselves for a round and take about as long for fewer; 64-wide ones, 0.036 us each: 5760 x
// 1920, 112 tokens, 4 samples (720 tiles) 28.2 against 32.9, 6 (1080) 39.1 / 34.3, 16 (2880) 96.3 / 68.9.  In samples of up
// to 64 tokens a 128-row tile is at least half empty: 16 of 32 tokens (1440) 42.4 / 56.7.
enum FewHow { FEW_PIECES, FEW_INREG, FEW_TILES };
constexpr long few_spread_tiles(bool bf16, int K) { return !bf16 ? 640 : K >= 60 * 64 ? 384 : 256; }
constexpr FewHow few_how(bool bf16, const FewPlan& p, int batch, int K) {
    const long tiles = (long)batch * p.tiles_m * p.tiles_n;
    if (p.nsplit > 1 && tiles < few_spread_tiles(bf16, K)) return FEW_PIECES;
    return bf16 && tiles > 768 && p.tiles_m > 1 ? FEW_TILES : FEW_INREG;
}

// scratch for the K pieces, [piece][row][column] in fp32; does not shrink with the batch
constexpr size_t few_workspace_bytes(bool bf16, const FewPlan& p, int batch, int tokens, int Nn, int K) {
    if (p.nsplit == 1) return 0;
    const long most = (few_spread_tiles(bf16, K) - 1) / ((long)p.tiles_m * p.tiles_n);   // the largest batch of FEW_PIECES
    return (size_t)p.nsplit * (batch < most ? batch : most) * tokens * Nn * sizeof(float);
}

}  // namespace ps
