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

// scratch for the K pieces, [piece][row][column] in fp32
constexpr size_t few_workspace_bytes(const FewPlan& p, int batch, int tokens, int Nn) {
    return p.nsplit > 1 ? (size_t)p.nsplit * batch * tokens * Nn * sizeof(float) : 0;
}

}  // namespace ps
