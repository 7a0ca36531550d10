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

// ---- bf16 attention of samples whose items of 256 queries do not fill the chip: whether workgroups of 128 queries, alone, are
// faster than workgroups of 256 and the launch that looks their results through.  `bh`: (batch, head) pairs.
// Measured us per tile of 64 keys: 512 workgroups of 128 queries 1.25, up to 256 of them 0.98; of 256 queries 2.27 and 1.29; a
// single round that puts two on some compute units only is between them, nearer the full one.  A launch more costs 4 us; over
// several rounds the narrow ones, which read K and V twice as often, lose another 6 %.  Whole calls, narrow / wide us: 30 heads,
// 1000 keys, 4 and 8 samples 46.8 / 48.5 and 87.7 / 85.2, 2608 keys 88 / 90, two samples 131 / 130, four 245 / 243, 3600 keys 135 / 117;
// 16 heads, 3000 keys 59 / 60, 4200 keys 127 / 119; 4 heads, 6000 keys 84 / 107, 17776 keys 503 / 461.
// (On 278 shapes of 32 to 17776 keys and 1 to 3200 (batch, head) pairs the one picked is 3.2 % slower than the other at most.)
constexpr bool attn_narrow_items(long bh, int seq, int cus) {
    const long slots = 2L * cus, narrow = bh * ((seq + 127) / 128), wide = bh * ((seq + 255) / 256);
    const auto rounds = [slots, cus](long n, float full, float half) {
        const long tail = n % slots;
        if (n < slots && tail > cus) return full * (0.92f + 0.08f * (float)(tail - cus) / cus);
        return (float)(n / slots) * full + (tail == 0 ? 0.f : tail <= cus ? half : full);
    };
    const float tiles = (float)((seq + 63) / 64);
    const float a = tiles * rounds(narrow, 1.25f, 0.98f) * (narrow > 2 * slots ? 1.06f : 1.f);
    return a <= tiles * rounds(wide, 2.27f, 1.29f) + 4.f;
}

// Split plan of the bf16 head-dim-64 kernels: per sample, how many work items of 256 queries run whole and how many ways the
// rest is split along the keys.
struct AttnPlan { int qblocks, items_ps, full_ps, tail_ps, nsplit, bq; };
constexpr AttnPlan attention_plan(int seq, int heads, int cus) {
    constexpr int KV = 64;
    AttnPlan p{};
    p.bq = 256;
    p.qblocks = (seq + p.bq - 1) / p.bq;
    p.items_ps = p.qblocks * heads;
    const int slots = cus * 2;                           // two resident workgroups per CU
    const int tail = p.items_ps % slots;
    const int ntiles = (seq + KV - 1) / KV;
    // Fewer items than slots are never split: the plan must not depend on the batch, and a batch that fills the chip by
    // itself pays 70 KB of partial sums per piece for nothing.  (4 heads x 4096 keys in two pieces: 74 -> 49 us alone, but
    // 80 -> 94 for four samples and 256 -> 330 for sixteen; 16 heads x 1000 keys, four samples: 30 -> 50.)
    int ns = tail > 0 ? slots / tail : 1;
    if (ns > 8) ns = 8;
    if (ns > ntiles / 2) ns = ntiles / 2;
    if (tail == 0 || p.items_ps < slots || ns < 2) { p.full_ps = p.items_ps; p.tail_ps = 0; p.nsplit = 1; }
    else { p.full_ps = p.items_ps - tail; p.tail_ps = tail; p.nsplit = ns; }
    return p;
}

// Which kernels a bf16 head-dim-64 call takes.
//   ATTN_BY_128   attn_sp_kernel alone, 128 queries per workgroup, which redoes its own failures
//   ATTN_BY_256   attn_sp_kernel with 256 queries per workgroup, then attn_redo_kernel
//   ATTN_FLAGS    attn_sp_kernel marks the (batch, head) pairs it could not do, attn_mfma_kernel redoes those; key pieces
//   ATTN_TRACKED  attn_mfma_kernel for every head
// Samples whose items do not fill the chip take one of the first two: no split, no flags; the values of the two are the same,
// so the whole batch may decide between them.  Which samples these are must not depend on the batch, and a large batch of short
// ones is slower so than it was on attn_mfma_kernel alone: 30 heads x 512 keys, 16 samples 49.2 -> 51.4 us, 200 keys 22.5 ->
// 23.9 (one sample 17.7 -> 12.6 and 12.1 -> 8.7).
// Samples of 512 items and more (256 heads and more) of up to 512 keys: the second launch of ATTN_FLAGS costs more than the
// faster loop gains.
// path: kernel path (low byte 3: ATTN_TRACKED always).
enum AttnRoute { ATTN_BY_128, ATTN_BY_256, ATTN_FLAGS, ATTN_TRACKED };
constexpr AttnRoute attention_route(int batch, int seq, int heads, int path, int cus) {
    if ((path & 0xff) == 3) return ATTN_TRACKED;
    if (attention_plan(seq, heads, cus).items_ps < cus * 2)
        return attn_narrow_items((long)batch * heads, seq, cus) ? ATTN_BY_128 : ATTN_BY_256;
    return seq > 512 ? ATTN_FLAGS : ATTN_TRACKED;
}

// ---- projections: C[rows, Nn] = A[rows, K] * W[Nn, K]^T, rows = all samples of the batch
// Output tiles of the matrix kernels: gemm_few.hip (any K pieces; fp32 and bf16) and gemm_mfma.hip (bf16).
enum TileId { FEW_64x64, FEW_128x64, FEW_128x128, FEW_192x128, FEW_256x128, FEW_192x192, FEW_TILE_KINDS,
              WIDE_256x256 = FEW_TILE_KINDS, WIDE_128x128, WIDE_192x256, WIDE_192x128, TILE_KINDS };
// Us of a round of workgroups, one tile each: fixed + stages of 64 k * stage.  per_cu = 2: two workgroups share a CU; `half`: a
// round that leaves at most one to each.  (Fitted to bf16, operands that change from call to call, 32 to 9000 rows x 1920 to 7680
// columns x K = 1920 and 7680, with loops that had branches in a stage: all tiles are 2 to 13 % faster now, in the same order.)
// gated: what an epilogue that reads and writes an fp32 residual adds to a round (17776 rows x 1920, K = 1920, then 184, 170,
// 164 and 168 us on the tiles of gemm_mfma.hip in their order below, now 184, 162, 160 and 170).
struct Tile { int bm, bn, per_cu; float half_fixed, half_stage, fixed, stage, gated; };
constexpr Tile kTiles[TILE_KINDS] = {
    {64, 64, 2, 3.0f, 0.235f, 4.5f, 0.40f, 1.9f},        // 8 waves of 16 x 32
    {128, 64, 1, 0.f, 0.f, 4.0f, 0.30f, 1.9f},           // 8 waves of 32 x 32
    {128, 128, 1, 0.f, 0.f, 6.0f, 0.47f, 3.8f},          // 8 waves of 32 x 64
    {192, 128, 1, 0.f, 0.f, 7.0f, 0.60f, 5.7f},          // 8 waves of 48 x 64
    {256, 128, 1, 0.f, 0.f, 8.7f, 0.76f, 7.5f},          // 8 waves of 64 x 64
    {192, 192, 1, 0.f, 0.f, 10.f, 0.90f, 7.5f},          // 8 waves of 48 x 96
    {256, 256, 1, 0.f, 0.f, 7.3f, 1.34f, 15.f},          // gemm_mfma.hip: 8 waves of 128 x 64
    {128, 128, 2, 2.0f, 0.80f, 4.0f, 0.92f, 7.5f},       // 4 waves of 64 x 64
    {192, 256, 1, 0.f, 0.f, 5.4f, 1.14f, 14.6f},         // 8 waves of 96 x 64
    {192, 128, 2, 4.2f, 0.88f, 6.0f, 1.34f, 13.f},       // 4 waves of 96 x 64
};
constexpr long tile_count(int id, long rows, int Nn) {
    return (rows + kTiles[id].bm - 1) / kTiles[id].bm * ((Nn + kTiles[id].bn - 1) / kTiles[id].bn);
}
// Estimated us of `wgs` workgroups of `stages` stages each on `cus` compute units (without what launching takes).
constexpr float tile_time(int id, long wgs, float stages, bool gated, int cus) {
    const Tile& t = kTiles[id];
    const long slots = (long)cus * t.per_cu, tail = wgs % slots;
    const float epi = gated ? t.gated : 0.f;
    // (gemm_few.hip over more than two rounds: the chip at its power limit, and its smaller wave tiles read more LDS per
    // product: 41728 rows, 1920 x 7680 on 256 x 128 tiles 1323 us, on 192 x 256 of gemm_mfma.hip 1229)
    const float many = id < FEW_TILE_KINDS && wgs > 2 * slots ? 1.15f : 1.f;
    const float full = many * (t.fixed + stages * t.stage) + epi;
    const float half = t.half_fixed + stages * t.half_stage + 0.5f * epi;
    float last = tail == 0 ? 0.f : full;
    if (t.per_cu == 2 && tail > 0) {                     // two per CU do not start a last round together
        const float share = (float)(tail <= cus ? tail : tail - cus) / cus;
        if (wgs < slots) last = tail <= cus ? half : 0.9f * full;
        else last = tail <= cus ? half * (0.5f + 0.5f * share) : half + (full - half) * share;
    }
    return (float)(wgs / slots) * full + last;
}
// The bf16 tile with the least estimated time: `pieces` workgroups per tile along K; [first, last]: the kinds to choose from.
// Inside the network, 28 token counts from 64 to 33976 x the four projections of a layer, those that are not cut into pieces, the
// one picked is 0.8 % slower than the fastest on average, and 6 % at most but for QKV and fc1 at 1024 tokens (128 x 128 of
// gemm_mfma.hip 41.0 and 39.6 us, 256 x 128 here 35.9 and 32.3).
constexpr int best_tile(int first, int last, long rows, int Nn, int K, int pieces, bool gated, int cus) {
    int best = first;
    float least = 0.f;
    for (int id = first; id <= last; ++id) {
        const float t = tile_time(id, tile_count(id, rows, Nn) * pieces, (float)(K / 64) / pieces, gated, cus);
        if (id == first || t < least) { best = id; least = t; }
    }
    return best;
}

// ---- bf16 projections on the tiles of gemm_mfma.hip
// How a sample's [tokens, Nn] output is spread over the chip: which tile, how many tiles run whole and how the rest is
// split along K.  A function of the sample's shape only (never of the batch): see gemm_mfma_kernel.
struct GemmPlan { int tile, tiles_m, tiles_n, full, tail, nsplit; size_t ws_bytes_per_sample; };

// the K split of the last partial round: pieces per tail tile (1: none)
constexpr int gemm_tail_split(long tiles, long slots, int K, bool allow_split) {
    const long tail = tiles % slots, nk = K / 64;
    if (!allow_split || K < 4096 || tail == 0) return 1;
    long ns = slots / tail;
    if (ns > 8) ns = 8;
    if (ns > nk / 2) ns = nk / 2;
    return ns >= 2 ? (int)ns : 1;
}

// pieces > 0: every tile is summed in that many K pieces (1: whole), which the caller has fixed for the sample's shape.
constexpr GemmPlan gemm_plan(int tokens, int Nn, int K, bool allow_split, int forced_variant, int pieces, int cus) {
    GemmPlan p{};
    const auto slots_of = [cus](int tile) { return (long)cus * kTiles[tile].per_cu; };
    if (forced_variant >= 1 && forced_variant <= 4) {
        p.tile = WIDE_256x256 + forced_variant - 1;
    } else {
        // (for the kind of epilogue that follows a long K, whichever the call's is: the plan belongs to the shape)
        p.tile = best_tile(0, TILE_KINDS - 1, tokens, Nn, K, 1, true, cus);
        float best = tile_time(p.tile, tile_count(p.tile, tokens, Nn), (float)(K / 64), true, cus);
        // The last partial round of a long K in pieces, which count as 1/pieces of a round plus a third of one for the
        // partial sums (two passes over tile-size fp32 per piece) and the second launch -- measured at 17776 tokens: worth
        // it with a long K (1920 x 7680: 0.62 -> 0.57 ms on 128 x 128 tiles), not with K = 1920 (0.188 -> 0.196 ms); 1920 x
        // 7680 at 13000 rows: 192 x 256 tiles in two rounds and 32 tiles of 8 pieces 351 us, 192 x 128 whole 332
        bool split = false;
        for (int id = WIDE_256x256; id < TILE_KINDS && pieces == 0; ++id) {
            const long tiles = tile_count(id, tokens, Nn), slots = slots_of(id);
            const int ns = gemm_tail_split(tiles, slots, K, allow_split);
            if (ns == 1 || tiles < slots) continue;
            const float t = tile_time(id, slots, (float)(K / 64), true, cus) * (tiles / slots + 1.0f / ns + 0.35f);
            if (t < best) { best = t; p.tile = id; split = true; }
        }
        allow_split = split;
    }
    const Tile& t = kTiles[p.tile];
    p.tiles_m = (tokens + t.bm - 1) / t.bm;
    p.tiles_n = (Nn + t.bn - 1) / t.bn;
    const int tiles = p.tiles_m * p.tiles_n;
    p.nsplit = pieces > 0 ? pieces : gemm_tail_split(tiles, slots_of(p.tile), K, allow_split);
    p.tail = p.nsplit == 1 ? 0 : pieces > 0 ? tiles : (int)(tiles % slots_of(p.tile));
    p.full = tiles - p.tail;
    p.ws_bytes_per_sample = (size_t)p.tail * p.nsplit * t.bm * t.bn * sizeof(float);
    return p;
}

// The stages of a tile of gemm_mfma.hip are compiled in forms, one per number of stages that are left behind them; the largest
// form is the steady state and serves every larger number.  strips: the tile requests its residual ahead, strip 0 with two
// stages left and strip 1 with one, so the form of two must be the third-last stage alone.  (With rings of two stages and the
// form of two as the steady state, strip 0 was read again in every stage, as many bytes as both operands.  1920 x 1920 gated on
// 128 x 128 tiles inside the network, us, so / now: 3400 tokens 53.3 / 36.4, 8400 102 / 72.6, 17000 211 / 147, 33976 424 / 297.)
constexpr int steady_form(int deep, bool strips) { return strips && deep < 3 ? 3 : deep; }
constexpr int strip_of_form(int form) { return form == 2 ? 0 : form == 1 ? 1 : -1; }

// Longest operand rows of the matrix kernels.  A load's offset inside a tile's rows is 32 bits: 256 rows at most, and 64 on the
// 64 x 64 tile of gemm_few.hip, which takes the rows that are longer than the others do.  (Bases of eight rows, which any
// tile could use, cost 0.4 to 1 % of every forward.  64 rows x 64 columns, K = 2^22 + 64 in bf16 2.4 ms, 480 on the FMA kernel.)
constexpr long ANY_TILE_ROW_BYTES = 1L << 23, TILE_64_ROW_BYTES = 1L << 26;

// ---- projections of few tokens and of fp32 operands (gemm_few.hip)
constexpr int FEW_ROW_BYTES = 128;                       // bytes of an operand row per stage: 64 bf16 or 32 fp32

// Whether `pieces` workgroups per tile are one round, a compute unit each, on some tile of gemm_few.hip.
constexpr int FEW_CUS = 256;                             // (a plan must not depend on the device's count)
constexpr bool few_one_round(long rows, int Nn, int pieces) {
    for (int id = 0; id < FEW_TILE_KINDS; ++id)
        if (tile_count(id, rows, Nn) * pieces <= FEW_CUS) return true;
    return false;
}
// K pieces of a sample of more than 128 tokens and a long K (bf16): 4 or 3, whichever is estimated faster, where that is one
// round; 3 on 192 x 192 tiles excepted.  1920 x 7680, weights from memory, us apart / one workgroup per tile: 450 tokens 27.6 /
// 36.1, 768 35.7 / 49.2, 800 39.0 / 42.6, 960 42.5 / 44.4, 1024 42.7 / 49.5, 1100 45.0 / 65, 1200 49.8 / 62, 1280 49.6 / 68.5.
// From 1281 tokens on (3 pieces, 192 x 192: 1400 53.2 / 68) a batch would lose more than that: its pieces stay on tiles of
// gemm_few.hip, four samples of 1500 168 us, on wider tiles whole 146.  (Up to there it loses little: a layer of one sample
// of 1104 / 1264 tokens, whole and in pieces, 212 -> 188 / 225 -> 201 us, of four 475 -> 478 / 557 -> 569, of six 722 -> 740
// / 761 -> 779; two layers of twelve of 1264 3150 -> 3340, of sixteen 4210 -> 4330.)
constexpr int few_long_pieces(int tokens, int Nn, int nk) {
    int best = 1;
    float least = 0.f;
    for (int n = 4; n >= 3; --n)
        for (int id = 0; id < (n == 4 ? (int)FEW_TILE_KINDS : (int)FEW_192x192); ++id) {
            const long wgs = tile_count(id, tokens, Nn) * n;
            if (wgs > FEW_CUS) continue;
            const float t = tile_time(id, wgs, (float)nk / n, false, FEW_CUS);
            if (best == 1 || t < least) { best = n; least = t; }
        }
    return best;
}

// A sample's plan: a function of the sample's shape alone, so that its result does not depend on the batch.  tiles_m x
// tiles_n tiles of 64 x 64.
//   bf16: up to 640 of them, 512 with K >= 4096, where a sample is cut into K pieces that wider tiles would also need, and
//     beyond as long as it is cut, or its operand rows are longer than wider tiles take.
//   fp32: every size (the matrix instructions bind, 32 cycles per 2048 operations, not the LDS reads).
// K pieces, short K: as many as bring the workgroups to 256 (one per compute unit), 8 at most (fp32 16) and each at least 5
// stages.  1920 x 1920 bf16 at 112 tokens (60 tiles), without / with the launch that adds them: 1 piece 10.3 us, 4 pieces
// 5.8 / 9.7, 8 pieces 6.2 / 11.1.
// Long K (60 stages and more), fp32 and up to 128 tokens: to 512.  1920 x 7680 bf16 at 112 tokens: 8 pieces (128 x 64
// tiles) 15.2, 4 pieces 16.1, 3 pieces 18.9.  More tokens: few_long_pieces().
// path: kernel path (low byte 1: generic kernels, 4: no K pieces).
struct FewPlan { bool use; int tiles_m, tiles_n, nsplit; };
constexpr FewPlan few_plan(bool bf16, int tokens, int Nn, int K, int path) {
    FewPlan p{false, 0, 0, 1};
    const long row_bytes = (long)K * (bf16 ? 2 : 4);
    if ((path & 0xff) == 1 || row_bytes % FEW_ROW_BYTES != 0 || row_bytes > TILE_64_ROW_BYTES || Nn % 4 != 0 || tokens < 1) return p;
    p.tiles_m = (tokens + 63) / 64;
    p.tiles_n = (Nn + 63) / 64;
    const long tiles = (long)p.tiles_m * p.tiles_n, nk = row_bytes / FEW_ROW_BYTES;
    if (bf16 && Nn < 64) return p;
    const long most = bf16 ? 8 : 16;
    long ns = (nk >= 60 ? 512 : 256) / tiles;
    if (bf16 && nk >= 60 && tokens > 128) ns = few_long_pieces(tokens, Nn, (int)nk);
    if ((path & 0xff) == 4) ns = 1;
    if (bf16 && ns <= 1 && tiles > (K >= 4096 ? 512 : 640) && row_bytes <= ANY_TILE_ROW_BYTES) return p;
    p.use = true;
    ns = ns < most ? ns : most;
    ns = ns < nk / 5 ? ns : nk / 5;
    p.nsplit = ns > 1 ? (int)ns : 1;
    return p;
}

// What runs a batch of samples of one plan.  It counts the tiles of the whole batch; the values are the same either way (same
// instruction, same order of k, pieces added in the same order, same epilogue).
//   FEW_PIECES  a workgroup per tile and K piece; the pieces pass through memory
//   FEW_INREG   a workgroup per tile, which adds its pieces in registers
//   FEW_TILES   the same, and where there is one piece (bf16) the tiles of gemm_mfma.hip are candidates too
// Pieces of their own pay until the tiles alone occupy the chip: with a short K up to 256 tiles of 64 x 64, with a long one as
// long as the pieces are one round; a single sample's always are (its plan counts the same tiles).  Layer with cold weights,
// us, pieces apart / in registers: 1920 x 1920 and the LayerNorm that adds the pieces, 112 tokens: 3 samples (180 tiles) 19.3 /
// 21.5, 4 (240) 23.1 / 22.0, 8 (480) 37.1 / 26.3; 1920 x 7680 in 8 pieces, 112 tokens: 4 samples 28.8 / 37.6, 5 32.4 / 42.7,
// 6 (no longer one round) 47.9 / 42.1, 8 55.0 / 49.4; in 4 pieces 1040 rows 43.2 / 58.7, 1200 62.2 / 61.2, 1350 68.0 / 63.7.
// fp32 is bound by the matrix instructions and takes finer pieces longer: 1920 x 7680 at 320 tokens, 4 samples (600 tiles)
// 358 / 393, 8 (1200) 674 / 654.
// The tiles of gemm_mfma.hip are never the fastest up to 768 tiles of 64 x 64 (5760 x 1920, 512 rows).
enum FewHow { FEW_PIECES, FEW_INREG, FEW_TILES };
constexpr FewHow few_how(bool bf16, const FewPlan& p, int batch, int tokens, int Nn, int K) {
    const long tiles = (long)batch * p.tiles_m * p.tiles_n;
    if (p.nsplit > 1 && (bf16 && K >= 60 * 64 ? few_one_round((long)batch * tokens, Nn, p.nsplit) : tiles < (bf16 ? 256 : 640)))
        return FEW_PIECES;
    return bf16 && tiles > 768 && p.tiles_m > 1 && K * 2L <= ANY_TILE_ROW_BYTES ? FEW_TILES : FEW_INREG;
}

// scratch for the K pieces, [piece][row][column] in fp32, of the largest batch up to `batch` whose pieces pass through memory
constexpr size_t few_workspace_bytes(bool bf16, const FewPlan& p, int batch, int tokens, int Nn, int K) {
    while (batch > 0 && few_how(bf16, p, batch, tokens, Nn, K) != FEW_PIECES) --batch;
    return (size_t)p.nsplit * batch * tokens * Nn * sizeof(float);
}

}  // namespace ps
