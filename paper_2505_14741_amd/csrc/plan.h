// Rules that say which thread or workgroup computes what: plain arithmetic on sizes, without device code, so that a host
// program can evaluate them at sizes no test can run.  (constexpr functions are callable from kernels as they are.)
#pragma once

namespace ps {

// ---- merge of attention's key pieces: 16 threads per query row, 16 rows per workgroup of 256
struct MergeRow { int item, row, d4; };              // split item (over all samples), its row, group of 4 outputs
// Counted in rows: a launch holds fewer than 2^32 threads, i.e. fewer than 2^28 rows, so a row index fits 32 bits where a
// thread index does not (524800 items of 256 rows are 2^31 + 2 * 10^6 threads).
constexpr MergeRow merge_row(int block, int thread, int bq) {
    const int rowid = block * 16 + (thread >> 4);
    return MergeRow{rowid / bq, rowid % bq, thread & 15};
}

}  // namespace ps
