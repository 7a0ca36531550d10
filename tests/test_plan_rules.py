"""Rules that say which thread or workgroup computes what (csrc/plan.h), evaluated on the CPU at sizes no GPU test can run."""
import ctypes as C
import os
import subprocess

import pytest

from paper_2505_14741_amd import build

WRAPPERS = """
#include "plan.h"
extern "C" void merge(int block, int thread, int bq, int* out) {
    const ps::MergeRow r = ps::merge_row(block, thread, bq);
    out[0] = r.item; out[1] = r.row; out[2] = r.d4;
}
extern "C" int few(int bf16, int tokens, int n, int k, int path) {   // 0: another kernel, else the number of K pieces
    const ps::FewPlan p = ps::few_plan(bf16 != 0, tokens, n, k, path);
    return p.use ? p.nsplit : 0;
}
extern "C" int how(int bf16, int tokens, int n, int k, int batch) {
    return ps::few_how(bf16 != 0, ps::few_plan(bf16 != 0, tokens, n, k, 0), batch, tokens, n, k);
}
extern "C" int best(int first, int last, long rows, int n, int k, int pieces, int gated) {
    return ps::best_tile(first, last, rows, n, k, pieces, gated != 0, 256);
}
extern "C" void wide(int tokens, int n, int k, int* out) {
    const ps::GemmPlan p = ps::gemm_plan(tokens, n, k, true, 0, 0, 256);
    out[0] = p.tile; out[1] = p.full; out[2] = p.tail; out[3] = p.nsplit;
}
extern "C" int narrow(long bh, int seq) { return ps::attn_narrow_items(bh, seq, 256); }
extern "C" int route(int batch, int seq, int heads, int path) { return ps::attention_route(batch, seq, heads, path, 256); }
extern "C" int kinds(int* few) { *few = ps::FEW_TILE_KINDS; return ps::TILE_KINDS; }
extern "C" long scratch(int bf16, int tokens, int n, int k, int batch) {
    return (long)ps::few_workspace_bytes(bf16 != 0, ps::few_plan(bf16 != 0, tokens, n, k, 0), batch, tokens, n, k);
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, lib = os.path.join(d, "rules.cpp"), os.path.join(d, "rules.so")
    with open(src, "w") as f:
        f.write(WRAPPERS)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", build.CSRC, src, "-o", lib], check=True)
    lib = C.CDLL(lib)
    lib.scratch.restype = C.c_long
    return lib


@pytest.mark.parametrize("nitems", [1, 28, 524800, 1 << 20])
def test_merge_rows_of_many_items(rules, nitems):
    """16 threads per row of 256-row items.  524800 items are more than 2^31 threads, 2^20 items the 2^32 a launch can hold."""
    out = (C.c_int * 3)()
    blocks = nitems * 16
    for block in {0, 1, blocks // 2, min(blocks, (1 << 31) // 256) - 1, min(blocks - 1, (1 << 31) // 256), blocks - 1}:
        for thread in (0, 15, 16, 255):
            rules.merge(block, thread, 256, out)
            gid = block * 256 + thread
            assert list(out) == [gid // 16 // 256, gid // 16 % 256, gid % 16] and 0 <= out[0] < nitems


def test_few_token_projections_end_where_wider_tiles_are_faster(rules):
    few = lambda *a: rules.few(1, *a, 0)
    # K = 1920: 640 tiles of 64 x 64; long K: as long as pieces are one round of workgroups
    assert few(1344, 1920, 1920) == 1 and few(1345, 1920, 1920) == 0
    assert few(1088, 1920, 7680) > 1 and few(1280, 1920, 7680) > 1 and few(1281, 1920, 7680) == 0
    assert few(112, 1920, 7680) == 8 and few(112, 1920, 1920) == 4 and few(112, 5760, 1920) == 1
    assert few(1344, 1920, 4032) == 1 and few(1344, 1920, 4096) == 0     # where 128-wide tiles start to be cut
    assert rules.few(0, 4096, 1920, 7680, 0) == 1                        # fp32: every size
    assert rules.few(1, 112, 1920, 1920, 4) == 1 and rules.few(1, 112, 1920, 1920, 1) == 0
    assert few(112, 1922, 1920) == 0 and few(112, 1920, 1928) == 0 and few(112, 62, 1920) == 0


PIECES, INREG, TILES = 0, 1, 2


def test_a_batch_that_fills_the_chip_takes_wide_tiles_and_no_pieces_of_its_own(rules):
    how = lambda *a: rules.how(1, *a)
    assert how(112, 1920, 1920, 1) == PIECES and how(112, 1920, 1920, 4) == PIECES      # 60 tiles, 240
    assert how(112, 1920, 1920, 8) == INREG and how(112, 1920, 1920, 16) == TILES       # 480, 960
    assert how(112, 1920, 7680, 5) == PIECES and how(112, 1920, 7680, 6) == INREG       # 192 x 192 x 8 pieces: 240, 320
    assert how(256, 7680, 1920, 1) == INREG and how(256, 7680, 1920, 8) == TILES
    assert how(1300, 1920, 1920, 1) == INREG and how(1300, 1920, 1920, 2) == TILES      # 630, 1260
    assert how(64, 7680, 1920, 16) == INREG                                             # a 128-row tile would be half empty
    assert rules.how(0, 112, 1920, 7680, 8) == PIECES and rules.how(0, 320, 1920, 7680, 16) == INREG   # fp32: one kernel


@pytest.mark.parametrize("bf16", [0, 1])
def test_pieces_that_are_planned_are_spread(rules, bf16):
    """A single sample's K pieces are workgroups of their own, with scratch to pass them: a tile that walks all of K has no use
    for pieces, and a call without scratch would be summed in another order."""
    for tokens in (*range(1, 2000, 13), 64, 128, 129, 768, 769, 960, 961, 1024, 1088, 1089, 1152, 1153, 1280, 1281):
        for n, k in ((64, 4096), (196, 1984), (1024, 4096), (1536, 6144), (1920, 1920), (1920, 7680), (2048, 8192), (7680, 3840)):
            pieces = rules.few(bf16, tokens, n, k, 0)
            if pieces > 1:
                assert rules.how(bf16, tokens, n, k, 1) == PIECES, (tokens, n, k)
                assert rules.scratch(bf16, tokens, n, k, 1) == 4 * pieces * tokens * n


@pytest.mark.parametrize("bf16", [0, 1])
def test_scratch_of_few_token_projections_serves_every_smaller_batch(rules, bf16):
    """A workspace sized for a batch is used for smaller ones (the last cycle of a step-batched run), and a batch whose pieces
    stay in registers needs no more than the largest one whose pieces do not."""
    for tokens in (1, 32, 64, 65, 112, 256, 520, 1040, 1200, 1300):
        for n, k in ((64, 1920), (1920, 1920), (5760, 1920), (7680, 1920), (1920, 7680), (196, 1984)):
            pieces = rules.few(bf16, tokens, n, k, 0)
            size = [rules.scratch(bf16, tokens, n, k, b) for b in range(1, 17)]
            assert size == sorted(size)
            for b in range(1, 17):
                if pieces > 1 and rules.how(bf16, tokens, n, k, b) == PIECES:
                    assert size[b - 1] >= 4 * pieces * b * tokens * n
                assert size[b - 1] <= 4 * max(pieces, 1) * tokens * n * b


def test_sizes_of_the_batch_tests_split_where_they_say_so(rules):
    from test_gpu_dit_sampler import SPLIT_GRIDS
    plan = lambda tokens: (rules.wide(tokens, 1920, 7680, out), list(out))[1]
    out = (C.c_int * 4)()
    tails = [plan(text + f * r * c) for f, r, c, text in SPLIT_GRIDS]
    assert [t[2:] for t in tails] == [[64, 4], [8, 8]] and all(t[1] % 256 == 0 for t in tails)
    assert plan(17776)[2] > 0 and plan(17776)[3] > 1     # the 30-layer run
    assert plan(4516)[2:] == [0, 1]                      # the block


FASTEST = [  # rows, columns, K, pieces (1920 columns: with the gated residual update): kinds within 6 % of the fastest measured one (0-5: gemm_few.hip, 6-9: gemm_mfma.hip)
    (112, 5760, 1920, 1, [0]), (224, 7680, 1920, 1, [1]), (448, 5760, 1920, 1, [2]), (640, 7680, 1920, 1, [3]),
    (1306, 5760, 1920, 1, [7]), (2048, 5760, 1920, 1, [9, 8]), (2600, 5760, 1920, 1, [6]), (4516, 7680, 1920, 1, [9, 8]),
    (17776, 5760, 1920, 1, [6]), (17776, 1920, 1920, 1, [8]), (33976, 1920, 1920, 1, [9, 7]), (8326, 1920, 1920, 1, [7]),
    (3600, 1920, 7680, 1, [4, 5]), (4516, 1920, 7680, 1, [5]),
    (112, 1920, 7680, 8, [1]), (448, 1920, 7680, 4, [2]), (768, 1920, 7680, 4, [3])]


@pytest.mark.parametrize("rows,n,k,pieces,kinds", FASTEST)
def test_tiles_are_the_fastest_measured(rules, rows, n, k, pieces, kinds):
    few = C.c_int()
    total = rules.kinds(C.byref(few))
    assert (few.value, total) == (6, 10)
    assert rules.best(0, (few.value if pieces > 1 else total) - 1, C.c_long(rows), n, k, pieces, n == 1920 and pieces == 1) in kinds


def test_sizes_of_the_tile_tests_take_the_tiles_they_name(rules):
    from test_gpu_small_shapes import TILE_SIZES
    for kind, rows, n, k in TILE_SIZES:
        assert rules.best(0, 9, C.c_long(rows), n, k, 1, 0) == kind


def test_attention_workgroups_of_128_queries_where_they_are_faster(rules):
    """(batch, head) pairs and keys on both sides, as measured; 16 samples of 16 heads and 1000 keys are what the test of
    overflowing queries takes to the wider kernel."""
    narrow = lambda bh, n: rules.narrow(C.c_long(bh), n)
    assert narrow(30, 112) and narrow(60, 1000) and narrow(30, 2000) and narrow(30, 2608) and narrow(4, 4200) and narrow(240, 520)
    assert not narrow(30, 3600) and not narrow(240, 1000) and not narrow(256, 1000)
    assert narrow(16, 1000) and narrow(256, 31) and narrow(256, 129)
    assert not narrow(16, 4200) and not narrow(16, 6000) and not narrow(8, 12000) and not narrow(4, 17776)
    assert narrow(8, 4200) and narrow(4, 6000) and narrow(4, 12000) and narrow(128, 700)


def test_sizes_of_the_attention_tests_take_the_kernels_they_name(rules):
    from test_gpu_kernels import BY_256, FLAGS, ROUTE_SIZES, TRACKED
    BY_128 = 0
    for route, batch, keys, heads in ROUTE_SIZES:
        assert rules.route(batch, keys, heads, 0) == route, (batch, keys, heads)
        assert rules.route(batch, keys, heads, 3) == TRACKED
    assert rules.route(16, 1000, 16, 0) == BY_256 and rules.route(1, 700, 200, 0) == FLAGS and rules.route(2, 513, 200, 0) == FLAGS
    assert rules.route(1, 4516, 30, 0) == FLAGS and rules.route(1, 17776, 30, 0) == FLAGS
    for batch, keys, heads in ((1, 700, 2), (3, 700, 3), (2, 1000, 3), (2, 1, 3), (2, 4096, 4), (1, 1000, 16)):
        assert rules.route(batch, keys, heads, 0) == BY_128, (batch, keys, heads)
    # samples of fewer than 512 items of 256 queries never take the last two, whatever the batch
    for heads in (1, 30, 200, 255):
        for keys in (1, 64, 300, 512, 513, 2000, 17776):
            small = heads * -(-keys // 256) < 512
            assert all((rules.route(b, keys, heads, 0) < FLAGS) == small for b in (1, 2, 16, 1024))
