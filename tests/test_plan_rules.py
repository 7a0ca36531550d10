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
extern "C" int steady(int deep, int strips) { return ps::steady_form(deep, strips != 0); }
extern "C" int strip(int form) { return ps::strip_of_form(form); }
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


SHAPES = {"qkv": (5760, 1920, 0), "o": (1920, 1920, 1), "fc1": (7680, 1920, 0), "fc2": (1920, 7680, 1)}   # gated: o, fc2
# us of a projection on every kind of tile (0-5: gemm_few.hip, 6-9: gemm_mfma.hip), whole inside the network, and in K pieces
# (the kinds of gemm_few.hip, stand-alone with weights from memory)
MEASURED = [
    (112, "qkv", 1, [13.5, 18.1, 25.8, 28.9, 32.6, 36.7, 54.8, 32.6, 39.4, 36.6]),
    (200, "fc1", 1, [18.4, 15.7, 22.5, 25.8, 31.9, 33.6, 55.5, 32.0, 38.4, 33.2]),
    (448, "qkv", 1, [29.3, 29.9, 23.9, 29.3, 36.0, 38.4, 56.1, 33.0, 40.9, 35.9]),
    (640, "o", 1, [19.6, 17.1, 24.4, 26.5, 32.7, 34.9, 56.4, 33.8, 41.2, 36.6]),
    (800, "qkv", 1, [41.5, 41.9, 42.6, 30.1, 35.5, 38.8, 55.0, 34.4, 41.6, 36.5]),
    (800, "fc1", 1, [50.8, 50.3, 39.9, 48.1, 34.3, 35.5, 52.3, 34.2, 40.6, 42.4]),
    (1306, "o", 1, [27.5, 27.5, 22.1, 29.9, 33.2, 37.3, 56.0, 33.6, 42.1, 38.8]),
    (1306, "fc2", 1, [85.6, 81.6, 59.7, 86.0, 91.9, 104, 173, 106, 161, 119]),
    (1700, "fc1", 1, [88.8, 95.1, 78.6, 76.9, 65.8, 71.1, 55.4, 65.2, 77.5, 68.6]),
    (2048, "qkv", 1, [95.4, 91.8, 71.8, 61.1, 73.7, 76.0, 56.7, 62.7, 46.6, 50.0]),
    (2600, "o", 1, [39.8, 41.6, 39.8, 29.6, 34.3, 36.9, 56.2, 35.9, 42.7, 38.9]),
    (2600, "fc1", 1, [132, 132, 106, 99.3, 95.3, 99.6, 102, 91.6, 80.4, 82.8]),
    (3000, "qkv", 1, [115, 123, 103, 90.2, 106, 80.8, 98.5, 87.4, 82.0, 77.6]),
    (3600, "fc2", 1, [180, 178, 127, 158, 105, 106, 169, 112, 150, 139]),
    (4516, "o", 1, [66.0, 68.3, 60.7, 53.6, 65.8, 41.9, 57.6, 61.7, 45.5, 48.7]),
    (4516, "fc1", 1, [214, 217, 167, 148, 157, 137, 142, 142, 119, 124]),
    (4516, "fc2", 1, [224, 212, 184, 160, 199, 118, 177, 198, 152, 144]),
    (6000, "qkv", 1, [226, 230, 183, 171, 176, 156, 150, 147, 127, 129]),
    (8326, "o", 1, [118, 121, 94.1, 86.2, 77.5, 80.2, 110, 75.3, 93.3, 87.6]),
    (8326, "fc2", 1, [428, 378, 280, 258, 225, 227, 351, 236, 290, 254]),
    (9500, "fc1", 1, [442, 442, 331, 300, 287, 273, 242, 269, 240, 244]),
    (12000, "qkv", 1, [440, 448, 346, 324, 303, 297, 248, 262, 244, 250]),
    (12000, "fc2", 1, [630, 535, 401, 355, 340, 356, 372, 358, 320, 331]),
    (17776, "qkv", 1, [653, 643, 512, 472, 452, 422, 348, 387, 375, 362]),
    (17776, "o", 1, [258, 243, 200, 183, 190, 175, 185, 172, 169, 173]),
    (17776, "fc1", 1, [826, 810, 612, 551, 530, 512, 436, 487, 455, 451]),
    (24000, "fc2", 1, [1202, 1120, 847, 769, 783, 660, 624, 738, 663, 701]),
    (33976, "qkv", 1, [1302, 1337, 1043, 952, 898, 863, 660, 770, 728, 727]),
    (112, "fc2", 8, [16.9, 15.2, 18.4, 18.9, 20.4, 22.1]), (448, "fc2", 8, [46.4, 51.9, 37.6, 39.4, 28.8, 30.2]),
    (450, "fc2", 4, [39.0, 35.5, 27.6, 31.2, 36.1, 36.9]), (768, "fc2", 4, [55.7, 59.0, 51.8, 35.7, 39.2, 40.6]),
    (1040, "fc2", 4, [72.6, 76.8, 64.2, 59.1, 64.6, 43.2]), (1280, "fc2", 3, [84.2, 79.9, 63.4, 73.7, 49.6, 50.6])]


def test_tiles_are_about_the_fastest_measured(rules):
    few = C.c_int()
    total = rules.kinds(C.byref(few))
    lost = []
    for rows, name, pieces, us in MEASURED:
        n, k, gated = SHAPES[name]
        assert len(us) == (total if pieces == 1 else few.value)
        kind = rules.best(0, len(us) - 1, C.c_long(rows), n, k, pieces, gated if pieces == 1 else 0)
        lost.append(us[kind] / min(us))
        assert lost[-1] <= 1.07, (rows, name, kind)
    assert sum(lost) / len(lost) <= 1.01


def test_sizes_of_the_tile_tests_reach_every_tile(rules):
    from test_gpu_small_shapes import TILE_SIZES
    few = C.c_int()
    rules.kinds(C.byref(few))
    assert {rules.best(0, 9, C.c_long(rows), n, k, 1, 0) for rows, n, k in TILE_SIZES} >= set(range(few.value))


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


@pytest.mark.parametrize("deep", [2, 3])
def test_a_tile_requests_each_strip_of_its_residual_once(rules, deep):
    """Stage by stage as the tile's loop takes its forms: the steady one while more stages are left than its number, then the
    written-out ones.  Strip 0 in the third-last stage, strip 1 in the second-last, nothing in any other."""
    assert rules.steady(deep, 0) == deep
    steady = rules.steady(deep, 1)
    for stages in (3, 4, 5, 30, 120):
        strips = [rules.strip(min(left, steady)) for left in reversed(range(stages))]
        assert strips == [-1] * (stages - 3) + [0, 1, -1]


@pytest.mark.parametrize("bf16", [0, 1])
def test_operand_rows_of_any_length_stay_on_matrix_kernels(rules, bf16):
    """256 rows of more than 8 MB are beyond a load's 32-bit offset: the 64 x 64 tile takes them at every token count and batch, up
    to 64 MB each."""
    size = 2 if bf16 else 4
    for row in ((1 << 23) + 128, 1 << 25, 1 << 26):
        for tokens in (1, 64, 129, 1281, 5000, 33976):
            for n in (64, 68, 1920):
                assert rules.few(bf16, tokens, n, row // size, 0) > 0, (row, tokens, n)
                assert all(rules.how(bf16, tokens, n, row // size, b) != TILES for b in (1, 16))
    assert rules.few(bf16, 5000, 1920, (1 << 23) // size, 0) == (0 if bf16 else 1)
    assert rules.few(bf16, 64, 64, ((1 << 26) + 128) // size, 0) == 0


def spilled_registers():
    """Vector registers each kernel of the built library spills, from its metadata."""
    import re
    with open(build.LIB, "rb") as f:
        d = f.read()
    out = {}
    for m in re.finditer(rb"\.vgpr_spill_count([\x00-\x7f]|\xcc.|\xcd..)", d, re.S):
        at = d.rfind(b".symbol", 0, m.start())
        name = re.match(rb"\.symbol(?:[\xa0-\xbf]|\xd9.|\xda..)(\w+)\.kd", d[at:at + 600], re.S).group(1).decode()
        out[name] = m.group(1)[0] if len(m.group(1)) == 1 else int.from_bytes(m.group(1)[1:], "big")
    return out


def test_matrix_kernels_keep_their_registers():
    """Few-token tiles spill nothing, the wide ones a handful at most (256 x 256, outside the loop)."""
    if not os.path.exists(build.LIB):
        build.build_library()
    spilled = spilled_registers()
    few, wide = ({n: v for n, v in spilled.items() if k in n} for k in ("gemm_few_kernel", "gemm_mfma_kernel"))
    assert len(few) >= 60 and len(wide) >= 20
    assert not any(few.values()), {n: v for n, v in few.items() if v}
    assert max(wide.values()) <= 4
