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
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, lib = os.path.join(d, "rules.cpp"), os.path.join(d, "rules.so")
    with open(src, "w") as f:
        f.write(WRAPPERS)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", build.CSRC, src, "-o", lib], check=True)
    return C.CDLL(lib)


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
