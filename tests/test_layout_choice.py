"""The choice of layout on the plan's host figures, compiled against the library's own header: no GPU takes part."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "common.h"

double gnn_plan_top_share(const gnn_plan *, int64_t) { return 0.5; }

// hot_lines block_lines min_degree: are there hot tables for fp32 rows of 100 columns on 1.8 M vertices, 26 M edges, half of them in long rows?
int main(int, char **argv) {
    gnn_plan p;
    p.n_rows = 1800000;
    p.n_edges = 26000000;
    p.params.n_thresholds = 2;
    p.params.thresholds[0] = 16;
    p.params.thresholds[1] = 256;
    p.n_bins = 3;
    p.bin_offsets[0] = 0;
    p.bin_offsets[1] = 1700000;
    p.bin_offsets[2] = 1785000;
    p.bin_offsets[3] = 1800000;
    p.bin_edges[0] = 6000000;
    p.bin_edges[1] = 7000000;
    p.bin_edges[2] = 13000000;
    p.bucket_vertices[3] = 1800000;
    p.bucket_edges[3] = 26000000;
    p.blocking.hot_lines = std::atoll(argv[1]);
    p.blocking.block_lines = std::atoll(argv[2]);
    p.blocking.min_degree = std::atoll(argv[3]);
    const bool blocks = gnn_call_blocks_expected(&p, 4, 100, GNN_WEIGHTS_NONE);
    const gnn_layout L = gnn_choose_layout(&p, p.n_rows, 100, 4, 100, true, 0, 0, true, false, blocks, false);
    std::printf("%d %d\n", int(L.hot_tables), int(L.padded_copy));
    return 0;
}
"""


@pytest.fixture(scope="module")
def choose(tmp_path_factory):
    folder = tmp_path_factory.mktemp("layout")
    source, binary = folder / "choose.cpp", folder / "choose"
    source.write_text(PROGRAM)
    subprocess.check_call([os.environ.get("CXX", "g++"), "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2104_06700_amd", "csrc"), str(source), "-o", str(binary)])
    return lambda *args: tuple(map(int, subprocess.check_output([str(binary), *map(str, args)], text=True).split()))


@pytest.mark.parametrize("hot_lines,block_lines,expected", [(0, 0, 1), (20000, 1000, 1), (65536, 65536, 1), (65537, 0, 0), (0, 65537, 0),
                                                           (100000, 100000, 0), (2 ** 31 - 1, 0, 0)])
def test_hot_tables_only_for_blocks_of_16_bit_indices(choose, hot_lines, block_lines, expected):
    """Their kernel tells the last block's pieces, which gather the caller's rows by vertex, by the 16-bit indices of the others: blocks
    too large for those leave every row where it lies."""
    assert choose(hot_lines, block_lines, 0) == (expected, 0)


def test_no_hot_tables_where_blocks_were_asked_for_by_degree(choose):
    assert choose(0, 0, 256)[0] == 0
