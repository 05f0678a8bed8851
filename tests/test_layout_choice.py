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

// hot_lines block_lines min_degree columns bytes-per-value long-edges: are there hot tables on 1.8 M vertices, 26 M edges?
// edges vertices: does a plan look at the order of the sources?
int main(int argc, char **argv) {
    if (argc == 3) {
        std::printf("%d\n", int(gnn_long_rows(std::atoll(argv[1]), std::atoll(argv[2]))));
        return 0;
    }
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
    p.bin_edges[1] = 20000000 - std::atoll(argv[6]);
    p.bin_edges[2] = std::atoll(argv[6]);
    p.bucket_vertices[3] = 1800000;
    p.bucket_edges[3] = 26000000;
    p.blocking.hot_lines = std::atoll(argv[1]);
    p.blocking.block_lines = std::atoll(argv[2]);
    p.blocking.min_degree = std::atoll(argv[3]);
    const int64_t F = std::atoll(argv[4]), esz = std::atoll(argv[5]);
    if (p.bin_edges[2] < 6500000) p.n_edges = 4 * p.bin_edges[2];  // a quarter in long rows is what makes blocks
    const bool blocks = gnn_call_blocks_expected(&p, int(esz), F, GNN_WEIGHTS_NONE);
    const gnn_layout L = gnn_choose_layout(&p, p.n_rows, F, int(esz), F, true, 0, 0, true, false, blocks, false);
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

    def run(hot_lines=0, block_lines=0, min_degree=0, f=100, esz=4, long_edges=13000000):
        args = (hot_lines, block_lines, min_degree, f, esz, long_edges)
        return tuple(map(int, subprocess.check_output([str(binary), *map(str, args)], text=True).split()))

    run.binary = str(binary)
    return run


@pytest.mark.parametrize("hot_lines,block_lines,expected", [(0, 0, 1), (20000, 1000, 1), (65536, 65536, 1), (65537, 0, 0), (0, 65537, 0),
                                                           (100000, 100000, 0), (2 ** 31 - 1, 0, 0)])
def test_hot_tables_only_for_blocks_of_16_bit_indices(choose, hot_lines, block_lines, expected):
    """Their kernel tells the last block's pieces, which gather the caller's rows by vertex, by the 16-bit indices of the others: blocks
    too large for those leave every row where it lies."""
    assert choose(hot_lines, block_lines) == (expected, 0)


def test_no_hot_tables_where_blocks_were_asked_for_by_degree(choose):
    assert choose(min_degree=256)[0] == 0


@pytest.mark.parametrize("f,esz,long_edges,expected", [
    (604, 4, 1890000, 0), (200, 4, 1890000, 0), (512, 4, 1890000, 0), (200, 4, 2420000, 0), (300, 4, 2420000, 1), (384, 4, 2420000, 0), (512, 4, 2420000, 1),
    (100, 4, 3070000, 1), (256, 4, 3260000, 1), (128, 4, 5650000, 0), (400, 2, 3260000, 0), (520, 2, 3260000, 1), (200, 2, 6480000, 1), (1024, 2, 2420000, 1)])
def test_hot_tables_only_where_the_long_rows_gather_enough(choose, f, esz, long_edges, expected):
    """Power-law graphs of 240,000 to 1,600,000 vertices, timed with and without: up to 1.3 times as long where the launches outweigh the lines."""
    assert choose(f=f, esz=esz, long_edges=long_edges)[0] == expected


@pytest.mark.parametrize("edges,vertices,expected", [(800000, 4000, 0), (1600000, 4000, 1), (12000000, 50000, 0), (23999999, 100000, 0), (24000000, 100000, 1),
                                                     (24000000, 160001, 0), (79000000, 500000, 1), (79000000, 132534, 1), (0, 1, 0)])
def test_order_of_the_sources_is_looked_at_only_where_a_rule_asks(choose, edges, vertices, expected):
    """The split of edge dot products asks for 400 edges a vertex, or for 150 and 24 M in all; for other graphs the launch would be for nothing."""
    assert int(subprocess.check_output([choose.binary, str(edges), str(vertices)], text=True)) == expected
