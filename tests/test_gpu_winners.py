"""Vertex gradient of max / min by sorting the winners (large outputs), against sums in 64 bits."""
import pytest
import torch

import paper_2104_06700_amd as gnn

pytestmark = pytest.mark.gpu


def _winners(n, d, n_out, e, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    indices = torch.randint(0, n_out, (e,), device="cuda", dtype=torch.int32, generator=gen)
    arg = torch.randint(-1, e, (n, d), device="cuda", dtype=torch.int32, generator=gen)
    do = torch.empty(n, d, device="cuda").normal_(generator=gen)
    return indices, arg, do


def _check(dv, indices, arg, do, columns, factor=None):
    """factor(positions, column): what the winner multiplies its gradient by, in 64 bits."""
    for j in columns:
        won = arg[:, j] >= 0
        at = arg[won, j].long()
        g = do[won, j].double()
        if factor is not None:
            g = g * factor(at, j)
        u = indices[at].long()
        ref = torch.zeros(dv.shape[0], dtype=torch.float64, device="cuda").index_add_(0, u, g)
        mag = torch.zeros_like(ref).index_add_(0, u, g.abs())
        # at most a few thousand additions per sum, in any order, of products rounded once: well below 1e-5 of the magnitudes
        assert bool(((dv[:, j].double() - ref).abs() <= 1e-5 * mag).all()), f"column {j}"


@pytest.mark.parametrize("n,d", [(2200000, 64), (2449029, 54)])
def test_scratch_of_large_outputs_comes_from_the_pool(n, d):
    """Sizes at which a round of 14 or 16 quads would take arrays of more than a block of the pool: the call returns while
    work launched before it still runs."""
    n_out, e = 50000, 12 * n
    indices, arg, do = _winners(n, d, n_out, e, 5)
    dv = torch.full((n_out, d), float("nan"), device="cuda")

    def call():
        gnn.gnn_ap_bwd_vertex_arg(indices, arg, do, None, dv, n_out, n, d, gnn.GNN_BIN_COPY_LHS)

    call()  # the pool has the blocks from now on
    a = torch.randn(8192, 8192, device="cuda")
    b = torch.mm(a, a)
    torch.cuda.synchronize()
    done = torch.cuda.Event()
    for _ in range(20):  # some 0.2 s of work
        torch.mm(a, a, out=b)
    done.record()
    call()
    assert not done.query(), "the call waited for the device"
    torch.cuda.synchronize()
    _check(dv, indices, arg, do, (0, 1, d // 2, d - 1))


def test_cached_memory_is_bounded_and_given_back():
    """Scratch of the largest kind and a dropped plan beside it: no more than the documented bytes are held afterwards."""
    n, d, n_out = 2097152, 64, 50000  # arrays of exactly one block of the pool
    indices, arg, do = _winners(n, d, n_out, 12 * n, 6)
    dv = torch.empty(n_out, d, device="cuda")
    gnn.gnn_ap_bwd_vertex_arg(indices, arg, do, None, dv, n_out, n, d, gnn.GNN_BIN_COPY_LHS)
    dst, src = (torch.sort(torch.randint(0, n, (40000000,), device="cuda", dtype=torch.int32))[0] for _ in range(2))
    g = gnn.build_device_graph(dst, src, n)
    torch.cuda.synchronize()
    del g
    free = torch.cuda.mem_get_info()[0]
    gnn.gnn_release_cached_memory()
    held = torch.cuda.mem_get_info()[0] - free
    # of the scratch alone there are 1792 MiB; the driver counts in steps of 2 MiB, a few dozen of which small blocks round up to
    assert 1 << 30 < held <= gnn.GNN_CACHED_MEMORY_BYTES + (64 << 20)
    free = torch.cuda.mem_get_info()[0]
    gnn.gnn_release_cached_memory()
    assert torch.cuda.mem_get_info()[0] == free


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("binop", [gnn.GNN_BIN_MUL, gnn.GNN_BIN_DIV])
def test_sorted_gradient_with_edge_operands_behind_an_edge_id_map(binop, wide):
    n, d, n_out = 140001, 33, 150000
    e = 16 * n
    indices, arg, do = _winners(n, d, n_out, e, 7)
    ids = torch.randperm(e, device="cuda")
    fe = torch.rand((e, d) if wide else (e,), device="cuda") + 0.5
    dv = torch.full((n_out, d), float("nan"), device="cuda")
    gnn.gnn_ap_bwd_vertex_arg(indices, arg, do, fe, dv, n_out, n, d, binop, edge_ids=ids)
    torch.cuda.synchronize()

    def factor(at, j):
        y = (fe[ids[at], j] if wide else fe[ids[at]]).double()
        return y if binop == gnn.GNN_BIN_MUL else 1.0 / y

    _check(dv, indices, arg, do, (0, 3, 4, 31, 32), factor)


def test_infinities_and_nan_reach_their_winners_only():
    n, d, n_out = 140000, 32, 9000
    indices, arg, do = _winners(n, d, n_out, 16 * n, 8)
    indices[: 8 * n] = 77  # a range that is cut into pieces
    for j, x in enumerate((float("inf"), float("-inf"), float("nan"))):
        do[5 + j, j] = x
        arg[5 + j, j] = 9 * n + j
        do[50 + j, 8 + j] = x
        arg[50 + j, 8 + j] = j
    dv = torch.zeros(n_out, d, device="cuda")
    gnn.gnn_ap_bwd_vertex_arg(indices, arg, do, None, dv, n_out, n, d, gnn.GNN_BIN_COPY_LHS)
    want = torch.zeros(n_out, d, device="cuda")
    for j, x in enumerate((float("inf"), float("-inf"), float("nan"))):
        want[indices[9 * n + j], j] = x
        want[77, 8 + j] = x
    special = ~torch.isfinite(want)
    assert torch.equal(~torch.isfinite(dv), special)
    assert torch.equal(torch.nan_to_num(dv[special], 1.0, 2.0, 3.0), torch.nan_to_num(want[special], 1.0, 2.0, 3.0))


def test_a_captured_call_adds_with_atomics():
    """The sorted form takes scratch, which a captured call cannot; every replay gives the sums of the eager call."""
    n, d, n_out = 140000, 32, 9000
    indices, arg, do = _winners(n, d, n_out, 16 * n, 9)
    dv = torch.full((n_out, d), float("nan"), device="cuda")
    gnn.gnn_ap_bwd_vertex_arg(indices, arg, do, None, dv, n_out, n, d, gnn.GNN_BIN_COPY_LHS)
    _check(dv, indices, arg, do, range(d))
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        gnn.gnn_ap_bwd_vertex_arg(indices, arg, do, None, dv, n_out, n, d, gnn.GNN_BIN_COPY_LHS)
    for _ in range(3):
        dv.fill_(float("nan"))
        do.mul_(-0.5)
        graph.replay()
        torch.cuda.synchronize()
        _check(dv, indices, arg, do, range(d))


@pytest.mark.parametrize("n", [600001, 598016])  # a row beyond whole tiles of 4096, and whole ones
@pytest.mark.parametrize("empty", ["none", "some", "a whole part", "all but one"])
def test_rows_without_winners_are_left_out(n, empty):
    d, n_out, e = 64, 70000, 12 * 600001
    indices, arg, do = _winners(n, d, n_out, e, 9)
    gone = torch.zeros(n, dtype=torch.bool, device="cuda")
    if empty == "some":
        gone = torch.rand(n, device="cuda", generator=torch.Generator(device="cuda").manual_seed(2)) < 0.45
        gone[:130] = True  # two whole workgroups' rows and the next one's first
        gone[-1] = True
    elif empty == "a whole part":
        gone[40960:200000] = True
    elif empty == "all but one":
        gone[:] = True
        gone[n - 1] = False
    arg[gone] = -1
    do[gone] = float("nan")  # nothing of such a row counts
    dv = torch.full((n_out, d), float("nan"), device="cuda")
    gnn.gnn_ap_bwd_vertex_arg(indices, arg, do, None, dv, n_out, n, d, gnn.GNN_BIN_COPY_LHS)
    _check(dv, indices, arg, do, (0, 3, 31, d - 1))
