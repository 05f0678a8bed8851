"""Long rows gathered from source tiles staged in LDS: the dense cells of the source-blocked layout.  The graphs
are dense enough that every block is staged; the cases put block and tile boundaries where they can go wrong (one
line more or less than a tile, a last short tile, rows cut into parts, lists filled up to whole units)."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2104_06700_amd as gnn
import synth
from helpers import OP_CODE, assert_close, device_graph, host_csr

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
SLICED = gnn.GNN_FLAG_FORCE_PADDED_COPY
THRESHOLDS = [4, 32, 256]


def _check(el, blocking, f, dtype, op_name, weights, bound, max_slices=8, expect_pieces=True):
    bf16 = dtype == torch.bfloat16
    indptr, indices, indptr_t, indices_t, perm = host_csr(el)
    din, dout = np.diff(indptr), np.diff(indptr_t)
    wts = (synth.uniform_features(el.e, 1, 7).reshape(-1) + 0.5) if weights else None
    w = None if wts is None else wts.numpy()
    dg = device_graph(el, weights=wts, plan_params=gnn.make_plan_params(THRESHOLDS, 64))
    for plan in (dg.plan_fwd, dg.plan_bwd):
        plan.set_blocking(**blocking)
    if bound:
        dg.plan_fwd.bind_edge_weights(dg.edge_w)
        dg.plan_bwd.bind_edge_weights(dg.edge_w_t)
    X = synth.normal_features(el.n, f, 3, dtype=dtype)
    Xd = X.to(DEV)
    op = OP_CODE[op_name]
    Yo, S = oracle.aggregate_fwd(indptr, indices, X.float().numpy(), op=op, w=w, dout=dout, nthreads=8, want_scale=True)
    dXo, St = oracle.aggregate_bwd(indptr_t, indices_t, X.float().numpy(), op=op, wt=None if w is None else w[perm], din=din,
                                   nthreads=8, want_scale=True)
    for _ in range(2):
        Y = torch.full((el.n, f), float("nan"), dtype=dtype, device=DEV)
        dX = torch.full((el.n, f), float("nan"), dtype=dtype, device=DEV)
        gnn.gnn_aggregate_fwd(dg.indptr, dg.indices, dg.edge_w, Xd, Y, el.n, f, op, plan=dg.plan_fwd, flags=SLICED, max_slices=max_slices)
        gnn.gnn_aggregate_bwd(dg.indptr_t, dg.indices_t, dg.edge_w_t, Xd, dX, el.n, f, op, plan=dg.plan_bwd, flags=SLICED,
                              max_slices=max_slices)
        torch.cuda.synchronize()
        assert_close(Y, Yo, S, bf16, "fwd")
        assert_close(dX, dXo, St, bf16, "bwd")
    assert (dg.plan_fwd.blocked_sizes()[2] > 0) == expect_pieces


@pytest.mark.parametrize("hot_lines,block_lines", [(990, 991), (991, 992), (992, 500), (1983, 2973), (5000, 300)])
@pytest.mark.parametrize("dtype,f,op_name,weights,bound", [
    (torch.float32, 64, "mean", False, False), (torch.float32, 300, "sage", False, False), (torch.float32, 65, "sum", True, True),
    (torch.float32, 100, "sum", True, False), (torch.bfloat16, 200, "gcn", False, False), (torch.bfloat16, 129, "mean", True, True)])
def test_staged_tiles_match_the_oracle(hot_lines, block_lines, dtype, f, op_name, weights, bound):
    el = synth.rmat_symmetric(5300, 1800000, (0.5, 0.2, 0.2, 0.1), 17)
    _check(el, dict(min_degree=32, hot_lines=hot_lines, block_lines=block_lines, max_piece=48, rest_min_count=0), f, dtype, op_name, weights, bound)


def test_rows_with_very_many_edges_into_one_tile_are_cut_into_parts():
    """More than 1,020 edges of one row into one tile do not fit the byte that counts a bundle's units."""
    el = synth.small_random_multigraph(400, 640000, 5)
    _check(el, dict(min_degree=32, hot_lines=320, block_lines=80, max_piece=48, rest_min_count=0), 96, torch.float32, "mean", False, False)


@pytest.mark.parametrize("f,dtype", [(3, torch.float32), (5, torch.float32), (8, torch.float32), (13, torch.float32), (16, torch.float32),
                                     (29, torch.float32), (9, torch.bfloat16), (25, torch.bfloat16), (64, torch.bfloat16)])
@pytest.mark.parametrize("op_name,weights,bound", [("mean", False, False), ("sage", False, False), ("sum", True, True), ("sum", True, False)])
def test_rows_of_at_most_one_line(f, dtype, op_name, weights, bound):
    """Tables of rows of 16 (no pieces), 32, 64 and 128 bytes: pieces, tiles and finalisation with 2, 4 and 8 lanes per line."""
    el = synth.rmat_symmetric(5300, 1800000, (0.5, 0.2, 0.2, 0.1), 17)
    row_bytes = f * (2 if dtype == torch.bfloat16 else 4)
    _check(el, dict(min_degree=32, hot_lines=1500, block_lines=1000, max_piece=48, rest_min_count=0), f, dtype, op_name, weights, bound,
           expect_pieces=row_bytes > 16)


def test_one_row_far_longer_than_the_others_is_cut_into_parts():
    n, hub = 6000, 5
    base = synth.erdos_renyi_directed(n, 900000, 3)
    keys = torch.cat([base.dst.long() * n + base.src.long(), hub * n + torch.arange(n)[torch.arange(n) != hub]]).unique()
    el = synth.EdgeList(n=n, src=(keys % n).to(torch.int32), dst=(keys // n).to(torch.int32), meta={})
    _check(el, dict(min_degree=32, hot_lines=2000, block_lines=4000, max_piece=96, rest_min_count=0), 72, torch.float32, "sum", False, False)


@pytest.mark.parametrize("f,dtype,bound", [(64, torch.float32, False), (64, torch.float32, True), (96, torch.bfloat16, False),
                                           (8, torch.float32, False), (16, torch.float32, True), (32, torch.bfloat16, True)])
def test_infinities_and_nan_reach_the_rows_that_gather_them_only(f, dtype, bound):
    """Lists are filled up with a line of zeros: rows must not see a neighbour's value, nor the lines beside it.  Column c
    holds one special value, in the vertex of a rank at the edges of blocks and tiles."""
    el = synth.rmat_symmetric(5300, 1800000, (0.5, 0.2, 0.2, 0.1), 17)
    wts = (synth.uniform_features(el.e, 1, 7).reshape(-1).abs() + 0.5) if bound else None  # positive: infinities keep their signs
    dg = device_graph(el, weights=wts, plan_params=gnn.make_plan_params(THRESHOLDS, 64))
    dg.plan_fwd.set_blocking(min_degree=32, hot_lines=992, block_lines=500, max_piece=48, rest_min_count=0)
    if bound:
        dg.plan_fwd.bind_edge_weights(dg.edge_w)
    x = synth.normal_features(el.n, f, 3, dtype=dtype).to(DEV)
    y = torch.empty_like(x)

    def call():
        gnn.gnn_aggregate_fwd(dg.indptr, dg.indices, dg.edge_w, x, y, el.n, f, gnn.GNN_SUM, plan=dg.plan_fwd,
                              flags=SLICED, max_slices=8)

    call()
    rank = dg.plan_fwd.export_blocked()[4]
    vertex = np.argsort(rank)
    edges = [0, 1, 495, 496, 990, 991, 992, 1242, 1491, 1492, 1991, 1992, 3000, 4491, 4492, 5298, 5299]
    values = [float("inf"), float("-inf"), float("nan")]
    want = torch.zeros(el.n, f, device=DEV)
    src, dst = el.src.to(DEV).long(), el.dst.to(DEV).long()
    for c in range(f):
        u, v = int(vertex[edges[c % len(edges)]]), values[c % 3]
        x[u, c] = v
        want[dst[src == u], c] = v
    call()
    torch.cuda.synchronize()
    special = ~torch.isfinite(want)
    assert int(special.sum()) > f and torch.equal(~torch.isfinite(y), special)
    assert torch.equal(torch.nan_to_num(y[special].float(), 1.0, 2.0, 3.0), torch.nan_to_num(want[special], 1.0, 2.0, 3.0))


@pytest.mark.parametrize("f,dtype,op_name", [(64, torch.float32, "sum"), (8, torch.float32, "sum"), (16, torch.float32, "sum"), (64, torch.bfloat16, "mean")])
@pytest.mark.parametrize("bound", [False, True])
def test_coefficients_follow_weights_that_change(f, dtype, op_name, bound):
    """Coefficients of tiles are filled in over and over, from the second time on through the positions kept for that: new weights in
    the same array and in another one, factors beside them (bf16 mean, backward), and a refill under capture, where no room for
    the positions can be had."""
    el = synth.rmat_symmetric(5300, 1800000, (0.5, 0.2, 0.2, 0.1), 17)
    indptr, indices, indptr_t, indices_t, perm = host_csr(el)
    backward = op_name == "mean"
    dg = device_graph(el, plan_params=gnn.make_plan_params(THRESHOLDS, 64))
    plan, ip, ix = (dg.plan_bwd, dg.indptr_t, dg.indices_t) if backward else (dg.plan_fwd, dg.indptr, dg.indices)
    plan.set_blocking(min_degree=32, hot_lines=992, block_lines=500, max_piece=48, rest_min_count=0)
    fn = gnn.gnn_aggregate_bwd if backward else gnn.gnn_aggregate_fwd
    x = synth.normal_features(el.n, f, 3, dtype=dtype)
    xd, y = x.to(DEV), torch.empty(el.n, f, dtype=dtype, device=DEV)
    weights = [synth.uniform_features(el.e, 1, seed).reshape(-1) + 0.5 for seed in range(4)]
    w = torch.empty(el.e, device=DEV)

    def call(array):
        fn(ip, ix, array, xd, y, el.n, f, OP_CODE[op_name], plan=plan, flags=SLICED, max_slices=8)

    def check(host, what):
        torch.cuda.synchronize()
        if backward:
            ref, S = oracle.aggregate_bwd(indptr_t, indices_t, x.float().numpy(), op=OP_CODE[op_name], wt=host.numpy(), din=np.diff(indptr),
                                          nthreads=8, want_scale=True)
        else:
            ref, S = oracle.aggregate_fwd(indptr, indices, x.float().numpy(), op=OP_CODE[op_name], w=host.numpy(), dout=np.diff(indptr_t),
                                          nthreads=8, want_scale=True)
        assert_close(y, ref, S, dtype == torch.bfloat16, what)

    def step(host):
        w.copy_(host)
        if bound:
            plan.bind_edge_weights(w)
        call(w)

    step(weights[0])
    check(weights[0], "first")
    if bound:  # the second filling, captured before there are positions
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            plan.bind_edge_weights(w)
            call(w)
        for host in weights[1:3]:
            w.copy_(host)
            y.fill_(float("nan"))
            graph.replay()
            check(host, "replay")
    for i, host in enumerate(weights[1:]):
        step(host)
        check(host, f"refill {i}")
        other = weights[i].to(DEV)
        call(other)  # unbound weights of another array between
        check(weights[i], f"other array {i}")
        call(w)
        check(host, f"refill {i}, after another array")


@pytest.mark.parametrize("n,rows,hot_lines", [(600, 512, 600), (1100, 700, 1099), (9500, 600, 9400)])
@pytest.mark.parametrize("f,op_name", [(96, "sum"), (100, "mean"), (131, "sage")])
def test_dense_cells_as_a_bit_matrix(n, rows, hot_lines, f, op_name):
    """Rows with a third of all sources: groups of 256 of them, the other rows and those with a repeated source as lists; sources that fill
    no chunk, and so many that a group is cut.  Columns of values whose parts are denormals and of values near the largest, against the oracle; infinities and
    NaN reach the rows that gather them only."""
    r = (synth.mix64(torch.arange(rows * n) + 7) & 0x7FFFFFFF) % 3 == 0
    key = r.nonzero().reshape(-1) // n * (n - rows + 1) % n * n + r.nonzero().reshape(-1) % n
    other = synth.mix64(torch.arange(4 * n) + 31) & 0x7FFFFFFFFFFF
    key = torch.cat([key.unique(), other % n * n + (other // n) % n]).unique()
    twice = key[(key // n == key[len(key) // 2] // n)][:3]
    key = torch.sort(torch.cat([key, twice])).values
    el = synth.EdgeList(n=n, src=(key % n).to(torch.int32), dst=(key // n).to(torch.int32), meta={})
    indptr, indices, indptr_t, *_ = host_csr(el)
    dg = device_graph(el, plan_params=gnn.make_plan_params(THRESHOLDS, 64))
    dg.plan_fwd.set_blocking(min_degree=32, hot_lines=hot_lines, block_lines=1000, max_piece=48, rest_min_count=0)
    X = synth.normal_features(n, f, 3)
    X[:, 5] *= 1e-36
    X[:, f - 1] *= 1e30
    X[11::97, 40] = 1e33
    op = OP_CODE[op_name]
    Yo, S = oracle.aggregate_fwd(indptr, indices, X.numpy(), op=op, dout=np.diff(indptr_t), nthreads=8, want_scale=True)
    Xd = X.to(DEV)
    Y = torch.full((n, f), float("nan"), device=DEV)

    def call():
        gnn.gnn_aggregate_fwd(dg.indptr, dg.indices, None, Xd, Y, n, f, op, plan=dg.plan_fwd, flags=SLICED, max_slices=8)
        torch.cuda.synchronize()

    call()
    assert dg.plan_fwd.bit_rows() >= 256
    assert_close(Y, Yo, S, False, op_name)
    specials = [float("inf"), float("-inf"), float("nan"), 1.5e38]  # the last one twice where a vertex is its own neighbour
    want = torch.zeros(n, f, device=DEV)
    src, dst = el.src.to(DEV).long(), el.dst.to(DEV).long()
    for i, u in enumerate([0, 1, n // 2, n - 2, n - 1, 127, 128, 511]):
        Xd[:, 7 + i] = 1.0
        Xd[u, 7 + i] = specials[i % 4]
        to = dst[src == u]
        want[to, 7 + i] = specials[i % 4]
        if op_name == "sage":
            want[u, 7 + i] = specials[i % 4]
    call()
    hit = want != 0
    for kind in (torch.isnan, torch.isposinf, torch.isneginf):  # one special source per column: its kind is the row's
        assert torch.equal(kind(Y), kind(want)), kind
    finite = hit & torch.isfinite(want)
    assert bool((Y[finite] > 1e33).all()) and bool((Y[:, 7:15][~hit[:, 7:15]].abs() < 1e6).all())


@pytest.mark.parametrize("first_f,first_weighted,f", [(128, False, 64), (128, True, 128)])
def test_a_captured_sum_takes_the_tiles_that_are_there(first_f, first_weighted, f):
    """After an eager call whose tiles are of the other kind (with a bit matrix, or lists only), a sum that would build its own is captured:
    it takes those, and every replay is right."""
    n, rows = 600, 512
    r = (synth.mix64(torch.arange(rows * n) + 7) & 0x7FFFFFFF) % 3 == 0
    key = torch.cat([r.nonzero().reshape(-1), torch.arange(n) * n + 5]).unique()
    el = synth.EdgeList(n=n, src=(key % n).to(torch.int32), dst=(key // n).to(torch.int32), meta={})
    indptr, indices, *_ = host_csr(el)
    dg = device_graph(el, plan_params=gnn.make_plan_params(THRESHOLDS, 64))
    dg.plan_fwd.set_blocking(min_degree=32, hot_lines=600, block_lines=1000, max_piece=48, rest_min_count=0)

    def call(x, y, w):
        gnn.gnn_aggregate_fwd(dg.indptr, dg.indices, w, x, y, n, x.shape[1], gnn.GNN_SUM, plan=dg.plan_fwd, flags=SLICED, max_slices=8)

    x0 = synth.normal_features(n, first_f, 2).to(DEV)
    call(x0, torch.empty_like(x0), torch.ones(len(key), device=DEV) if first_weighted else None)
    X = synth.normal_features(n, f, 3)
    xd, y = X.to(DEV), torch.empty(n, f, device=DEV)
    torch.cuda.synchronize()
    assert (dg.plan_fwd.bit_rows() == 0) == first_weighted
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(xd, y, None)
    assert (dg.plan_fwd.bit_rows() == 0) == first_weighted
    for rep in range(3):
        Yo, S = oracle.aggregate_fwd(indptr, indices, X.numpy(), op=OP_CODE["sum"], nthreads=8, want_scale=True)
        y.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert_close(y, Yo, S, False, f"replay {rep}")
        X = X * 0.75
        xd.copy_(X)
        call(x0, torch.empty_like(x0), None)  # eager work between


def _rows_with_a_third_of_all_sources(n, rows):
    r = (synth.mix64(torch.arange(rows * n) + 7) & 0x7FFFFFFF) % 3 == 0
    key = torch.cat([r.nonzero().reshape(-1), torch.arange(n) * n + 5]).unique()
    return synth.EdgeList(n=n, src=(key % n).to(torch.int32), dst=(key // n).to(torch.int32), meta={})


@pytest.mark.parametrize("first_f,first_weighted,f,later", [(128, True, 128, (128,)), (128, False, 64, (64, 512)), (64, False, 64, (128, 256))])
def test_a_graph_keeps_the_memory_it_recorded(first_f, first_weighted, f, later):
    """Calls that come after a capture and take more room (with tiles of their own, or wider) leave the graph its buffers: no plan that is
    built meanwhile is written into by a replay, and the replays stay right."""
    n = 9500
    el = _rows_with_a_third_of_all_sources(n, 600)
    indptr, indices, *_ = host_csr(el)
    dg = device_graph(el, plan_params=gnn.make_plan_params(THRESHOLDS, 64))
    dg.plan_fwd.set_blocking(min_degree=32, hot_lines=9400, block_lines=1000, max_piece=48, rest_min_count=0)

    def call(x, y, w=None):
        gnn.gnn_aggregate_fwd(dg.indptr, dg.indices, w, x, y, n, x.shape[1], gnn.GNN_SUM, plan=dg.plan_fwd, flags=SLICED, max_slices=8)

    x0 = synth.normal_features(n, first_f, 2).to(DEV)
    call(x0, torch.empty_like(x0), torch.ones(el.e, device=DEV) if first_weighted else None)
    X = synth.normal_features(n, f, 3)
    xd, y = X.to(DEV), torch.empty(n, f, device=DEV)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(xd, y)
    for width in later:
        x = synth.normal_features(n, width, 4).to(DEV)
        call(x, torch.empty_like(x))

    others, m = [], 4000  # the arrays of their plans fit free blocks of 0.1 to 10 MB
    while m < 500000:
        o = synth.erdos_renyi_directed(m, 4 * m, 5, device=DEV)
        g = gnn.build_device_graph(o.dst, o.src, m)
        v, out = torch.ones(m, 8, device=DEV), [torch.empty(m, 8, device=DEV) for _ in range(2)]
        gnn.gnn_aggregate_fwd(g.indptr, g.indices, None, v, out[0], m, 8, gnn.GNN_SUM, plan=g.plan_fwd)
        others.append((g, v, out, m, g.plan_fwd.export()))
        m = m * 7 // 5
    for rep in range(3):
        Yo, S = oracle.aggregate_fwd(indptr, indices, X.numpy(), op=OP_CODE["sum"], nthreads=8, want_scale=True)
        y.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert_close(y, Yo, S, False, f"replay {rep}")
        eager = torch.empty_like(y)
        call(xd, eager)
        assert_close(eager, Yo, S, False, f"eager {rep}")
        X = X * 0.75
        xd.copy_(X)
    for g, v, out, m, before in others:
        gnn.gnn_aggregate_fwd(g.indptr, g.indices, None, v, out[1], m, 8, gnn.GNN_SUM, plan=g.plan_fwd)
        torch.cuda.synchronize()
        assert torch.equal(out[0], out[1]), m
        assert all(np.array_equal(a, b) for a, b in zip(before, g.plan_fwd.export())), m


def test_a_refused_capture_does_not_decide_for_later_calls():
    """Nothing can be built in a capture: a call whose tiles are not there yet is refused, and the next eager call builds them."""
    n, f = 1100, 128
    el = _rows_with_a_third_of_all_sources(n, 600)
    indptr, indices, *_ = host_csr(el)
    dg = device_graph(el, plan_params=gnn.make_plan_params(THRESHOLDS, 64))
    dg.plan_fwd.set_blocking(min_degree=32, hot_lines=1099, block_lines=1000, max_piece=48, rest_min_count=0)
    X = synth.normal_features(n, f, 3)
    xd, y = X.to(DEV), torch.empty(n, f, device=DEV)

    def call(x, y, flags=0):
        gnn.gnn_aggregate_fwd(dg.indptr, dg.indices, None, x, y, n, x.shape[1], gnn.GNN_SUM, plan=dg.plan_fwd, flags=SLICED | flags, max_slices=8)

    call(xd, y, gnn.GNN_FLAG_NO_SOURCE_BLOCKS)      # all a call takes but pieces and tiles
    narrow = xd[:, :16].contiguous()
    call(narrow, torch.empty_like(narrow))          # pieces
    torch.cuda.synchronize()
    assert dg.plan_fwd.blocked_sizes()[2] > 0 and dg.plan_fwd.bit_rows() == 0
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        o = gnn.GnnOpts(stream=torch.cuda.current_stream().cuda_stream, plan=dg.plan_fwd.handle, flags=SLICED, max_slices=8)
        status = gnn.load_library().gnn_aggregate_fwd(dg.indptr.data_ptr(), dg.indices.data_ptr(), None, xd.data_ptr(), y.data_ptr(), n, f,
                                                      gnn.GNN_SUM, ctypes.byref(o))
    assert status == gnn.GNN_ERR_ALLOC
    call(xd, y)
    torch.cuda.synchronize()
    assert dg.plan_fwd.bit_rows() >= 256
    Yo, S = oracle.aggregate_fwd(indptr, indices, X.numpy(), op=OP_CODE["sum"], nthreads=8, want_scale=True)
    assert_close(y, Yo, S, False, "after the refused capture")


def test_a_captured_sum_without_room_for_the_bits_takes_the_lists():
    """The bit matrix is there, but its scratch for so many columns is not and cannot be had in a capture: the lists have room and serve
    the call, with the bits that a call with coefficients of one gets."""
    n, f = 9500, 256
    el = _rows_with_a_third_of_all_sources(n, 600)
    dg = device_graph(el, plan_params=gnn.make_plan_params(THRESHOLDS, 64))
    dg.plan_fwd.set_blocking(min_degree=32, hot_lines=9400, block_lines=1000, max_piece=48, rest_min_count=0)
    ones = torch.ones(el.e, device=DEV)

    def call(x, y, w=None):
        gnn.gnn_aggregate_fwd(dg.indptr, dg.indices, w, x, y, n, x.shape[1], gnn.GNN_SUM, plan=dg.plan_fwd, flags=SLICED, max_slices=8)

    x = synth.normal_features(n, f, 3).to(DEV)
    by_lists, by_bits, y = (torch.empty_like(x) for _ in range(3))
    narrow = x[:, :96].contiguous()
    call(x, by_lists, ones)
    call(narrow, torch.empty_like(narrow))
    assert dg.plan_fwd.bit_rows() >= 256
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(x, y)
    for _ in range(3):
        y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, by_lists)
        call(x, by_bits)  # eager: with the bit matrix
        torch.cuda.synchronize()
        assert not torch.equal(by_bits, by_lists) and torch.allclose(by_bits, by_lists, rtol=1e-4, atol=1e-3)


def _ms(fn, reps=5):
    times = []
    fn()
    for _ in range(reps):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        fn()
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b))
    return sorted(times)[reps // 2]


def test_a_packed_copy_in_memory_that_held_nan():
    """Columns behind the last one of a caller's packed copy, and the rows of vertices that nobody gathers, keep what its memory held: the
    bit matrix does not look at them, neither in the result nor in the time (a value that is not finite takes a way of its own)."""
    n, f = 9500, 602
    el = _rows_with_a_third_of_all_sources(n, 600)
    dg = device_graph(el, plan_params=gnn.make_plan_params(THRESHOLDS, 64))
    dg.plan_fwd.set_blocking(min_degree=32, hot_lines=9400, block_lines=1000, max_piece=48, rest_min_count=0)
    x = synth.normal_features(n, f, 3).to(DEV)
    buf = torch.empty(gnn.gnn_packed_bytes(n, f, gnn.GNN_F32) // 4, device=DEV)
    results, times = [], []
    for held in (0.0, float("nan"), 3e38):
        buf.fill_(held)
        gnn.gnn_pack_rows(dg.indptr, dg.indices, x, buf, n, f, gnn.GNN_SUM, False, plan=dg.plan_fwd)
        y = torch.full_like(x, float("nan"))

        def call():
            gnn.gnn_aggregate_packed(dg.indptr, dg.indices, None, buf, y, n, f, gnn.GNN_SUM, False, plan=dg.plan_fwd)

        times.append(_ms(call))
        results.append(y)
    assert dg.plan_fwd.bit_rows() >= 256
    assert torch.equal(results[0], results[1]) and torch.equal(results[0], results[2])
    assert max(times[1:]) < 1.5 * times[0], times


@pytest.mark.parametrize("n,rows,hot_lines", [(1100, 700, 1099), (9500, 600, 9400)])
def test_columns_of_values_that_the_products_leave_out(n, rows, hot_lines):
    """Infinities, NaN and values from 2^90 on, in one source and in all of them, against the oracle: the kind and the sign of what is not
    finite, the values of what is.  A whole column of them costs little."""
    el = _rows_with_a_third_of_all_sources(n, rows)
    indptr, indices, *_ = host_csr(el)
    dg = device_graph(el, plan_params=gnn.make_plan_params(THRESHOLDS, 64))
    dg.plan_fwd.set_blocking(min_degree=32, hot_lines=hot_lines, block_lines=1000, max_piece=48, rest_min_count=0)
    f, inf = 160, float("inf")
    X = synth.normal_features(n, f, 3)
    X[:, 0] = inf
    X[:, 33] = -inf
    X[::2, 34], X[1::2, 34] = inf, 1e30
    X[::3, 35], X[1::7, 35] = inf, -inf
    X[5, 36], X[70, 36] = inf, -inf
    X[::64, 37] = float("nan")
    X[:, 38] = float("nan")
    X[64:128, 39] = -inf
    X[3, 64] = float("nan")
    X[:, 65] *= 1e30
    X[:, 66] *= torch.ldexp(torch.ones(n), (torch.arange(n) * 29) % 60 + 60)
    X[1::2, 67] *= 1e33
    X[:64, 68] *= 1e33
    X[:, 69] = 2.0 ** 90
    X[:, 70] = -(2.0 ** 90 - 2.0 ** 66)
    X[9::10, 71], X[4::10, 72] = 1e35, inf
    X[:, 159] = inf
    with np.errstate(invalid="ignore"):
        Yo, S = oracle.aggregate_fwd(indptr, indices, X.numpy(), op=OP_CODE["sum"], nthreads=8, want_scale=True)
    xd, y = X.to(DEV), torch.full((n, f), float("nan"), device=DEV)

    def call():
        gnn.gnn_aggregate_fwd(dg.indptr, dg.indices, None, xd, y, n, f, gnn.GNN_SUM, plan=dg.plan_fwd, flags=SLICED, max_slices=8)

    call()
    torch.cuda.synchronize()
    assert dg.plan_fwd.bit_rows() >= 256
    got = y.cpu().numpy()
    for kind in (np.isnan, np.isposinf, np.isneginf):
        assert np.array_equal(kind(got), kind(Yo)), kind
    finite = np.isfinite(Yo).all(axis=0)
    assert finite.sum() > 140
    assert_close(y[:, torch.from_numpy(finite)], Yo[:, finite], S[:, finite], False, "finite columns")
    slow = _ms(call)
    xd.copy_(synth.normal_features(n, f, 3))
    assert slow < 5 * _ms(call)
