"""Graphs of so many short rows that wavefronts take up to 64 of them one after the other (run_kernel), against the oracle: rows
of 0 to 9 edges, a last wavefront that is not full, one pass over the columns and several, every layout of the gathered matrix."""
import numpy as np
import pytest
import torch

import oracle
import paper_2104_06700_amd as gnn
import synth
from helpers import OP_CODE, assert_close, device_graph, host_csr

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
N = 300007


def _graph(N=N):
    """Rows of 0 ... 9 edges (0 most often), 40 of 300 edges, hubs of 5,000 edges; sources with a bias to small ids, duplicates allowed."""
    v = torch.arange(N)
    lengths = (synth.mix64(v + 5) & 0x7FFFFFFF) % 16
    lengths = torch.where(lengths > 9, torch.zeros_like(lengths), lengths)
    lengths[11::7501] = 300
    lengths[77], lengths[N - 1] = 5000, 5000
    dst = v.repeat_interleave(lengths)
    r = synth.mix64(torch.arange(dst.numel()) + 99) & 0x7FFFFFFF
    src = torch.where(r % 3 == 0, (r // 3) % N, (r // 3) % 3000)
    key = torch.sort(dst * N + src).values
    return synth.EdgeList(n=N, src=(key % N).to(torch.int32), dst=(key // N).to(torch.int32), meta={})


@pytest.fixture(scope="module")
def graph():
    el = _graph()
    return el, host_csr(el)


@pytest.mark.parametrize("op_name,weights", [("mean", False), ("sage", False), ("sum", True), ("gcn", False)])
@pytest.mark.parametrize("f,dtype,shift", [(32, torch.float32, 0), (33, torch.float32, 1), (100, torch.float32, 0), (261, torch.float32, 0),
                                           (64, torch.bfloat16, 0), (129, torch.bfloat16, 1)])
def test_short_rows_served_many_per_wavefront(graph, f, dtype, shift, op_name, weights):
    el, (indptr, indices, indptr_t, indices_t, perm) = graph
    bf16 = dtype == torch.bfloat16
    din, dout = np.diff(indptr), np.diff(indptr_t)
    wts = (synth.uniform_features(el.e, 1, 7).reshape(-1) + 0.5) if weights else None
    w = None if wts is None else wts.numpy()
    X = synth.normal_features(N, f, 3, dtype=dtype)
    op = OP_CODE[op_name]
    Yo, S = oracle.aggregate_fwd(indptr, indices, X.float().numpy(), op=op, w=w, dout=dout, nthreads=8, want_scale=True)
    dXo, St = oracle.aggregate_bwd(indptr_t, indices_t, X.float().numpy(), op=op, wt=None if w is None else w[perm], din=din, nthreads=8,
                                   want_scale=True)
    flat = torch.full((N * f + shift,), float("nan"), dtype=dtype, device=DEV)
    Xd = flat[shift:].view(N, f)
    Xd.copy_(X)
    dg = device_graph(el, weights=wts, indptr64=f == 100)
    for what in ("as chosen", "copied", "rows of the copy whole", "blocked"):
        flags = {"copied": gnn.GNN_FLAG_FORCE_PADDED_COPY,
                 "rows of the copy whole": gnn.GNN_FLAG_FORCE_PADDED_COPY | gnn.GNN_FLAG_NO_SLICE_TABLES}.get(what, 0)
        if what == "blocked":  # the 300-edge rows as pieces, the others beside them
            flags = gnn.GNN_FLAG_FORCE_PADDED_COPY
            dg = device_graph(el, weights=wts, indptr64=f == 100)
            for p in (dg.plan_fwd, dg.plan_bwd):
                p.set_blocking(256, 4096, 4096, 96, 2)
            if weights:
                dg.plan_fwd.bind_edge_weights(dg.edge_w)
                dg.plan_bwd.bind_edge_weights(dg.edge_w_t)
        out = torch.full((2, N * f + shift), float("nan"), dtype=dtype, device=DEV)
        Y, dX = (o[shift:].view(N, f) for o in out)
        gnn.gnn_aggregate_fwd(dg.indptr, dg.indices, dg.edge_w, Xd, Y, N, f, op, plan=dg.plan_fwd, flags=flags)
        gnn.gnn_aggregate_bwd(dg.indptr_t, dg.indices_t, dg.edge_w_t, Xd, dX, N, f, op, plan=dg.plan_bwd, flags=flags)
        torch.cuda.synchronize()
        assert_close(Y, Yo, S, bf16, f"fwd {what}")
        assert_close(dX, dXo, St, bf16, f"bwd {what}")


@pytest.mark.parametrize("dtype,widths", [(torch.float32, (4, 5, 8, 12, 16, 29, 47)), (torch.bfloat16, (8, 10, 16, 32, 66))])
@pytest.mark.parametrize("weights", [False, True])
def test_small_graph_rows_of_few_lanes(dtype, widths, weights):
    """gather_kernel: rows of 1, 2, 4 and more lanes, slots without an edge, long rows shared by a workgroup; infinities stay in the
    rows and columns that have them (slots without an edge read zeros, lanes without columns nothing)."""
    n, bf16 = 900, dtype == torch.bfloat16
    lengths = torch.tensor([0, 1, 2, 3, 7, 8, 9, 31, 33, 64, 65, 300, 1500, 5000] + [6] * (n - 14))
    dst = torch.arange(n).repeat_interleave(lengths)
    src = (synth.mix64(torch.arange(dst.numel()) + 9) & 0x7FFFFFFF) % (n - 1)
    key = torch.sort(dst * n + src).values
    el = synth.EdgeList(n=n, src=(key % n).to(torch.int32), dst=(key // n).to(torch.int32), meta={})
    indptr, indices, *_ = host_csr(el)
    wts = (synth.uniform_features(el.e, 1, 7).reshape(-1).abs() + 0.5) if weights else None
    dg = device_graph(el, weights=wts)
    for f in widths:
        X = synth.normal_features(n, f, 3, dtype=dtype)
        Yo, S = oracle.aggregate_fwd(indptr, indices, X.float().numpy(), op=oracle.OP_SUM, w=None if wts is None else wts.numpy(), nthreads=8,
                                     want_scale=True)
        X[n - 1] = float("inf")  # nobody gathers it
        Y = torch.full((n, f), float("nan"), dtype=dtype, device=DEV)
        gnn.gnn_aggregate_fwd(dg.indptr, dg.indices, dg.edge_w, X.to(DEV), Y, n, f, gnn.GNN_SUM, plan=dg.plan_fwd)
        torch.cuda.synchronize()
        assert_close(Y, Yo, S, bf16, f"F={f}")
        X[n - 1], X[5, f - 1] = 0.0, float("inf")
        gnn.gnn_aggregate_fwd(dg.indptr, dg.indices, dg.edge_w, X.to(DEV), Y, n, f, gnn.GNN_SUM, plan=dg.plan_fwd)
        torch.cuda.synchronize()
        has = torch.zeros(n, dtype=torch.bool)
        has[el.dst[el.src == 5].long()] = True
        assert torch.equal(torch.isinf(Y[:, f - 1]).cpu(), has) and bool(torch.isfinite(Y[:, :f - 1]).all())


def test_last_segment_narrower_than_a_strip():
    """1025 columns gathered where they lie, 16 x 64 and one more: the strip of the last segment begins before its first column."""
    n, f = 50021, 1025
    lengths = (synth.mix64(torch.arange(n) + 5) & 0x7FFFFFFF) % 6
    lengths[7], lengths[n - 1] = 6000, 900
    dst = torch.arange(n).repeat_interleave(lengths)
    src = (synth.mix64(torch.arange(dst.numel()) + 9) & 0x7FFFFFFF) % n
    src[::50] = 0
    key = torch.sort(dst * n + src).values
    el = synth.EdgeList(n=n, src=(key % n).to(torch.int32), dst=(key // n).to(torch.int32), meta={})
    indptr, indices, *_ = host_csr(el)
    dg = device_graph(el)
    X = synth.normal_features(n, f, 3)
    Yo, S = oracle.aggregate_fwd(indptr, indices, X.numpy(), op=oracle.OP_SUM, nthreads=8, want_scale=True)
    Y = torch.full((n, f), float("nan"), device=DEV)
    gnn.gnn_aggregate_fwd(dg.indptr, dg.indices, None, X.to(DEV), Y, n, f, gnn.GNN_SUM, plan=dg.plan_fwd, flags=gnn.GNN_FLAG_NO_PADDED_COPY)
    torch.cuda.synchronize()
    assert_close(Y, Yo, S, False, "1025 columns")


@pytest.mark.parametrize("d,shift", [(33, 1), (100, 0), (261, 1)])
@pytest.mark.parametrize("reduce", [gnn.GNN_RED_MAX, gnn.GNN_RED_MIN])
def test_short_rows_of_max_and_min(graph, d, shift, reduce):
    """Values and winners of rows served many per wavefront, whole and in column slices, with ties, infinities and rows of nothing else."""
    el, (indptr, indices, *_) = graph
    dg, N = device_graph(el), el.n
    X = synth.normal_features(N, d, 3).mul_(2.0).round_()
    X[7, :] = float("-inf") if reduce == gnn.GNN_RED_MAX else float("inf")
    X[:3000:5, d - 1] = X[7, 0]
    flat = torch.full((N * d + shift,), float("nan"), device=DEV)
    Xd = flat[shift:].view(N, d)
    Xd.copy_(X)
    want, won = oracle.ap_fwd(indptr, indices, X.numpy(), None, d, oracle.BIN_COPY_LHS,
                              oracle.RED_MAX if reduce == gnn.GNN_RED_MAX else oracle.RED_MIN)
    for flags in (0, gnn.GNN_FLAG_FORCE_PADDED_COPY, gnn.GNN_FLAG_NO_COLUMN_SLICES):
        out = torch.full((N * d + shift,), float("nan"), device=DEV)
        arg = torch.full((N, d), -7, dtype=torch.int32, device=DEV)
        gnn.gnn_ap_fwd(dg.indptr, dg.indices, Xd, None, out[shift:].view(N, d), arg, N, d, gnn.GNN_BIN_COPY_LHS, reduce, plan=dg.plan_fwd, flags=flags)
        torch.cuda.synchronize()
        assert np.array_equal(out[shift:].view(N, d).cpu().numpy().astype(np.float64), want), flags
        assert np.array_equal(arg.cpu().numpy().astype(np.int64), won), flags


@pytest.fixture(scope="module")
def larger_graph():
    el = _graph(460007)
    return el, host_csr(el)


def test_sums_of_one_line_on_as_many_short_rows_as_they_need(larger_graph):
    """fp32 rows of one line go through run_kernel from 390,000 short rows on."""
    el, (indptr, indices, *_) = larger_graph
    dg = device_graph(el)
    X = synth.normal_features(el.n, 32, 3)
    Yo, S = oracle.aggregate_fwd(indptr, indices, X.numpy(), op=oracle.OP_SUM, nthreads=8, want_scale=True)
    Y = torch.full((el.n, 32), float("nan"), device=DEV)
    gnn.gnn_aggregate_fwd(dg.indptr, dg.indices, None, X.to(DEV), Y, el.n, 32, gnn.GNN_SUM, plan=dg.plan_fwd)
    torch.cuda.synchronize()
    assert_close(Y, Yo, S, False, "32 columns")


@pytest.mark.parametrize("d,shift", [(33, 1), (100, 0)])
@pytest.mark.parametrize("reduce", [gnn.GNN_RED_MAX, gnn.GNN_RED_MIN])
def test_max_and_min_of_as_many_short_rows_as_a_launch_of_their_own_takes(larger_graph, d, shift, reduce):
    """The same through ap_run_kernel, which takes 390,000 of them and more."""
    test_short_rows_of_max_and_min(larger_graph, d, shift, reduce)


@pytest.mark.parametrize("d", [68, 70, 72, 77, 80, 100, 132])  # a last line of 4, 6, 8, 13, 16 and 4 columns
@pytest.mark.parametrize("reducer", ["max", "min"])
def test_pooling_with_a_last_line_of_few_columns(d, reducer):
    """max / min from a copy whose last, short line is a table of its own: short rows, rows of every class and a hub row; the lowest position among equals."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(d)
    n = 600_000
    lens = torch.randint(0, 5, (n,), generator=gen, device=DEV)
    lens[:300] = torch.arange(300, device=DEV)
    lens[1000] = 9000
    dst = torch.repeat_interleave(torch.arange(n, device=DEV), lens)
    src = (dst * n + torch.randint(0, n, (dst.numel(),), generator=gen, device=DEV)).sort().values % n
    g = gnn.build_device_graph(dst.int(), src.int(), n)
    v = torch.randint(-4, 5, (n, d), generator=gen, device=DEV).float()  # ties
    v[7::50] = float("-inf") if reducer == "max" else float("inf")
    out = torch.full((n, d), float("nan"), device=DEV)
    arg = torch.full((n, d), -7, dtype=torch.int32, device=DEV)
    red = gnn.GNN_RED_MAX if reducer == "max" else gnn.GNN_RED_MIN
    gnn.gnn_ap_fwd(g.indptr, g.indices, v, None, out, arg, n, d, gnn.GNN_BIN_COPY_LHS, red, plan=g.plan_fwd, flags=gnn.GNN_FLAG_FORCE_PADDED_COPY)
    torch.cuda.synchronize()
    for c0 in range(0, d, 20):
        cols = slice(c0, min(c0 + 20, d))
        msgs = v[src][:, cols]
        to = dst[:, None].expand_as(msgs)
        want = torch.zeros_like(out[:, cols]).scatter_reduce(0, to, msgs, "amax" if reducer == "max" else "amin", include_self=False)
        pos = torch.arange(dst.numel(), device=DEV)[:, None].expand_as(msgs)
        first = torch.where(msgs == want[dst], pos, dst.numel())
        where = torch.full(want.shape, dst.numel(), device=DEV).scatter_reduce(0, to, first, "amin")
        where = torch.where(lens[:, None] > 0, where, -1)
        assert torch.equal(out[:, cols], want)
        assert torch.equal(arg[:, cols].long(), where)


def test_pooling_captured_with_room_for_one_table():
    """A captured call cannot make room: where the plan has it for rows of three lines, 68 columns take one table, not the two that need 400 bytes a row."""
    n, flags = 20_000, gnn.GNN_FLAG_FORCE_PADDED_COPY
    el = synth.rmat_directed(n, 400_000, (0.57, 0.19, 0.19, 0.05), 3, device=DEV)
    g, eager = gnn.build_device_graph(el.dst, el.src, n), gnn.build_device_graph(el.dst, el.src, n)
    gen = torch.Generator(device=DEV).manual_seed(1)
    x, v = torch.randn(n, 96, generator=gen, device=DEV), torch.randn(n, 68, generator=gen, device=DEV)

    def call(h, rows, out, arg):
        gnn.gnn_ap_fwd(h.indptr, h.indices, rows, None, out, arg, n, rows.shape[1], gnn.GNN_BIN_COPY_LHS, gnn.GNN_RED_MAX, plan=h.plan_fwd, flags=flags)

    call(g, x, torch.empty_like(x), torch.empty(x.shape, dtype=torch.int32, device=DEV))
    out, want = torch.empty_like(v), torch.empty_like(v)
    arg, want_arg = (torch.empty(v.shape, dtype=torch.int32, device=DEV) for _ in range(2))
    torch.cuda.synchronize()
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.stream(side), torch.cuda.graph(graph, stream=side):
        call(g, v, out, arg)
    for _ in range(3):
        v.normal_(generator=gen)
        graph.replay()
        torch.cuda.synchronize()
        call(eager, v, want, want_arg)
        assert torch.equal(out, want) and torch.equal(arg, want_arg)
