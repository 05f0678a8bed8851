"""Graphs of few edges per vertex whose long rows gather the most-gathered sources from tables and everything else in place, against the call
that stays in place."""
import pytest
import torch

import paper_2104_06700_amd as gnn
import synth

pytestmark = pytest.mark.gpu

F32, BF16 = torch.float32, torch.bfloat16
STRONG = (0.57, 0.19, 0.19, 0.05)
IN_PLACE = gnn.GNN_FLAG_NO_SOURCE_BLOCKS
_graphs = {}


def _graph(n, e, weights=False, indptr64=False):
    key = (n, e, weights, indptr64)
    if key not in _graphs:
        _graphs.clear()
        el = synth.rmat_directed(n, e, STRONG, 17, device="cuda")
        w = torch.rand(e, device="cuda") + 0.5 if weights else None
        g = gnn.build_device_graph(el.dst, el.src, n, edge_w=w, indptr64=indptr64)
        if weights:
            g.plan_fwd.bind_edge_weights(g.edge_w)
            g.plan_bwd.bind_edge_weights(g.edge_w_t)
        _graphs[key] = g
    return _graphs[key]


def _call(g, x, op, backward, flags=0, out=None, stream=None):
    n, f = x.shape
    y = torch.full((n, f), float("nan"), device="cuda", dtype=x.dtype) if out is None else out
    if backward:
        gnn.gnn_aggregate_bwd(g.indptr_t, g.indices_t, g.edge_w_t, x, y, n, f, op, plan=g.plan_bwd, flags=flags)
    else:
        gnn.gnn_aggregate_fwd(g.indptr, g.indices, g.edge_w, x, y, n, f, op, plan=g.plan_fwd, flags=flags)
    return y


def _bound(g, x, op, backward):
    # fp32 sums in two orders; a bf16 result is rounded once more on either side, to 2^-9 of the value
    return (2.0 ** -8 if x.dtype == BF16 else 1e-5) * _call(g, x.abs(), op, backward, IN_PLACE).double()


# whole lines, a last line of one strip, rows off line boundaries, rows of one line and a bit, two launches of slices; every factor, the own row
FORMS = [(F32, 256, gnn.GNN_MEAN, False), (F32, 256, gnn.GNN_MEAN, True), (F32, 36, gnn.GNN_SUM, False), (F32, 100, gnn.GNN_SAGE_GCN, True),
         (F32, 100, gnn.GNN_SAGE_GCN, False), (F32, 292, gnn.GNN_GCN_SYM, False), (F32, 604, gnn.GNN_MEAN, False), (BF16, 128, gnn.GNN_MEAN, False),
         (BF16, 72, gnn.GNN_MEAN, True), (BF16, 200, gnn.GNN_SAGE_GCN, False), (BF16, 264, gnn.GNN_GCN_SYM, True)]


@pytest.mark.parametrize("dtype,f,op,backward", FORMS)
def test_agrees_with_the_call_in_place(dtype, f, op, backward):
    g = _graph(1800000, 26000000)
    x = torch.randn(g.n, f, device="cuda").to(dtype)
    y = _call(g, x, op, backward)
    plan = g.plan_bwd if backward else g.plan_fwd
    assert plan.blocked_sizes()[2] > 0  # it went over hot tables
    y0 = _call(g, x, op, backward, IN_PLACE)
    assert bool(((y.double() - y0.double()).abs() <= _bound(g, x, op, backward)).all())


@pytest.mark.parametrize("dtype,f", [(F32, 100), (BF16, 136)])
@pytest.mark.parametrize("weights", [False, True])
def test_strides_weights_and_wide_row_pointers(dtype, f, weights):
    g = _graph(1500000, 21000000, weights=weights, indptr64=True)
    wide = torch.randn(g.n, f + 8, device="cuda").to(dtype)
    x = wide[:, 4:4 + f]  # 16 and 8 bytes behind a line, rows of another stride
    y = _call(g, x, gnn.GNN_SUM, False)
    y0 = _call(g, x, gnn.GNN_SUM, False, IN_PLACE)
    assert g.plan_fwd.blocked_sizes()[2] > 0
    assert bool(((y.double() - y0.double()).abs() <= _bound(g, x.contiguous(), gnn.GNN_SUM, False)).all())


def test_infinities_and_nan_stay_where_they_are_gathered():
    g = _graph(1800000, 26000000)
    x = torch.randn(g.n, 100, device="cuda")
    counts = torch.bincount(g.indices, minlength=g.n)
    order = torch.argsort(counts, descending=True)
    for place, value in ((3, float("inf")), (40000, float("nan")), (200000, -float("inf")), (700000, float("nan"))):
        x[order[place], place % 100] = value
    y, y0 = _call(g, x, gnn.GNN_SUM, False), _call(g, x, gnn.GNN_SUM, False, IN_PLACE)
    assert bool((torch.isnan(y) == torch.isnan(y0)).all())
    inf = torch.isinf(y0)
    assert bool((torch.isinf(y) == inf).all()) and bool((y[inf] == y0[inf]).all()) and bool(inf.any())


def _exact_sum(g, x):
    """Sums over the rows in 64 bits, and those of the magnitudes."""
    dst = torch.repeat_interleave(torch.arange(g.n, device="cuda"), (g.indptr[1:] - g.indptr[:-1]).long())
    want, size = (torch.zeros(x.shape, dtype=torch.float64, device="cuda") for _ in range(2))
    for c in range(0, x.shape[1], 32):
        terms = x[:, c:c + 32].double()[g.indices.long()]
        want[:, c:c + 32].index_add_(0, dst, terms)
        size[:, c:c + 32].index_add_(0, dst, terms.abs())
    return want, size


@pytest.mark.parametrize("blocking,tables", [(dict(hot_lines=65537), False), (dict(block_lines=100000), False), (dict(hot_lines=40001, block_lines=9999), True)])
def test_blocks_of_any_size(blocking, tables):
    """Blocks beyond 16-bit indices leave the rows in place; sizes that are no whole tiles or chunks have tables."""
    el = synth.rmat_directed(1200000, 18000000, STRONG, 19, device="cuda")
    g = gnn.build_device_graph(el.dst, el.src, el.n)
    g.plan_fwd.set_blocking(**blocking)
    x = torch.empty(g.n, 100, device="cuda").normal_(generator=torch.Generator(device="cuda").manual_seed(1))
    g.plan_fwd.prepare(g.indices, gnn.GNN_SUM, False, 100)
    y = _call(g, x, gnn.GNN_SUM, False)
    assert (g.plan_fwd.blocked_sizes()[2] > 0) == tables
    want, size = _exact_sum(g, x)
    assert bool(((y.double() - want).abs() <= 1e-5 * size).all())


def test_bit_matrix_over_tables_that_end_within_a_chunk():
    """All sources of the tables are in the bit matrix, and their number is no multiple of the 128 sources that its kernel takes at a time."""
    n, hot, gen = 300000, 20000, torch.Generator(device="cuda").manual_seed(2)
    rows = torch.randperm(n, device="cuda", generator=gen)[:520]
    chosen = torch.rand(520, hot, device="cuda", generator=gen) < 0.4
    long_dst, long_src = chosen.nonzero(as_tuple=True)
    short = (torch.randint(0, n, (500000,), device="cuda", generator=gen), torch.randint(hot, n, (500000,), device="cuda", generator=gen))
    dst, src = torch.cat([rows[long_dst], short[0]]), torch.cat([long_src, short[1]])
    dst, order = dst.sort()
    g = gnn.build_device_graph(dst.int(), src[order].int(), n)
    g.plan_fwd.set_blocking(hot_lines=hot)
    x = torch.empty(n, 100, device="cuda").normal_(generator=gen)
    g.plan_fwd.prepare(g.indices, gnn.GNN_SUM, False, 100)
    assert g.plan_fwd.bit_rows() >= 256 and g.plan_fwd.blocked_sizes()[3] == 2
    y = _call(g, x, gnn.GNN_SUM, False)
    want, size = _exact_sum(g, x)
    assert bool(((y.double() - want).abs() <= 1e-5 * size).all())


@pytest.mark.parametrize("prepared", [False, True])
def test_capture(prepared):
    el = synth.rmat_directed(1200000, 18000000, STRONG, 18, device="cuda")
    g = gnn.build_device_graph(el.dst, el.src, el.n)
    x, other = torch.randn(g.n, 128, device="cuda"), torch.randn(g.n, 128, device="cuda")
    if prepared:
        g.plan_fwd.prepare(g.indices, gnn.GNN_MEAN, False, 128)
    else:
        g.plan_fwd.reserve(128)
    y = torch.empty_like(x)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            _call(g, x, gnn.GNN_MEAN, False, out=y)
    assert (g.plan_fwd.blocked_sizes()[2] > 0) == prepared  # nothing is built in a capture: that call stays in place
    for values in (x.clone(), other, x.clone()):
        x.copy_(values)
        graph.replay()
        torch.cuda.synchronize()
        eager = _call(g, x, gnn.GNN_MEAN, False, 0 if prepared else IN_PLACE)
        assert torch.equal(y, eager)
