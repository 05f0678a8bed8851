"""Graphs of few edges per vertex whose long rows gather the most-gathered sources from tables and everything else in place, against sums in
64 bits; the call that stays in place is held to the same bound."""
import pytest
import torch

import paper_2104_06700_amd as gnn
import synth

pytestmark = pytest.mark.gpu

F32, BF16 = torch.float32, torch.bfloat16
STRONG = (0.57, 0.19, 0.19, 0.05)
IN_PLACE = gnn.GNN_FLAG_NO_SOURCE_BLOCKS
_edges = {}


def _graph(n, e, weights=False, indptr64=False):
    """With plans of its own, so that what one form has built does not serve another."""
    if (n, e) not in _edges:
        _edges.clear()
        _edges[n, e] = synth.rmat_directed(n, e, STRONG, 17, device="cuda")
    el = _edges[n, e]
    w = torch.rand(e, device="cuda", generator=_gen(5)) + 0.5 if weights else None
    g = gnn.build_device_graph(el.dst, el.src, n, edge_w=w, indptr64=indptr64)
    if weights:
        g.plan_fwd.bind_edge_weights(g.edge_w)
        g.plan_bwd.bind_edge_weights(g.edge_w_t)
    return g


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _normal(seed, n, f, dtype=F32):
    return torch.empty(n, f, device="cuda").normal_(generator=_gen(seed)).to(dtype)


def _prepare(g, f, op, backward=False, dtype=F32):
    (g.plan_bwd if backward else g.plan_fwd).prepare(g.indices_t if backward else g.indices, op, backward, f, dtype)


def _call(g, x, op, backward, flags=0, out=None, stream=None):
    n, f = x.shape
    y = torch.full((n, f), float("nan"), device="cuda", dtype=x.dtype) if out is None else out
    if backward:
        gnn.gnn_aggregate_bwd(g.indptr_t, g.indices_t, g.edge_w_t, x, y, n, f, op, plan=g.plan_bwd, flags=flags)
    else:
        gnn.gnn_aggregate_fwd(g.indptr, g.indices, g.edge_w, x, y, n, f, op, plan=g.plan_fwd, flags=flags)
    return y


def _exact(g, x, op, backward):
    """The result in 64 bits, and the sum of its terms' magnitudes."""
    indptr, indices, w = (g.indptr_t, g.indices_t, g.edge_w_t) if backward else (g.indptr, g.indices, g.edge_w)
    n = g.n
    count = (indptr[1:] - indptr[:-1]).long()
    dst, src = torch.repeat_interleave(torch.arange(n, device="cuda"), count), indices.long()
    of_row, of_source = count.double(), torch.bincount(src, minlength=n).double()  # edges that end, and that begin
    ones = torch.ones(n, dtype=torch.float64, device="cuda")
    into, out = {gnn.GNN_SUM: (ones, ones), gnn.GNN_GCN_SYM: (of_source.clamp(min=1).rsqrt(), of_row.clamp(min=1).rsqrt()),
                 gnn.GNN_MEAN: (1 / of_source.clamp(min=1), ones) if backward else (ones, 1 / of_row.clamp(min=1)),
                 gnn.GNN_SAGE_GCN: (1 / (of_source + 1), ones) if backward else (ones, 1 / (of_row + 1))}[op]
    want, size = (torch.zeros(x.shape, dtype=torch.float64, device="cuda") for _ in range(2))
    for c in range(0, x.shape[1], 32):
        own = x[:, c:c + 32].double() * into[:, None]
        terms = own[src]
        if w is not None:
            terms *= w.double()[:, None]
        for total, at, mine in ((want, terms, own), (size, terms.abs(), own.abs())):
            cols = total[:, c:c + 32]
            if op == gnn.GNN_SAGE_GCN:
                cols += mine
            cols.index_add_(0, dst, at)
            cols *= out[:, None]
    return want, size


def _assert_within(y, exact):
    # fp32 sums of terms that are rounded themselves; a bf16 result is rounded once more, by up to 2^-8 of the value (8 significant bits)
    want, size = exact
    bound = 1e-5 * size
    if y.dtype == BF16:
        bound += 2.0 ** -8 * (want.abs() + bound)
    assert bool(((y.double() - want).abs() <= bound).all())


# whole lines, a last line of one strip, rows off line boundaries, rows of one line and a bit, two launches of slices; every factor, the own row
FORMS = [(F32, 256, gnn.GNN_MEAN, False), (F32, 256, gnn.GNN_MEAN, True), (F32, 36, gnn.GNN_SUM, False), (F32, 100, gnn.GNN_SAGE_GCN, True),
         (F32, 100, gnn.GNN_SAGE_GCN, False), (F32, 292, gnn.GNN_GCN_SYM, False), (F32, 604, gnn.GNN_MEAN, False), (BF16, 128, gnn.GNN_MEAN, False),
         (BF16, 72, gnn.GNN_MEAN, True), (BF16, 200, gnn.GNN_SAGE_GCN, False), (BF16, 264, gnn.GNN_GCN_SYM, True)]


@pytest.mark.parametrize("dtype,f,op,backward", FORMS)
def test_agrees_with_sums_in_64_bits(dtype, f, op, backward):
    g = _graph(1800000, 26000000)
    x = _normal(f, g.n, f, dtype)
    _prepare(g, f, op, backward, dtype)
    y, y0 = _call(g, x, op, backward), _call(g, x, op, backward, IN_PLACE)
    exact = _exact(g, x, op, backward)
    _assert_within(y, exact)
    _assert_within(y0, exact)
    assert not torch.equal(y, y0), "sums in another order: some bit differs where the tables were used"


@pytest.mark.parametrize("dtype,f", [(F32, 100), (BF16, 136)])
@pytest.mark.parametrize("weights", [False, True])
def test_strides_weights_and_wide_row_pointers(dtype, f, weights):
    g = _graph(1500000, 21000000, weights=weights, indptr64=True)
    x = _normal(f, g.n, f + 8, dtype)[:, 4:4 + f]  # 16 and 8 bytes behind a line, rows of another stride
    _prepare(g, f, gnn.GNN_SUM, dtype=dtype)
    y, y0 = _call(g, x, gnn.GNN_SUM, False), _call(g, x, gnn.GNN_SUM, False, IN_PLACE)
    exact = _exact(g, x, gnn.GNN_SUM, False)
    _assert_within(y, exact)
    _assert_within(y0, exact)
    assert not torch.equal(y, y0)


def test_infinities_and_nan_stay_where_they_are_gathered():
    g = _graph(1800000, 26000000)
    x = _normal(6, g.n, 100)
    counts = torch.bincount(g.indices, minlength=g.n)
    order = torch.argsort(counts, descending=True)
    for place, value in ((3, float("inf")), (40000, float("nan")), (200000, -float("inf")), (700000, float("nan"))):
        x[order[place], place % 100] = value
    _prepare(g, 100, gnn.GNN_SUM)
    y, y0 = _call(g, x, gnn.GNN_SUM, False), _call(g, x, gnn.GNN_SUM, False, IN_PLACE)
    want, _ = _exact(g, x, gnn.GNN_SUM, False)
    assert bool(torch.isinf(want).any()) and not torch.equal(torch.nan_to_num(y), torch.nan_to_num(y0))
    for got in (y, y0):
        assert bool((torch.isnan(got) == torch.isnan(want)).all())
        inf = torch.isinf(want)
        assert bool((torch.isinf(got) == inf).all()) and bool((got[inf].double() == want[inf]).all())


def test_a_plan_that_is_not_prepared_builds_none():
    """A new subgraph's plans serve a call or two each: the first calls cost no more than those that stay in place."""
    g = _graph(1800000, 26000000)
    x = _normal(9, g.n, 100)
    y, y0 = _call(g, x, gnn.GNN_SUM, False), _call(g, x, gnn.GNN_SUM, False, IN_PLACE)
    assert torch.equal(y, y0) and g.plan_fwd.blocked_sizes()[2] == 0
    _prepare(g, 100, gnn.GNN_SUM)
    assert not torch.equal(_call(g, x, gnn.GNN_SUM, False), y0) and g.plan_fwd.blocked_sizes()[2] > 0
    # prepared for sums without factors: symmetric factors have none of their own there
    assert torch.equal(_call(g, x, gnn.GNN_GCN_SYM, False), _call(g, x, gnn.GNN_GCN_SYM, False, IN_PLACE))


def test_nothing_is_left_of_tables_that_there_is_no_room_for():
    """gnn_plan_prepare finds room for a part only: it gives that back and holds what it holds for a plan without tables, the call stays in
    place, and with room again they are built."""
    def held_after_prepare(g):
        torch.cuda.synchronize()
        gnn.gnn_release_cached_memory()
        before = torch.cuda.mem_get_info()[0]
        _prepare(g, 100, gnn.GNN_SUM)
        torch.cuda.synchronize()
        gnn.gnn_release_cached_memory()
        return before - torch.cuda.mem_get_info()[0]

    g, without = _graph(1800000, 26000000), _graph(1800000, 26000000)
    without.plan_fwd.set_blocking(hot_lines=65537)
    x = _normal(10, g.n, 100)
    y, y0 = torch.full_like(x, float("nan")), _call(g, x, gnn.GNN_SUM, False, IN_PLACE)
    _call(without, x, gnn.GNN_SUM, False, out=y)
    _prepare(_graph(1800000, 26000000), 100, gnn.GNN_SUM)  # the kernels that build them are loaded
    least = held_after_prepare(without)
    torch.cuda.empty_cache()
    # 260 MB: the mapped index copy takes 126 with its row pointers, the sort of the long rows more than the rest
    filler = [torch.empty(torch.cuda.mem_get_info()[0] - (2 << 30), dtype=torch.uint8, device="cuda")]
    while torch.cuda.mem_get_info()[0] > 260 << 20:
        filler.append(torch.empty(32 << 20, dtype=torch.uint8, device="cuda"))
    assert held_after_prepare(g) <= least + (4 << 20)
    _call(g, x, gnn.GNN_SUM, False, out=y)
    del filler
    torch.cuda.empty_cache()
    assert g.plan_fwd.blocked_sizes()[2] == 0 and torch.equal(y, y0)
    _prepare(g, 100, gnn.GNN_SUM)
    assert g.plan_fwd.blocked_sizes()[2] > 0 and not torch.equal(_call(g, x, gnn.GNN_SUM, False), y0)


def test_memory_that_torch_has_cached_is_room_for_tables():
    """The device is full of blocks that torch's allocator keeps for later: preparing hands them back to the driver and builds the tables."""
    g = _graph(1800000, 26000000)
    x = _normal(13, g.n, 100)
    y0 = _call(g, x, gnn.GNN_SUM, False, IN_PLACE)
    y = torch.empty_like(y0)
    torch.cuda.synchronize()
    gnn.gnn_release_cached_memory()
    filler = [torch.empty(torch.cuda.mem_get_info()[0] - (2 << 30), dtype=torch.uint8, device="cuda")]
    while torch.cuda.mem_get_info()[0] > 260 << 20:
        filler.append(torch.empty(32 << 20, dtype=torch.uint8, device="cuda"))
    _prepare(g, 100, gnn.GNN_SUM)
    assert g.plan_fwd.blocked_sizes()[2] == 0 and gnn.load_library().gnn_plan_lacks_room(g.plan_fwd.handle) == 1
    del filler
    assert torch.cuda.mem_get_info()[0] < 520 << 20
    _prepare(g, 100, gnn.GNN_SUM)
    assert g.plan_fwd.blocked_sizes()[2] > 0 and gnn.load_library().gnn_plan_lacks_room(g.plan_fwd.handle) == 0
    assert not torch.equal(_call(g, x, gnn.GNN_SUM, False, out=y), y0)
    torch.cuda.empty_cache()


@pytest.mark.parametrize("prepared", [False, True])
def test_packed_copies_of_all_rows(prepared):
    """A plan whose blocks a call over a packed copy has made has them as for any graph, tables for the last one's sources included, and its other calls
    stay in place; over a plan prepared for hot tables that call takes their blocks."""
    g, as_given = _graph(1800000, 26000000), _graph(1800000, 26000000)
    as_given.plan_fwd.set_blocking(max_piece=96, rest_min_count=16)
    x = _normal(12, g.n, 100)
    packed = torch.empty(gnn.gnn_packed_bytes(g.n, 100, gnn.GNN_F32), dtype=torch.uint8, device="cuda")

    def packed_call(h):
        y = torch.full_like(x, float("nan"))
        gnn.gnn_pack_rows(h.indptr, h.indices, x, packed, h.n, 100, gnn.GNN_SUM, False, h.plan_fwd)
        gnn.gnn_aggregate_packed(h.indptr, h.indices, None, packed, y, h.n, 100, gnn.GNN_SUM, False, h.plan_fwd)
        return y

    if prepared:
        _prepare(g, 100, gnn.GNN_SUM)
    y, y_given = packed_call(g), packed_call(as_given)
    assert (g.plan_fwd.blocked_sizes() == as_given.plan_fwd.blocked_sizes()) != prepared
    assert prepared or torch.equal(y, y_given)
    exact = _exact(g, x, gnn.GNN_SUM, False)
    _assert_within(y, exact)
    _prepare(g, 100, gnn.GNN_SUM)
    y, y0 = _call(g, x, gnn.GNN_SUM, False), _call(g, x, gnn.GNN_SUM, False, IN_PLACE)
    assert torch.equal(y, y0) != prepared
    _assert_within(y, exact)


@pytest.mark.parametrize("blocking,tables", [(dict(hot_lines=65537), False), (dict(block_lines=100000), False), (dict(hot_lines=40001, block_lines=9999), True)])
def test_blocks_of_any_size(blocking, tables):
    """Blocks beyond 16-bit indices leave the rows in place; sizes that are no whole tiles or chunks have tables."""
    el = synth.rmat_directed(1200000, 18000000, STRONG, 19, device="cuda")
    g = gnn.build_device_graph(el.dst, el.src, el.n)
    g.plan_fwd.set_blocking(**blocking)
    x = _normal(1, g.n, 100)
    _prepare(g, 100, gnn.GNN_SUM)
    y = _call(g, x, gnn.GNN_SUM, False)
    assert (g.plan_fwd.blocked_sizes()[2] > 0) == tables
    _assert_within(y, _exact(g, x, gnn.GNN_SUM, False))


def test_bit_matrix_over_tables_that_end_within_a_chunk():
    """All sources of the tables are in the bit matrix, and their number is no multiple of the 128 sources that its kernel takes at a time."""
    n, hot, gen = 300000, 20000, _gen(2)
    rows = torch.randperm(n, device="cuda", generator=gen)[:520]
    chosen = torch.rand(520, hot, device="cuda", generator=gen) < 0.4
    long_dst, long_src = chosen.nonzero(as_tuple=True)
    short = (torch.randint(0, n, (500000,), device="cuda", generator=gen), torch.randint(hot, n, (500000,), device="cuda", generator=gen))
    dst, src = torch.cat([rows[long_dst], short[0]]), torch.cat([long_src, short[1]])
    dst, order = dst.sort()
    g = gnn.build_device_graph(dst.int(), src[order].int(), n)
    g.plan_fwd.set_blocking(hot_lines=hot)
    x = torch.empty(n, 100, device="cuda").normal_(generator=gen)
    _prepare(g, 100, gnn.GNN_SUM)
    assert g.plan_fwd.bit_rows() >= 256 and g.plan_fwd.blocked_sizes()[3] == 2
    _assert_within(_call(g, x, gnn.GNN_SUM, False), _exact(g, x, gnn.GNN_SUM, False))


@pytest.mark.parametrize("prepared", [False, True])
def test_capture(prepared):
    el = synth.rmat_directed(1200000, 18000000, STRONG, 18, device="cuda")
    g = gnn.build_device_graph(el.dst, el.src, el.n)
    x, other = _normal(7, g.n, 128), _normal(8, g.n, 128)
    if prepared:
        _prepare(g, 128, gnn.GNN_MEAN)
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
