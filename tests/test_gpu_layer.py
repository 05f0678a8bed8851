"""GPU parity of the dense update (gnn_matmul on the matrix cores) and of the GraphSAGE layer
(aggregation + update, forward and gradients) against the fp64 CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2104_06700_amd as gnn
import synth
from helpers import device_graph, host_csr

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
# fp32 products are exact on the matrix cores but for 2^-24 of S; the accumulation of K terms in fp32 (in steps of
# 16, partial planes of >= GNN_SPLIT_MIN_K = 128 rows) and the fp32 aggregation before or after it leave an error of
# at most (1e-5 + K * 2^-24) * S in the worst case and ~sqrt(K) * 2^-24 * S typically, S being the
# sum of the absolute values of all terms; gate at 2e-5 * S.
RTOL_LAYER = 2e-5


def _close(g, ref, S, what, rtol=RTOL_LAYER):
    g = g.detach().cpu().numpy().astype(np.float64)
    assert g.shape == ref.shape, (g.shape, ref.shape)
    assert np.isfinite(g).all(), what
    err = np.abs(g - ref)
    bound = rtol * S
    bad = err > bound
    if bad.any():
        i = np.unravel_index(np.argmax(err - bound), err.shape)
        raise AssertionError(f"{what}: {bad.sum()} of {bad.size} out of tolerance; worst at {i}: gpu={g[i]!r} "
                             f"oracle={ref[i]!r} err={err[i]:.3e} bound={bound[i]:.3e}")


@pytest.mark.parametrize("m,n,k", [(1, 1, 1), (128, 128, 16), (130, 127, 17), (300, 47, 100), (1000, 256, 100),
                                   (257, 300, 602), (64, 16, 602), (5, 7, 0)])
@pytest.mark.parametrize("ta,tb", [(False, False), (False, True), (True, False), (True, True)])
def test_matmul_every_layout(m, n, k, ta, tb):
    rng = np.random.default_rng(m * 7 + n * 3 + k)
    A = rng.normal(size=(k, m) if ta else (m, k)).astype(np.float32)
    B = rng.normal(size=(n, k) if tb else (k, n)).astype(np.float32)
    bias = rng.normal(size=n).astype(np.float32)
    for use_bias, relu in ((False, False), (True, True)):
        print(f"matmul m={m} n={n} k={k} ta={ta} tb={tb} bias={use_bias} relu={relu}", flush=True)
        C = torch.full((m, n), float("nan"), device=DEV)
        gnn.gnn_matmul(torch.from_numpy(A).to(DEV), torch.from_numpy(B).to(DEV), C, ta, tb,
                       torch.from_numpy(bias).to(DEV) if use_bias else None, relu)
        torch.cuda.synchronize()
        ref, S = oracle.matmul(A, B, ta, tb, bias if use_bias else None, relu)
        _close(C, ref, np.maximum(S, 1e-30), "matmul")


def test_matmul_strided_and_misaligned():
    rng = np.random.default_rng(5)
    m, n, k = 200, 90, 75
    for lda, ldb, ldc, off in ((75, 90, 90, 1), (80, 96, 100, 0), (77, 91, 93, 3)):
        bufA = torch.from_numpy(rng.normal(size=m * lda + 8).astype(np.float32)).to(DEV)
        bufB = torch.from_numpy(rng.normal(size=k * ldb + 8).astype(np.float32)).to(DEV)
        bufC = torch.full((m * ldc + 8,), float("nan"), device=DEV)
        A = torch.as_strided(bufA, (m, k), (lda, 1), off)
        B = torch.as_strided(bufB, (k, n), (ldb, 1), off)
        C = torch.as_strided(bufC, (m, n), (ldc, 1), off)
        gnn.gnn_matmul(A, B, C)
        torch.cuda.synchronize()
        ref, S = oracle.matmul(A.cpu().numpy(), B.cpu().numpy())
        _close(C, ref, S, f"strided {lda}/{ldb}/{ldc}+{off}")
        written = torch.zeros_like(bufC, dtype=torch.bool)
        torch.as_strided(written, (m, n), (ldc, 1), off).fill_(True)
        assert torch.isnan(bufC[~written]).all(), "stores outside C"


def test_matmul_long_reduction_is_split_and_deterministic():
    """The weight-gradient shape: few output tiles, a reduction over many rows."""
    rng = np.random.default_rng(6)
    rows, fi, fo = 200_000, 100, 47
    Z = rng.normal(size=(rows, fi)).astype(np.float32)
    G = rng.normal(size=(rows, fo)).astype(np.float32)
    need = gnn.gnn_matmul_workspace_bytes(fi, fo, rows)
    assert need > 0
    ws = torch.empty(need // 4, device=DEV)
    Zd, Gd = torch.from_numpy(Z).to(DEV), torch.from_numpy(G).to(DEV)
    out = []
    for _ in range(2):
        C = torch.full((fi, fo), float("nan"), device=DEV)
        gnn.gnn_matmul(Zd, Gd, C, trans_a=True, workspace=ws)
        torch.cuda.synchronize()
        out.append(C.clone())
    assert torch.equal(out[0], out[1])
    ref = Z.astype(np.float64).T @ G.astype(np.float64)   # the oracle's triple loop would take minutes here;
    S = np.abs(Z.astype(np.float64)).T @ np.abs(G.astype(np.float64))  # it is pinned to this very routine
    _close(out[0], ref, S, "split reduction")
    C = torch.full((fi, fo), float("nan"), device=DEV)
    gnn.gnn_matmul(Zd, Gd, C, trans_a=True)  # no workspace: unsplit, still right
    torch.cuda.synchronize()
    _close(C, ref, S, "unsplit long reduction", rtol=2e-4)


@pytest.mark.parametrize("m,n,k,ta,tb", [(128 * 21 + 5, 256, 40, False, False), (128 * 17, 300, 64, False, True),
                                         (256 * 19 + 1, 47, 100, False, False), (128 * 40, 130, 33, True, True)])
def test_matmul_tall_results_with_the_tile_order_for_the_xcds(m, n, k, ta, tb):
    """Many row tiles and a few column tiles: the column tiles of one row tile get workgroup ids 8 apart
    (same XCD), the last group of 8 row tiles is incomplete."""
    rng = np.random.default_rng(m + n)
    A = rng.normal(size=(k, m) if ta else (m, k)).astype(np.float32)
    B = rng.normal(size=(n, k) if tb else (k, n)).astype(np.float32)
    bias = rng.normal(size=n).astype(np.float32)
    C = torch.full((m, n), float("nan"), device=DEV)
    gnn.gnn_matmul(torch.from_numpy(A).to(DEV), torch.from_numpy(B).to(DEV), C, ta, tb, torch.from_numpy(bias).to(DEV), True)
    torch.cuda.synchronize()
    A64, B64 = A.astype(np.float64), B.astype(np.float64)   # the oracle's loop is pinned to this routine; see above
    opA, opB = (A64.T if ta else A64), (B64.T if tb else B64)
    ref = np.maximum(opA @ opB + bias, 0.0)
    S = np.abs(opA) @ np.abs(opB) + np.abs(bias)
    _close(C, ref, S, "tall product")


def test_matmul_split_reduction_of_several_tiles():
    """Four output tiles and a long reduction: all tiles of one part run on one XCD, parts on all eight."""
    rng = np.random.default_rng(61)
    rows, fi, fo = 70_000, 200, 140
    Z = rng.normal(size=(rows, fi)).astype(np.float32)
    G = rng.normal(size=(rows, fo)).astype(np.float32)
    ws = torch.empty(gnn.gnn_matmul_workspace_bytes(fi, fo, rows) // 4, device=DEV)
    assert ws.numel() >= 16 * fi * fo
    C = torch.full((fi, fo), float("nan"), device=DEV)
    gnn.gnn_matmul(torch.from_numpy(Z).to(DEV), torch.from_numpy(G).to(DEV), C, trans_a=True, workspace=ws)
    torch.cuda.synchronize()
    ref = Z.astype(np.float64).T @ G.astype(np.float64)
    S = np.abs(Z.astype(np.float64)).T @ np.abs(G.astype(np.float64))
    _close(C, ref, S, "split reduction over several tiles")


# ------------------------------------------------------------------ one layer
def _graph(kind):
    if kind == "multi":
        return synth.small_random_multigraph(900, 7000, 3), None
    if kind == "rmat_hubs":
        return synth.rmat_symmetric(4000, 120000, (0.57, 0.19, 0.19, 0.05), 5), gnn.make_plan_params([2, 8, 32, 128], 64)
    raise KeyError(kind)


def _layer_case(el, params, fi, fo, relu, order, seed, use_bias=True, want_dx=True, flags=0):
    rng = np.random.default_rng(seed)
    n = el.n
    dg = device_graph(el, plan_params=params)
    indptr, indices, *_ = host_csr(el)
    X = rng.normal(size=(n, fi)).astype(np.float32)
    W = (rng.normal(size=(fi, fo)) / np.sqrt(fi)).astype(np.float32)
    b = rng.normal(size=fo).astype(np.float32) if use_bias else None
    dH = rng.normal(size=(n, fo)).astype(np.float32)
    what = f"n={n} E={el.e} {fi}->{fo} relu={relu} order={order} bias={use_bias}"
    print(what, flush=True)
    Xd, Wd, dHd = (torch.from_numpy(a).to(DEV) for a in (X, W, dH))
    bd = None if b is None else torch.from_numpy(b).to(DEV)
    saved = torch.full((gnn.gnn_sage_layer_saved_elems(n, fi, fo, order),), float("nan"), device=DEV)
    H = torch.full((n, fo), float("nan"), device=DEV)
    gnn.gnn_sage_layer_fwd(dg.indptr, dg.indices, Xd, Wd, bd, saved, H, dg.plan_fwd, relu=relu, order=order, flags=flags)
    torch.cuda.synchronize()
    Z, Ho, SH = oracle.sage_layer_fwd(indptr, indices, X, W, b, relu)
    _close(H, Ho, SH, "forward " + what)
    # backward; the stored forward output that decides the rectifier's mask is the oracle's, for both sides
    Hs = Ho.astype(np.float32)
    extra = n * fo + 64 if flags & gnn.GNN_LAYER_NO_GATE_FOLD else 0  # room for the masked gradient
    ws = torch.empty(max(1, gnn.gnn_sage_layer_workspace_bytes(n, fi, fo, relu, order) // 4) + extra, device=DEV)
    dX = torch.full((n, fi), float("nan"), device=DEV) if want_dx else None
    dW = torch.full((fi, fo), float("nan"), device=DEV)
    db = torch.full((fo,), float("nan"), device=DEV)
    gnn.gnn_sage_layer_bwd(dg.indptr_t, dg.indices_t, Xd, Wd, saved, torch.from_numpy(Hs).to(DEV), dHd, dX, dW, db,
                           dg.plan_bwd, ws, relu=relu, order=order, flags=flags)
    torch.cuda.synchronize()
    g = oracle.sage_layer_bwd(indptr, indices, X, W, Hs, dH, relu)
    _close(dW, g["dW"][0], g["dW"][1], "dW " + what)
    _close(db, g["db"][0], g["db"][1], "db " + what)
    if want_dx:
        _close(dX, g["dX"][0], g["dX"][1], "dX " + what)


@pytest.mark.parametrize("kind", ["multi", "rmat_hubs"])
@pytest.mark.parametrize("fi,fo", [(100, 256), (256, 47), (602, 16), (5, 3), (64, 64), (33, 130)])
@pytest.mark.parametrize("relu", [True, False])
def test_layer_forward_and_gradients(kind, fi, fo, relu):
    el, params = _graph(kind)
    _layer_case(el, params, fi, fo, relu, order=0, seed=fi + fo)


@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("fi,fo", [(100, 256), (256, 47)])
def test_layer_either_order_gives_the_same_layer(order, fi, fo):
    el, params = _graph("rmat_hubs")
    _layer_case(el, params, fi, fo, True, order=order, seed=9)


@pytest.mark.parametrize("order", [0, 1, 2])
@pytest.mark.parametrize("fi,fo", [(100, 256), (256, 47), (64, 64), (40, 132), (130, 33)])
@pytest.mark.parametrize("flags", [gnn.GNN_LAYER_FORCE_PRODUCER_LAYOUT, gnn.GNN_LAYER_NO_PRODUCER_LAYOUT])
def test_layer_producer_side_layouts(order, fi, fo, flags):
    """The matrix a layer's aggregation gathers (X W, the masked output gradient, its product with W^T)
    written by its producer straight into the tables of the plan -- forced here on a small graph, with
    hub rows, a dense tail (47, 100, 130) and both orders -- and, for comparison, never."""
    el, params = _graph("rmat_hubs")
    _layer_case(el, params, fi, fo, True, order=order, seed=21, flags=flags)
    _layer_case(el, params, fi, fo, False, order=order, seed=22, flags=flags, use_bias=False)


@pytest.mark.parametrize("fi,fo", [(100, 256), (40, 47), (64, 64), (20, 24), (130, 133)])
@pytest.mark.parametrize("flags", [0, gnn.GNN_LAYER_NO_GATE_FOLD, gnn.GNN_LAYER_FORCE_PRODUCER_LAYOUT])
def test_layer_backward_with_the_rectifier_folded_into_the_products(fi, fo, flags):
    """Aggregating first, the two backward products read dH and H themselves (the gate is applied while
    the operand is staged, the bias gradient is added up from the staged tiles) -- all three tile shapes of
    the product (outputs of up to 32, up to 64 and more columns), with and without a rectifier, with and
    without an input gradient -- and, for comparison, with the masked gradient written first."""
    el, params = _graph("rmat_hubs")
    _layer_case(el, params, fi, fo, True, order=1, seed=31, flags=flags)
    _layer_case(el, params, fi, fo, False, order=1, seed=32, flags=flags)
    _layer_case(el, params, fi, fo, True, order=1, seed=33, flags=flags, want_dx=False)
    _layer_case(el, params, fi, fo, True, order=1, seed=34, flags=flags, use_bias=False)


@pytest.mark.parametrize("flags", [0, gnn.GNN_LAYER_NO_GATE_FOLD])
def test_layer_backward_folded_rectifier_with_a_split_reduction(flags):
    """Enough vertices that the weight-gradient product splits its reduction: the bias gradient then comes
    in one plane per part and is added in plane order; twice the same bits."""
    el = synth.small_random_multigraph(9500, 60000, 8)
    assert gnn.gnn_matmul_workspace_bytes(72, 40, el.n) > 0
    _layer_case(el, None, 72, 40, True, order=1, seed=41, flags=flags)
    _layer_case(el, None, 24, 140, True, order=0, seed=42, flags=flags)
    big = synth.small_random_multigraph(40000, 150000, 9)   # 39 parts of 4 tiles: the tile order for the XCDs
    _layer_case(big, None, 130, 140, True, order=1, seed=43, flags=flags)
    n, fi, fo = el.n, 24, 140
    dg = device_graph(el)
    g = torch.Generator(device="cpu").manual_seed(3)
    X, W, H, dH = (torch.randn(s_, generator=g).to(DEV) for s_ in ((n, fi), (fi, fo), (n, fo), (n, fo)))
    saved = torch.randn(n, fi, generator=g).to(DEV)
    ws = torch.empty(gnn.gnn_sage_layer_workspace_bytes(n, fi, fo, True, 0) // 4 + n * fo + 64, device=DEV)
    outs = []
    for _ in range(2):
        dX, dW, db = torch.empty(n, fi, device=DEV), torch.empty(fi, fo, device=DEV), torch.empty(fo, device=DEV)
        gnn.gnn_sage_layer_bwd(dg.indptr_t, dg.indices_t, X, W, saved, H, dH, dX, dW, db, dg.plan_bwd, ws, relu=True, order=0,
                               flags=flags)
        torch.cuda.synchronize()
        outs.append((dX, dW, db))
    for a, b in zip(*outs):
        assert torch.equal(a, b)


_narrow = {}


def _narrow_graph():
    """30 edges per vertex: the aggregation of narrow rows has a copy to gather from, and the weight gradient runs beside it."""
    if not _narrow:
        _narrow["el"] = synth.rmat_symmetric(200_000, 6_000_000, (0.45, 0.22, 0.22, 0.11), 8)
    return _narrow["el"]


@pytest.mark.parametrize("fi,fo,relu", [(16, 16, True), (24, 41, False), (32, 64, True)])
def test_layer_weight_gradient_beside_the_aggregation(fi, fo, relu):
    _layer_case(_narrow_graph(), None, fi, fo, relu, 0, seed=fi)


def test_layer_weight_gradient_beside_the_aggregation_under_capture():
    """The second stream joins the capture; replays with other gradients and eager work between them give the eager call's bits."""
    el, fi, fo = _narrow_graph(), 16, 24
    dg, n = device_graph(el), el.n
    gen = torch.Generator(device=DEV).manual_seed(4)
    rand = lambda *shape: torch.empty(shape, device=DEV).normal_(generator=gen)
    x, w, h, saved = rand(n, fi), rand(fi, fo), rand(n, fo).clamp_(min=0.0), rand(gnn.gnn_sage_layer_saved_elems(n, fi, fo))
    dh, other = rand(n, fo), rand(n, fo)
    ws = torch.empty(gnn.gnn_sage_layer_workspace_bytes(n, fi, fo, True) // 4 + 1, device=DEV)
    dg.plan_bwd.prepare(dg.indices_t, gnn.GNN_SAGE_GCN, True, fi)
    outs = [[torch.full(shape, float("nan"), device=DEV) for shape in ((n, fi), (fi, fo), (fo,))] for _ in range(2)]

    def call(out):
        gnn.gnn_sage_layer_bwd(dg.indptr_t, dg.indices_t, x, w, saved, h, dh, *out, dg.plan_bwd, ws, relu=True)

    call(outs[0])
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(outs[1])
    for values in (dh.clone(), other, dh.clone()):
        dh.copy_(values)
        for t in outs[1]:
            t.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        call(outs[0])
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(*outs))


def test_layer_without_bias_and_without_input_gradient():
    el, params = _graph("multi")
    _layer_case(el, params, 40, 24, True, order=0, seed=10, use_bias=False, want_dx=False)
    _layer_case(el, params, 24, 40, False, order=0, seed=11, use_bias=False, want_dx=False)


def test_layer_gradients_are_reproducible():
    el, params = _graph("rmat_hubs")
    n, fi, fo = el.n, 100, 47
    dg = device_graph(el, plan_params=params)
    X = torch.randn(n, fi, device=DEV)
    W = torch.randn(fi, fo, device=DEV)
    H = torch.randn(n, fo, device=DEV)
    dH = torch.randn(n, fo, device=DEV)
    ws = torch.empty(gnn.gnn_sage_layer_workspace_bytes(n, fi, fo, True, 0) // 4 + n * fo + 64, device=DEV)
    outs = []
    for _ in range(2):
        dX, dW, db = torch.empty(n, fi, device=DEV), torch.empty(fi, fo, device=DEV), torch.empty(fo, device=DEV)
        gnn.gnn_sage_layer_bwd(dg.indptr_t, dg.indices_t, X, W, None, H, dH, dX, dW, db, dg.plan_bwd, ws)
        torch.cuda.synchronize()
        outs.append((dX, dW, db))
    for a, b in zip(*outs):
        assert torch.equal(a, b)


def test_layer_argument_errors():
    el, params = _graph("multi")
    dg = device_graph(el, plan_params=params)
    n = el.n
    X = torch.randn(n, 8, device=DEV)
    W = torch.randn(8, 4, device=DEV)
    H = torch.empty(n, 4, device=DEV)
    saved = torch.empty(n * 8, device=DEV)
    with pytest.raises(gnn.GnnError):   # no plan
        gnn.gnn_sage_layer_fwd(dg.indptr, dg.indices, X, W, None, saved, H, None)
    with pytest.raises(gnn.GnnError):   # workspace too small
        gnn.gnn_sage_layer_bwd(dg.indptr_t, dg.indices_t, X, W, saved, H, H, torch.empty_like(X), torch.empty_like(W), None,
                               dg.plan_bwd, torch.empty(16, device=DEV))
    with pytest.raises(ValueError):
        gnn.gnn_sage_layer_fwd(dg.indptr, dg.indices, X[:, ::2], W, None, saved, H, dg.plan_fwd)


@pytest.mark.timeout(900)
def test_layer_fullsize_sparse_workload():
    """2,449,029 vertices / 123,718,280 edges, the first layer of the paper's model for this graph
    (100 -> 256, aggregate first) and its last (256 -> 47, transform first), default plans.
    Forward: sampled rows against the oracle on the compacted neighbourhood of the sample.
    Backward: the identities that tie the gradients to the forward map, in fp64 on the whole output:
    <G, H> = <dW, W> + <db, b> = <dX, X> + <db, b> with G = dH where H > 0."""
    el = synth.make_graph("rmat_sparse_stack", device=DEV)
    n = el.n
    dg = gnn.build_device_graph(el.dst, el.src, n)
    dst_h, src_h = synth.to_csr_numpy(el)
    indptr = oracle.csr_indptr(dst_h, n)
    deg = np.diff(indptr)
    rng = np.random.default_rng(4)
    rows = np.unique(np.concatenate([np.argsort(deg)[-16:], rng.choice(n, 1500, replace=False), np.flatnonzero(deg == 0)[:8]]))
    # compacted problem: the sampled rows first (their own vectors are needed), then every neighbour
    nbr = np.concatenate([src_h[indptr[r]:indptr[r + 1]] for r in rows]).astype(np.int64)
    ids = np.concatenate([rows, np.setdiff1d(np.unique(nbr), rows)])
    local = np.full(n, -1, dtype=np.int64)
    local[ids] = np.arange(len(ids))
    sub_ptr = np.zeros(len(ids) + 1, dtype=np.int64)
    sub_ptr[1:len(rows) + 1] = np.cumsum(deg[rows])
    sub_ptr[len(rows) + 1:] = sub_ptr[len(rows)]
    sub_idx = local[nbr].astype(np.int32)
    for fi, fo, relu in ((100, 256, True), (256, 47, False)):
        print(f"[fullsize layer] {fi}->{fo} relu={relu}", flush=True)
        X = synth.normal_features(n, fi, 1, device=DEV)
        W = synth.normal_features(fi, fo, 2, device=DEV) / fi ** 0.5
        b = synth.normal_features(1, fo, 3, device=DEV).reshape(fo)
        dH = synth.normal_features(n, fo, 4, device=DEV)
        saved = torch.empty(gnn.gnn_sage_layer_saved_elems(n, fi, fo), device=DEV)
        H = torch.full((n, fo), float("nan"), device=DEV)
        gnn.gnn_sage_layer_fwd(dg.indptr, dg.indices, X, W, b, saved, H, dg.plan_fwd, relu=relu)
        torch.cuda.synchronize()
        assert bool(torch.isfinite(H).all())
        _, Ho, SH = oracle.sage_layer_fwd(sub_ptr, sub_idx, X[torch.from_numpy(ids).to(DEV)].cpu().numpy(), W.cpu().numpy(),
                                          b.cpu().numpy(), relu)
        k = len(rows)
        _close(H[torch.from_numpy(rows).to(DEV)], Ho[:k], SH[:k], f"fullsize forward {fi}->{fo}")
        ws = torch.empty(gnn.gnn_sage_layer_workspace_bytes(n, fi, fo, relu) // 4, device=DEV)
        dX, dW, db = torch.empty((n, fi), device=DEV), torch.empty((fi, fo), device=DEV), torch.empty(fo, device=DEV)
        gnn.gnn_sage_layer_bwd(dg.indptr_t, dg.indices_t, X, W, saved, H, dH, dX, dW, db, dg.plan_bwd, ws, relu=relu)
        torch.cuda.synchronize()
        G = torch.where(H > 0, dH, torch.zeros_like(dH)) if relu else dH
        lhs = (G.double() * H.double()).sum().item()
        scale = (G.double().abs() * H.double().abs()).sum().item() + (db.double().abs() * b.double().abs()).sum().item()
        via_w = (dW.double() * W.double()).sum().item() + (db.double() * b.double()).sum().item()
        via_x = (dX.double() * X.double()).sum().item() + (db.double() * b.double()).sum().item()
        assert abs(lhs - via_w) <= 2e-6 * scale, (lhs, via_w, scale)
        assert abs(lhs - via_x) <= 2e-6 * scale, (lhs, via_x, scale)
        del X, dH, saved, H, ws, dX, G


@pytest.mark.parametrize("seed", range(12))
def test_layer_randomised(seed):
    rng = np.random.default_rng(700 + seed)
    n = int(rng.integers(2, 3000))
    e = int(rng.integers(1, 25 * n + 1))
    if n < 64 or rng.random() < 0.5:
        el = synth.small_random_multigraph(n, e, seed)
    else:
        e = min(e - e % 2, n * (n - 1) // 4 * 2)
        el = synth.rmat_symmetric(n, max(e, 2), (0.57, 0.19, 0.19, 0.05), seed)
    k = int(rng.integers(0, 5))
    thr = sorted(set(int(t) for t in rng.integers(1, 100, size=k)))
    params = gnn.make_plan_params(thr, int(rng.choice([0, 7, 64, 1024])))
    fi = int(rng.choice([1, 3, 16, 31, 47, 100, 129, 300]))
    fo = int(rng.choice([1, 2, 16, 41, 47, 64, 130, 256]))
    _layer_case(el, params, fi, fo, relu=bool(rng.random() < 0.6), order=int(rng.integers(0, 3)), seed=seed,
                use_bias=bool(rng.random() < 0.7), want_dx=bool(rng.random() < 0.8))


def test_layer_int64_row_pointers():
    el, params = _graph("rmat_hubs")
    rng = np.random.default_rng(43)
    n, fi, fo = el.n, 48, 20
    dg = device_graph(el, indptr64=True, plan_params=params)
    indptr, indices, *_ = host_csr(el)
    X = rng.normal(size=(n, fi)).astype(np.float32)
    W = rng.normal(size=(fi, fo)).astype(np.float32)
    Xd, Wd = torch.from_numpy(X).to(DEV), torch.from_numpy(W).to(DEV)
    saved = torch.empty(gnn.gnn_sage_layer_saved_elems(n, fi, fo), device=DEV)
    H = torch.empty((n, fo), device=DEV)
    gnn.gnn_sage_layer_fwd(dg.indptr, dg.indices, Xd, Wd, None, saved, H, dg.plan_fwd, relu=False)
    torch.cuda.synchronize()
    _, Ho, SH = oracle.sage_layer_fwd(indptr, indices, X, W, None, False)
    _close(H, Ho, SH, "layer forward, int64 row pointers")


@pytest.mark.parametrize("n,fi,fo", [(4000, 100, 256), (4000, 20, 24), (4000, 40, 47), (4000, 130, 133), (4000, 30, 9), (66_000, 130, 133),
                                     (66_000, 100, 40), (66_000, 64, 64), (66_000, 20, 16)])
@pytest.mark.parametrize("flags", [0, gnn.GNN_LAYER_FORCE_PRODUCER_LAYOUT, gnn.GNN_LAYER_NO_GATE_FOLD])
def test_layer_backward_of_operands_outside_the_split(n, fi, fo, flags):
    """The tiles that are computed again read the operands, their gates and the producer's layout in a way of their own: infinities and
    NaNs on both sides of the gate, in the operand, in the weights and in the gate itself, and finite numbers beyond the split."""
    el = synth.rmat_symmetric(n, 30 * n, (0.57, 0.19, 0.19, 0.05), 5) if n == 4000 else synth.erdos_renyi_directed(n, 3 * n, 5)
    dg = device_graph(el, plan_params=gnn.make_plan_params([2, 8, 32, 128], 64))
    indptr, indices, indptr_t, indices_t, _ = host_csr(el)
    rng = np.random.default_rng(n + fi + fo)
    X, saved, H, dH = (rng.normal(size=s_).astype(np.float32) for s_ in ((n, fi), (n, fi), (n, fo), (n, fo)))
    W = (rng.normal(size=(fi, fo)) / np.sqrt(fo)).astype(np.float32)
    inf, nan = float("inf"), float("nan")
    for v, c, h, d in ((7, 0, -1, inf), (n - 1, fo - 1, 0, nan), (n // 2, 1, nan, 1), (n // 3, 2, 1, inf), (n // 3 + 1, 3, 1, -inf),
                       (n - 2, 4, 2, 2.0 ** 113), (n // 4, 5, 1, nan), (n // 4 + 40, fo // 2, -2, -inf)):
        H[v, c], dH[v, c] = h, d
    dH[n // 5] *= 2.0 ** -118
    saved[n // 6, fi // 2], saved[n - 3, 1], saved[n - 1, 2] = nan, -inf, 2.0 ** 113
    W[fi // 3, fo // 3] = -inf
    G = np.where(H > 0, dH, np.float32(0)).astype(np.float64)
    with np.errstate(invalid="ignore", over="ignore"):
        Z64, W64 = saved.astype(np.float64), W.astype(np.float64)
        dW, SW, db, Sb = Z64.T @ G, np.abs(Z64).T @ np.abs(G), G.sum(0), np.abs(G).sum(0)
        dZ = (G @ W64.T).astype(np.float32)
        dZ_abs = (np.abs(G) @ np.abs(W64).T).astype(np.float32)
    op = gnn.GNN_SAGE_GCN
    dX = oracle.aggregate_bwd(indptr_t, indices_t, dZ, op=op, din=np.diff(indptr), nthreads=8)
    SX = oracle.aggregate_bwd(indptr_t, indices_t, dZ_abs, op=op, din=np.diff(indptr), nthreads=8)
    ws = torch.empty(gnn.gnn_sage_layer_workspace_bytes(n, fi, fo, True, 1) // 4 + n * fo + 64, device=DEV)
    got = [torch.full(s_, nan, device=DEV) for s_ in ((n, fi), (fi, fo), (fo,))]
    Xd, Wd, sd, Hd, dHd = (torch.from_numpy(a).to(DEV) for a in (X, W, saved, H, dH))
    gnn.gnn_sage_layer_bwd(dg.indptr_t, dg.indices_t, Xd, Wd, sd, Hd, dHd, *got, dg.plan_bwd, ws, relu=True, order=1, flags=flags)
    torch.cuda.synchronize()
    for what, g, ref, S in zip(("dX", "dW", "db"), got, (dX, dW, db), (SX, SW, Sb)):
        g, ref = g.cpu().numpy().astype(np.float64), np.asarray(ref, dtype=np.float64)
        finite = np.isfinite(ref)
        assert finite.any() and not finite.all(), what
        assert np.array_equal(np.isnan(g), np.isnan(ref)), what
        assert np.array_equal(g[np.isinf(ref)], ref[np.isinf(ref)]), what
        err = np.abs(g[finite] - ref[finite])
        assert (err <= RTOL_LAYER * np.asarray(S)[finite] + 2.0 ** -140).all(), (what, err.max())


# ------------------------------------------------------------------ the split operands of the matrix cores
@pytest.mark.parametrize("k", [1, 9, 15, 17, 32, 47])
@pytest.mark.parametrize("m,n", [(31, 33), (300, 65), (513, 257)])
@pytest.mark.parametrize("ta,tb", [(False, False), (False, True), (True, False), (True, True)])
def test_matmul_edges_of_the_steps_of_k(m, n, k, ta, tb):
    """Steps of 16 k: less than one, a last one that is moved back over the step before, odd and even numbers of them; tiles of every
    width.  A product drops at most 2^-24 of S (three of nine partial products, 2^-26 each) and its sums are fp32: with
    k <= 100 far below 1e-6 * S."""
    rng = np.random.default_rng(1000 * k + m + n)
    A = rng.normal(size=(k, m) if ta else (m, k)).astype(np.float32)
    B = rng.normal(size=(n, k) if tb else (k, n)).astype(np.float32)
    C = torch.full((m, n), float("nan"), device=DEV)
    gnn.gnn_matmul(torch.from_numpy(A).to(DEV), torch.from_numpy(B).to(DEV), C, ta, tb)
    torch.cuda.synchronize()
    A64, B64 = A.astype(np.float64), B.astype(np.float64)
    A64, B64 = (A64.T if ta else A64), (B64.T if tb else B64)
    _close(C, A64 @ B64, np.abs(A64) @ np.abs(B64), f"m={m} n={n} k={k} ta={ta} tb={tb}", rtol=1e-6)


@pytest.mark.parametrize("tb", [False, True])
@pytest.mark.parametrize("m,n,k,ta", [(70_000, 200, 40, False), (60_000, 47, 33, False), (66_000, 16, 50, False), (200, 140, 30_011, True),
                                      (130, 60, 2_000, True), (100, 20, 5_003, True), (100, 100, 3_000, True), (64, 64, 2_048, False)])
def test_matmul_of_operands_outside_the_split(m, n, k, ta, tb):
    """Infinities, NaNs and values from 2^112 on have no exact three parts: the tiles they take part in are computed from the operands
    as they are."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(m + n + k)
    A = torch.empty(k if ta else m, m if ta else k, device=DEV).normal_(generator=gen)
    B = torch.empty(k, n, device=DEV).normal_(generator=gen)
    flat = A.view(-1)
    flat[17], flat[1000], flat[-3], flat[-1] = float("inf"), float("nan"), -float("inf"), 3.4e38
    rows = A.t() if ta else A
    rows[5] = 0.0          # a row of zeros stays zero
    rows[7] *= 2.0 ** -118
    B[k // 2, n // 2] = 0.0
    need = gnn.gnn_matmul_workspace_bytes(m, n, k)
    ws = torch.empty(max(need // 4, 4), device=DEV)
    C = torch.empty(m, n, device=DEV)
    gnn.gnn_matmul(A, B.t().contiguous() if tb else B, C, trans_a=ta, trans_b=tb, workspace=ws)
    torch.cuda.synchronize()
    a64, b64 = rows.double(), B.double()
    ref = torch.cat([a64[i:i + 4096].contiguous() @ b64 for i in range(0, m, 4096)])
    S = torch.cat([a64[i:i + 4096].abs().contiguous() @ b64.abs() for i in range(0, m, 4096)])
    ref32 = ref.float()
    odd = ~torch.isfinite(ref32)
    # where a sum passes the largest float on its way depends on its order: 3.4e38 is one operand of it
    near = (S > 1e37) & ~odd
    assert torch.equal(torch.isnan(C) & ~near, torch.isnan(ref32) & ~near)
    assert torch.equal(C[odd & ~torch.isnan(ref32)], ref32[odd & ~torch.isnan(ref32)])
    good = ~odd & ~near
    assert good.any()
    err = (C.double() - ref).abs()[good]
    assert bool((err <= 2e-5 * S[good] + 2.0 ** -148).all())
    assert bool((C[5][good[5]] == 0).all())


@pytest.mark.parametrize("m,n,k,ta", [(64, 64, 64, False), (300, 47, 100, False), (300, 130, 33, False), (130, 33, 9, False), (70, 65, 9, True),
                                      (66_000, 16, 20, False), (96, 140, 64, True), (130, 60, 2_048, True), (64, 64, 2_048, False)])
@pytest.mark.parametrize("tb", [False, True])
def test_matmul_of_tiny_operands_beside_large_ones(m, n, k, ta, tb):
    """Every magnitude of a float in either operand, subnormal ones included, against every magnitude of the other; results on both
    sides of 2^96, where the sums of scaled products end.  The error of a product is 3 * 2^-26 (the partial products left out), that of
    a chain of k additions k * 2^-24, of the sum of absolute terms; a split reduction has parts of 128 and 16 of them here."""
    if ta and tb:
        tb = False  # the remaining layout of a weight gradient
    rng = np.random.default_rng(17 * m + n + k)
    A = rng.normal(size=(m, k)) * 2.0 ** rng.integers(-145, 118, size=(m, 1))
    B = rng.normal(size=(k, n)) * 2.0 ** rng.integers(-145, 118, size=(1, n))
    A[:, ::5] *= 2.0 ** -20  # and different ones within a row
    A[3], B[:, 3] = rng.normal(size=k) * 2.0 ** -136, rng.normal(size=k) * 2.0 ** 110
    A, B = A.astype(np.float32), B.astype(np.float32)
    Ad = torch.from_numpy(np.ascontiguousarray(A.T) if ta else A).to(DEV)
    Bd = torch.from_numpy(np.ascontiguousarray(B.T) if tb else B).to(DEV)
    ws = torch.empty(max(gnn.gnn_matmul_workspace_bytes(m, n, k) // 4, 4), device=DEV)
    C = torch.empty(m, n, device=DEV)
    gnn.gnn_matmul(Ad, Bd, C, ta, tb, workspace=ws)
    torch.cuda.synchronize()
    A64, B64 = A.astype(np.float64), B.astype(np.float64)
    ref, S = A64 @ B64, np.abs(A64) @ np.abs(B64)
    fits = S < 2.0 ** 127  # no order of the additions passes the largest float
    got = C.cpu().numpy().astype(np.float64)
    assert np.isfinite(got[fits]).all()
    # subnormal sums: each addition rounds to a multiple of 2^-149 (the tiles of results above 2^96 are one chain of k)
    bound = (min(k, 128 + 16) + 1) * 2.0 ** -24 * S + k * 2.0 ** -149
    err = np.abs(got - ref)
    bad = fits & (err > bound)
    worst = np.unravel_index(np.argmax(np.where(fits, err / bound, 0)), err.shape)
    assert not bad.any(), f"{bad.sum()} of {bad.size}, worst {worst}: {got[worst]!r} for {ref[worst]!r}, S {S[worst]!r}"
    for lo, hi in ((0.0, 2.0 ** -100), (2.0 ** -100, 2.0 ** 90), (2.0 ** 90, 2.0 ** 100), (2.0 ** 100, 2.0 ** 127)):
        assert ((S > lo) & (S < hi)).any()


@pytest.mark.parametrize("k", [5, 16, 40])
def test_matmul_of_sums_that_cancel_where_scaled_products_overflow(k):
    """Products of 2^94 to 2^126 of both signs whose sums are small or cancel: no step may lose an overflow."""
    rng = np.random.default_rng(k)
    m, n = 256, 64
    A = rng.normal(size=(m, k)) * 2.0 ** rng.integers(47, 60, size=(m, 1))
    B = rng.normal(size=(k, n)) * 2.0 ** rng.integers(47, 60, size=(1, n))
    A[:, k // 2:2 * (k // 2)] = A[:, :k // 2]
    B[k // 2:2 * (k // 2)] = -B[:k // 2] * (1 + 2.0 ** -12)
    A, B = A.astype(np.float32), B.astype(np.float32)
    C = torch.empty(m, n, device=DEV)
    gnn.gnn_matmul(torch.from_numpy(A).to(DEV), torch.from_numpy(B).to(DEV), C)
    torch.cuda.synchronize()
    A64, B64 = A.astype(np.float64), B.astype(np.float64)
    err, S = np.abs(C.cpu().numpy().astype(np.float64) - A64 @ B64), np.abs(A64) @ np.abs(B64)
    assert S.max() < 2.0 ** 127 and (err <= (k + 1) * 2.0 ** -24 * S).all()


@pytest.mark.parametrize("m,n", [(33, 31), (300, 130), (2048, 256)])
@pytest.mark.parametrize("tb", [False, True])
def test_matmul_of_one_or_two_products_rounds_as_fp32_does(m, n, tb):
    """One product is rounded once, to half a last bit; two are one product and one multiply-add, half a last bit each."""
    rng = np.random.default_rng(m + n)
    for k in (1, 2):
        A = rng.normal(size=(m, k)).astype(np.float32)
        B = rng.normal(size=(n, k) if tb else (k, n)).astype(np.float32)
        C = torch.empty(m, n, device=DEV)
        gnn.gnn_matmul(torch.from_numpy(A).to(DEV), torch.from_numpy(B).to(DEV), C, False, tb)
        torch.cuda.synchronize()
        A64, B64 = A.astype(np.float64), B.astype(np.float64).T if tb else B.astype(np.float64)
        err, S = np.abs(C.cpu().numpy().astype(np.float64) - A64 @ B64), np.abs(A64) @ np.abs(B64)
        assert (err <= k * 2.0 ** -24 * S).all(), (k, (err / S).max() * 2 ** 24)


@pytest.mark.parametrize("m,n,k", [(602, 256, 100_000), (2000, 2560, 10_000), (3000, 3000, 10_000), (1500, 1500, 4_000)])
def test_matmul_parts_of_long_reductions_are_short_enough(m, n, k):
    """Weight gradients of 5, 160, 288 and 72 tiles (128 x 256): as many parts as make two workgroups per compute unit, or as close a result.
    Square of the relative 2-norm error of normal operands: 0.3e-14 + 0.0021e-14 per row of a part as measured from 128 rows
    to 50,000; the bound takes a seventh more."""
    gen = torch.Generator(device=DEV).manual_seed(m)
    a, b = (torch.empty(k, cols, device=DEV).normal_(generator=gen) for cols in (m, n))
    work = torch.empty(gnn.gnn_matmul_workspace_bytes(m, n, k) // 4, device=DEV)
    c = torch.empty(m, n, device=DEV)
    gnn.gnn_matmul(a, b, c, trans_a=True, workspace=work)
    want = a.double().t().contiguous() @ b.double()
    parts = -(-512 // (-(-m // 128) * -(-n // 256)))
    assert float((c.double() - want).norm() / want.norm()) <= 1e-7 * (8 / 7 * (0.3 + 0.0021 * k / parts)) ** 0.5
