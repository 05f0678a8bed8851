"""The one-call graph setup against a stable sort on the host and against the separate calls, at the edges of the sort's
tiles (4096 pairs) and digits (8 bits); blocks of destroyed plans in use again, on another stream too."""
import threading

import numpy as np
import pytest
import torch

import paper_2104_06700_amd as gnn

pytestmark = pytest.mark.gpu


def _edges(n, e, seed):
    rng = np.random.default_rng(seed)
    src = np.minimum((n * rng.random(e) ** 3).astype(np.int64), n - 1)  # some sources far more frequent than others
    dst = np.sort(rng.integers(0, n, e))
    if e > 20:
        dst[: e // 2] = dst[e // 2]  # a long row
        dst.sort()
    order = np.lexsort((src, dst))
    return dst[order].astype(np.int32), src[order].astype(np.int32)


@pytest.mark.parametrize("indptr64", [False, True])
@pytest.mark.parametrize("weights", [False, True])
@pytest.mark.parametrize("n,e", [(1, 0), (5, 0), (1, 1), (200, 63), (256, 4095), (257, 4096), (3000, 4097), (70000, 40961),
                                 (17, 300000), (131073, 524288)])
def test_graph_build(n, e, weights, indptr64):
    dst, src = _edges(n, e, n + e)
    d, s = torch.from_numpy(dst).cuda(), torch.from_numpy(src).cuda()
    w = torch.rand(e, device="cuda") if weights else None
    for _ in range(2):  # the second time from the blocks of the first
        g = gnn.build_device_graph(d, s, n, edge_w=w, indptr64=indptr64, want_perm=weights)
        perm = np.argsort(src, kind="stable")
        bounds = np.arange(n + 1)
        assert np.array_equal(g.indptr.cpu().numpy(), np.searchsorted(dst, bounds, side="left"))
        assert np.array_equal(g.indptr_t.cpu().numpy(), np.searchsorted(src[perm], bounds, side="left"))
        assert np.array_equal(g.indices_t.cpu().numpy(), dst[perm])
        if weights:
            assert np.array_equal(g.perm.cpu().numpy(), perm)
            assert torch.equal(g.edge_w_t.cpu(), w.cpu()[torch.from_numpy(perm)])
        for plan, indptr, indices in ((g.plan_fwd, g.indptr, g.indices), (g.plan_bwd, g.indptr_t, g.indices_t)):
            alone = gnn.gnn_plan_create(indptr, indices, n)
            for a, b in zip(plan.export(), alone.export()):
                assert np.array_equal(a, b)
            for k in (1, 7, n):
                assert plan.gather_share(k) == alone.gather_share(k)
        del g, plan, alone


def test_blocks_move_between_streams():
    """Plans dropped with their work still running, and the next ones built on another stream from the same blocks."""
    n, e, f = 20000, 400000, 40
    dst, src = _edges(n, e, 3)
    d, s = torch.from_numpy(dst).cuda(), torch.from_numpy(src).cuda()
    x = torch.randn(n, f, device="cuda")
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    ys = []
    for i in range(6):
        with torch.cuda.stream(side if i % 2 else torch.cuda.default_stream()):
            g = gnn.build_device_graph(d, s, n)
            y = torch.empty_like(x)
            gnn.gnn_aggregate_fwd(g.indptr, g.indices, None, x, y, n, f, gnn.GNN_MEAN, plan=g.plan_fwd)
            ys.append(y)
            if i < 5:
                del g
    torch.cuda.synchronize()
    for y in ys[1:]:
        assert torch.equal(ys[0], y)
    gnn.gnn_release_cached_memory()
    y = torch.empty_like(x)
    gnn.gnn_aggregate_fwd(g.indptr, g.indices, None, x, y, n, f, gnn.GNN_MEAN, plan=g.plan_fwd)
    assert torch.equal(ys[0], y)


def test_two_threads_share_the_pool():
    """Graphs are built, used and dropped by two threads on a stream each; either may get the blocks of the other."""
    n, e, f = 140000, 2400000, 32  # the gradient of the winners is sorted, with scratch from the pool
    problems, errors = [], []
    for i in range(2):
        dst, src = (torch.from_numpy(a).cuda() for a in _edges(n, e, 11 + i))
        x = torch.randn(n, f, device="cuda")
        arg = torch.randint(-1, e, (n, f), device="cuda", dtype=torch.int32)
        u = src[arg.clamp(min=0).long()].long()
        g = torch.where(arg >= 0, x.double(), torch.zeros((), dtype=torch.float64, device="cuda"))
        grad, mag = (torch.zeros(n, f, dtype=torch.float64, device="cuda").scatter_add_(0, u, t) for t in (g, g.abs()))
        problems.append((dst, src, x, arg, grad, mag))
    torch.cuda.synchronize()

    def work(problem):
        try:
            dst, src, x, arg, grad, mag = problem
            first = None
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(6):
                    g = gnn.build_device_graph(dst, src, n)
                    y, dv = torch.empty_like(x), torch.empty_like(x)
                    gnn.gnn_aggregate_fwd(g.indptr, g.indices, None, x, y, n, f, gnn.GNN_MEAN, plan=g.plan_fwd)
                    gnn.gnn_ap_bwd_vertex_arg(g.indices, arg, x, None, dv, n, n, f, gnn.GNN_BIN_COPY_LHS)
                    del g
                    assert bool(((dv.double() - grad).abs() <= 1e-5 * mag).all())
                    first = y if first is None else first
                    assert torch.equal(first, y)
        except BaseException as err:
            errors.append(err)

    threads = [threading.Thread(target=work, args=(p,)) for p in problems]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not errors, errors
