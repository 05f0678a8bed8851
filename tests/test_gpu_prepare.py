"""gnn_plan_prepare reserves what the calls take, whether they come without weights, with bound or with other ones: the first
call after it allocates nothing, and can be captured."""
import pytest
import torch

import paper_2104_06700_amd as gnn
import synth

pytestmark = pytest.mark.gpu


# the sizes lie where calls with and without weights choose differently: a copy for coefficients only, in rows of several lines
# and of one; a copy only without them, and hints for cold sources with them; pieces asked for, whose tiles take coefficients
CASES = [
    dict(n=100000, e=6000000, f=100), dict(n=60000, e=6000000, f=100, op=gnn.GNN_MEAN), dict(n=200000, e=8000000, f=20),
    dict(n=1400000, e=33000000, f=64), dict(n=20000, e=4000000, f=512, blocking=dict(min_degree=32)),
    dict(n=20000, e=4000000, f=1000, blocking=dict(min_degree=32), dtype=torch.bfloat16, op=gnn.GNN_MEAN, backward=True, bound=True),
    dict(n=150000, e=30000000, f=20, bound=True),
]


@pytest.mark.parametrize("case,weights", [(c, w) for c in CASES for w in ("none", "bound", "other") if w != "bound" or c.get("bound")],
                         ids=lambda v: v if isinstance(v, str) else f"{v['n']}-{v['e']}-{v['f']}")
def test_nothing_is_allocated_after_prepare(case, weights):
    f, op, backward, dtype = case["f"], case.get("op", gnn.GNN_SUM), case.get("backward", False), case.get("dtype", torch.float32)
    el = synth.rmat_directed(case["n"], case["e"], (0.57, 0.19, 0.19, 0.05), 3, device="cuda")
    n, e = el.n, el.e
    w = torch.rand(e, device="cuda") + 0.5
    passed = None if weights == "none" else (w if weights == "bound" else w.clone())
    x = torch.randn(n, f, device="cuda").to(dtype)
    y = torch.empty_like(x)
    fn = gnn.gnn_aggregate_bwd if backward else gnn.gnn_aggregate_fwd
    for first in (True, False):  # with the first plan the call also loads its kernels
        g = gnn.build_device_graph(el.dst, el.src, n)
        plan, indptr, indices = (g.plan_bwd, g.indptr_t, g.indices_t) if backward else (g.plan_fwd, g.indptr, g.indices)
        if "blocking" in case:
            plan.set_blocking(**case["blocking"])
        if case.get("bound"):
            plan.bind_edge_weights(w)
        plan.prepare(indices, op, backward, f, dtype)
        torch.cuda.synchronize()
        gnn.gnn_release_cached_memory()  # so that an allocation has to come from the driver
        free = torch.cuda.mem_get_info()[0]
        fn(indptr, indices, passed, x, y, n, f, op, plan=plan)
        torch.cuda.synchronize()
        assert first or torch.cuda.mem_get_info()[0] == free

    captured = torch.empty_like(y)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        fn(indptr, indices, passed, x, captured, n, f, op, plan=plan)
    for _ in range(3):
        captured.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(captured, y)
