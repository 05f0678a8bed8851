"""Hub rows whose pieces are added by the wavefront that is done last: rows of one piece and of many, at the turns of the loop
over pieces, over column slices, repeated calls and replays (the counters of done pieces have to be back at zero), and
beside calls with scratch of the caller's, where a kernel of its own adds the pieces."""
import numpy as np
import pytest
import torch

import oracle
import paper_2104_06700_amd as gnn
import synth
from helpers import OP_CODE, assert_close, device_graph, host_csr

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
CHUNK = 6


def _graph():
    """Hub rows (of 5 edges and more) of 1, 2, 3, 4, 5, 8, 9 and 40 pieces of 6 edges, whole and not."""
    n = 300
    lengths = [5, 6, 7, 12, 13, 18, 23, 24, 25, 30, 48, 49, 54, 239]
    dst = torch.cat([torch.full((k,), 17 * i + 3, dtype=torch.int64) for i, k in enumerate(lengths)] + [torch.arange(n).repeat_interleave(2)])
    src = (synth.mix64(torch.arange(dst.numel()) + 5) & 0x7FFFFFFF) % n
    key = torch.sort(dst * n + src).values
    return synth.EdgeList(n=n, src=(key % n).to(torch.int32), dst=(key // n).to(torch.int32), meta={})


@pytest.mark.parametrize("thresholds", [[5], []])  # without thresholds all rows are hub rows
@pytest.mark.parametrize("dtype,f", [(torch.float32, 3), (torch.float32, 100), (torch.float32, 290), (torch.bfloat16, 66), (torch.bfloat16, 530)])
def test_sums_of_hub_rows(thresholds, dtype, f):
    el = _graph()
    indptr, indices, *_ = host_csr(el)
    dg = device_graph(el, plan_params=gnn.make_plan_params(thresholds, CHUNK))
    bf16 = dtype == torch.bfloat16
    own_scratch = torch.empty(dg.plan_fwd.workspace_bytes(f) // 4 + 4, device=DEV)
    for seed, flags in ((1, 0), (2, gnn.GNN_FLAG_FORCE_PADDED_COPY), (3, gnn.GNN_FLAG_NO_COLUMN_SLICES)):
        X = synth.normal_features(el.n, f, seed, dtype=dtype)
        Xd = X.to(DEV)
        for op_name in ("sage", "mean"):
            op = OP_CODE[op_name]
            Yo, S = oracle.aggregate_fwd(indptr, indices, X.float().numpy(), op=op, want_scale=True)
            Y, Yw = torch.full_like(Xd, float("nan")), torch.full_like(Xd, float("nan"))
            gnn.gnn_aggregate_fwd(dg.indptr, dg.indices, None, Xd, Y, el.n, f, op, plan=dg.plan_fwd, flags=flags)
            gnn.gnn_aggregate_fwd(dg.indptr, dg.indices, None, Xd, Yw, el.n, f, op, plan=dg.plan_fwd, flags=flags, workspace=own_scratch)
            torch.cuda.synchronize()
            assert_close(Y, Yo, S, bf16, f"{op_name} F={f} flags={flags}")
            assert torch.equal(Y, Yw), "the pieces are added in order either way"


@pytest.mark.parametrize("d", [3, 33, 100, 2100])  # 2,100 columns: more column slabs than there are counters
def test_operator_table_on_hub_rows(d):
    el = _graph()
    indptr, indices, *_ = host_csr(el)
    dg = device_graph(el, plan_params=gnn.make_plan_params([5], CHUNK))
    V, E = synth.normal_features(el.n, d, 3), synth.normal_features(el.e, d, 4)
    V[::3] = 0.25  # ties
    args = dict(plan=dg.plan_fwd)
    for _ in range(2):
        O, A = torch.full((el.n, d), float("nan"), device=DEV), torch.full((el.n, d), -7, dtype=torch.int32, device=DEV)
        gnn.gnn_ap_fwd(dg.indptr, dg.indices, V.to(DEV), None, O, A, el.n, d, gnn.GNN_BIN_COPY_LHS, gnn.GNN_RED_MAX, **args)
        M = torch.full((el.n, d), float("nan"), device=DEV)
        gnn.gnn_ap_fwd(dg.indptr, dg.indices, V.to(DEV), E.to(DEV), M, None, el.n, d, gnn.GNN_BIN_MUL, gnn.GNN_RED_SUM, **args)
        torch.cuda.synchronize()
        msgs = V.numpy()[indices]
        prod = msgs.astype(np.float64) * E.numpy().astype(np.float64)
        for v in range(el.n):
            b, e = int(indptr[v]), int(indptr[v + 1])
            if b == e:
                continue
            win = msgs[b:e].argmax(axis=0)  # the lowest position among equals
            assert np.array_equal(A[v].cpu().numpy(), b + win), v
            assert np.array_equal(O[v].cpu().numpy(), msgs[b:e].max(axis=0)), v
            err = np.abs(M[v].cpu().numpy() - prod[b:e].sum(axis=0))
            assert (err <= 1e-5 * np.abs(prod[b:e]).sum(axis=0)).all(), v


def test_replays_leave_the_counters_at_zero():
    el = _graph()
    f = 100
    dg = device_graph(el, plan_params=gnn.make_plan_params([5], CHUNK))
    X = synth.normal_features(el.n, f, 8).to(DEV)
    Y = torch.empty_like(X)
    dg.plan_fwd.prepare(dg.indices, gnn.GNN_MEAN, False, f)
    call = lambda out: gnn.gnn_aggregate_fwd(dg.indptr, dg.indices, None, X, out, el.n, f, gnn.GNN_MEAN, plan=dg.plan_fwd)  # noqa: E731
    call(Y)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(Y)
    for seed in range(4):
        X.copy_(synth.normal_features(el.n, f, 20 + seed))
        Y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        eager = torch.full_like(Y, float("nan"))
        call(eager)
        torch.cuda.synchronize()
        assert torch.equal(Y, eager)
