"""Launches that leave most of the chip idle (more edge slots per row, long rows and hub pieces shared by the wavefronts of
a workgroup) and rows of any width, stride and alignment (16-byte loads at the alignment of an element, the last strip
of a row beginning early enough to end with it), against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2104_06700_amd as gnn
import synth
from helpers import OP_CODE, assert_close, device_graph, host_csr

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _graph():
    """Rows of every length class up to a hub of 6,000 edges (duplicates allowed)."""
    n = 700
    lengths = [0, 1, 3, 4, 5, 15, 31, 63, 64, 255, 256, 257, 1023, 1025, 4095, 6000]
    dst = torch.cat([torch.full((k,), 11 * i + 2, dtype=torch.int64) for i, k in enumerate(lengths)] +
                    [torch.arange(n).repeat_interleave(7)])
    src = (synth.mix64(torch.arange(dst.numel()) + 99) & 0x7FFFFFFF) % n
    key = torch.sort(dst * n + src).values
    return synth.EdgeList(n=n, src=(key % n).to(torch.int32), dst=(key // n).to(torch.int32), meta={})


@pytest.mark.parametrize("dtype,widths", [(torch.float32, (1, 2, 3, 4, 5, 7, 33, 64, 99, 257, 515)),
                                          (torch.bfloat16, (1, 3, 7, 8, 9, 33, 65, 130, 515, 1031))])
@pytest.mark.parametrize("op_name,weights", [("sage", False), ("mean", True), ("gcn", False)])
def test_rows_of_every_length_width_and_alignment(dtype, widths, op_name, weights):
    el = _graph()
    bf16 = dtype == torch.bfloat16
    indptr, indices, indptr_t, indices_t, perm = host_csr(el)
    din, dout = np.diff(indptr), np.diff(indptr_t)
    wts = (synth.uniform_features(el.e, 1, 7).reshape(-1) + 0.5) if weights else None
    w = None if wts is None else wts.numpy()
    dg = device_graph(el, weights=wts)
    op = OP_CODE[op_name]
    for f in widths:
        X = synth.normal_features(el.n, f, 3, dtype=dtype)
        Yo, S = oracle.aggregate_fwd(indptr, indices, X.float().numpy(), op=op, w=w, dout=dout, nthreads=8, want_scale=True)
        dXo, St = oracle.aggregate_bwd(indptr_t, indices_t, X.float().numpy(), op=op, wt=None if w is None else w[perm], din=din,
                                       nthreads=8, want_scale=True)
        for pad_in, pad_out, shift in ((0, 0, 0), (1, 3, 1), (0, 1, 3)):
            # exactly the elements that belong to the matrix, `shift` elements behind an aligned address
            flat = torch.full((el.n * (f + pad_in) + shift,), float("nan"), dtype=dtype, device=DEV)
            Xd = flat[shift:].view(el.n, f + pad_in)[:, :f]
            Xd.copy_(X)
            out = torch.full((2, el.n * (f + pad_out) + shift), 7.0, dtype=dtype, device=DEV)
            Y, dX = (o[shift:].view(el.n, f + pad_out) for o in out)
            gnn.gnn_aggregate_fwd(dg.indptr, dg.indices, dg.edge_w, Xd, Y[:, :f], el.n, f, op, plan=dg.plan_fwd)
            gnn.gnn_aggregate_bwd(dg.indptr_t, dg.indices_t, dg.edge_w_t, Xd, dX[:, :f], el.n, f, op, plan=dg.plan_bwd)
            torch.cuda.synchronize()
            assert_close(Y[:, :f], Yo, S, bf16, f"fwd F={f} pads {pad_in} {pad_out} shift {shift}")
            assert_close(dX[:, :f], dXo, St, bf16, f"bwd F={f} pads {pad_in} {pad_out} shift {shift}")
            assert bool((Y[:, f:] == 7.0).all()) and bool((dX[:, f:] == 7.0).all()) and bool((out[:, :shift] == 7.0).all()), "written outside the rows"


@pytest.mark.parametrize("d", [1, 3, 4, 5, 33, 66, 101])
@pytest.mark.parametrize("shift", [0, 1, 3])
def test_operator_table_on_rows_of_every_length_and_alignment(d, shift):
    """max with winners and the edge gradients (full width, and the dot products of a scalar operand), on operands that lie
    `shift` floats behind an aligned address with one column of padding."""
    el = _graph()
    indptr, indices, *_ = host_csr(el)
    dg = device_graph(el)
    fV, dO = synth.normal_features(el.n, d, 3), synth.normal_features(el.n, d, 4)

    def place(t):
        flat = torch.full((t.shape[0] * (t.shape[1] + 1) + shift,), float("nan"), device=DEV)
        out = flat[shift:].view(t.shape[0], t.shape[1] + 1)[:, :t.shape[1]]
        out.copy_(t)
        return out

    out = torch.full((el.n * d + shift,), float("nan"), device=DEV)
    fO = out[shift:].view(el.n, d)
    arg = torch.empty((el.n, d), dtype=torch.int32, device=DEV)
    gnn.gnn_ap_fwd(dg.indptr, dg.indices, place(fV), None, fO, arg, el.n, d, gnn.GNN_BIN_COPY_LHS, gnn.GNN_RED_MAX, plan=dg.plan_fwd)
    dfE = torch.full((el.e, d), float("nan"), device=DEV)
    dw = torch.full((el.e,), float("nan"), device=DEV)
    gnn.gnn_ap_bwd_edge(dg.indptr, dg.indices, None, place(fV), dfE, place(dO), dfE, el.n, d, gnn.GNN_BIN_MUL, plan=dg.plan_fwd)
    gnn.gnn_ap_bwd_edge(dg.indptr, dg.indices, None, place(fV), dw, place(dO), dw, el.n, d, gnn.GNN_BIN_MUL, plan=dg.plan_fwd)
    torch.cuda.synchronize()
    O, won = oracle.ap_fwd(indptr, indices, fV.numpy(), None, d, oracle.BIN_COPY_LHS, oracle.RED_MAX)
    assert np.array_equal(fO.cpu().numpy().astype(np.float64), O) and np.array_equal(arg.cpu().numpy().astype(np.int64), won)
    prod = dO.double()[el.dst.long()] * fV.double()[el.src.long()]
    assert torch.equal(dfE.cpu(), (dO[el.dst.long()] * fV[el.src.long()]))
    err = (dw.cpu().double() - prod.sum(1)).abs()
    assert bool((err <= 1e-5 * prod.abs().sum(1)).all())


@pytest.mark.parametrize("n,e,f,dtype", [(50000, 400000, 113, torch.float32), (50000, 200000, 163, torch.float32),
                                         (50000, 400000, 601, torch.bfloat16), (3000, 20000, 2051, torch.float32),
                                         (3000, 20000, 4099, torch.bfloat16), (20000, 300000, 101, torch.float32)])
def test_column_slices_of_rows_in_place(n, e, f, dtype):
    """Rows off line boundaries in slices of their own: a number of slices that is no power of two, a last one that is short
    or empty, and more of them than one launch takes."""
    el = synth.rmat_symmetric(n, e, (0.57, 0.19, 0.19, 0.05), 4)
    indptr, indices, indptr_t, indices_t, _ = host_csr(el)
    din, dout = np.diff(indptr), np.diff(indptr_t)
    X = synth.normal_features(el.n, f, 3, dtype=dtype)
    dg = device_graph(el)
    Yo, S = oracle.aggregate_fwd(indptr, indices, X.float().numpy(), op=oracle.OP_MEAN, dout=dout, nthreads=8, want_scale=True)
    dXo, St = oracle.aggregate_bwd(indptr_t, indices_t, X.float().numpy(), op=oracle.OP_MEAN, din=din, nthreads=8, want_scale=True)
    flat = torch.full((el.n * f + 1,), float("nan"), dtype=dtype, device=DEV)
    Xd = flat[1:].view(el.n, f)
    Xd.copy_(X)
    Y, dX = torch.full_like(Xd, float("nan")), torch.full_like(Xd, float("nan"))
    gnn.gnn_aggregate_fwd(dg.indptr, dg.indices, None, Xd, Y, el.n, f, gnn.GNN_MEAN, plan=dg.plan_fwd)
    gnn.gnn_aggregate_bwd(dg.indptr_t, dg.indices_t, None, Xd, dX, el.n, f, gnn.GNN_MEAN, plan=dg.plan_bwd)
    torch.cuda.synchronize()
    assert_close(Y, Yo, S, dtype == torch.bfloat16, "fwd")
    assert_close(dX, dXo, St, dtype == torch.bfloat16, "bwd")


@pytest.mark.parametrize("d", [4, 6, 8, 9, 12, 16, 17, 31, 32, 35, 63, 64, 67, 95, 96, 97, 127, 128, 129])
def test_dot_products_on_rows_of_every_length(d):
    """The gradient of a scalar edge operand where its strips per edge and lanes per edge change, with edge ids, and an
    infinite value that the strips of a ragged row may not count twice."""
    el = _graph()
    dg = device_graph(el)
    fV, dO = synth.normal_features(el.n, d, 3), synth.normal_features(el.n, d, 4)
    fV[5, d - 2] = float("inf")
    ids = torch.randperm(el.e, generator=torch.Generator().manual_seed(d))
    dw = torch.full((el.e + 1,), 7.0, device=DEV)
    gnn.gnn_ap_bwd_edge(dg.indptr, dg.indices, None, fV.to(DEV), dw[:el.e], dO.to(DEV), dw[:el.e], el.n, d, gnn.GNN_BIN_MUL,
                        plan=dg.plan_fwd, edge_ids=ids.to(DEV))
    torch.cuda.synchronize()
    prod = dO.double()[el.dst.long()] * fV.double()[el.src.long()]
    got, want = dw[:el.e].cpu().double()[ids], prod.sum(1)
    finite = torch.isfinite(want)
    assert torch.equal(got[~finite], want[~finite]) and int((~finite).sum()) > 0
    assert bool(((got - want).abs()[finite] <= 1e-5 * prod.abs().sum(1)[finite]).all()) and float(dw[el.e]) == 7.0
