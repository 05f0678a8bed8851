"""Edge gradients whose rows leave through LDS as whole lines, and sums that read f_E non-temporally: both only apply to arrays
beyond the caches, so the graphs here have few vertices and wide rows.  Every element is compared with the product of its own
operands, one correctly rounded fp32 operation, exactly; what lies around the array must stay as it was."""
import pytest
import torch

import paper_2104_06700_amd as gnn
import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _graph(n, e, seed=3):
    """Rows of every length class beside R-MAT ones: none, 1, the turns of 4, 16 and 64 edges, and hub rows."""
    el = synth.rmat_symmetric(n, e, (0.57, 0.19, 0.19, 0.05), seed, device=DEV)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    dst, src = [el.dst.long()], [el.src.long()]
    for i, k in enumerate([1, 3, 4, 5, 15, 16, 17, 63, 64, 65, 255, 4097, 9000]):
        dst.append(torch.full((k,), 7 * i, device=DEV))
        src.append(torch.randint(0, n, (k,), device=DEV, generator=gen))
    dst, src = torch.cat(dst), torch.cat(src)
    order = torch.argsort(dst * n + src)
    return gnn.build_device_graph(dst[order].int(), src[order].int(), n, want_perm=True), dst[order], src[order]


# widths at the edges of strips (4 columns) and lines (16), powers of two and not, up to the largest that is staged
@pytest.mark.parametrize("n,e,d,binop", [(60000, 5400000, 13, "mul"), (60000, 4200000, 16, "mul"), (60000, 2100000, 33, "mul"), (60000, 1100000, 61, "mul"),
                                         (60000, 1100000, 64, "mul"), (60000, 500000, 255, "mul"), (60000, 500000, 256, "mul"), (60000, 5200000, 19, "add"),
                                         (60000, 3000000, 33, "sub"), (60000, 1500000, 65, "copyrhs")])
@pytest.mark.parametrize("shift", [0, 3])  # floats behind an aligned address
def test_rows_of_the_edge_gradient(n, e, d, binop, shift):
    g, dst, src = _graph(n, e)
    E = dst.numel()
    gen = torch.Generator(device=DEV)
    gen.manual_seed(d)
    v, do = (torch.empty(n, d, device=DEV).normal_(generator=gen) for _ in range(2))
    v[5::97] = float("inf")
    do[11::101] = 0.0
    room = torch.full((E * d + 64,), 7.0, device=DEV)
    out = room[16 + shift:16 + shift + E * d].view(E, d)
    fe = room[:E * d].view(E, d) if binop != "mul" else torch.zeros(1, device=DEV).expand(E, d)  # the gradients read no f_E
    code = dict(add=gnn.GNN_BIN_ADD, sub=gnn.GNN_BIN_SUB, mul=gnn.GNN_BIN_MUL, copyrhs=gnn.GNN_BIN_COPY_RHS)[binop]
    gnn.gnn_ap_bwd_edge(g.indptr, g.indices, None, None if binop == "copyrhs" else v, None, do, out, n, d, code, plan=g.plan_fwd)
    torch.cuda.synchronize()
    assert bool((room[:16 + shift] == 7.0).all()) and bool((room[16 + shift + E * d:] == 7.0).all()), "written outside the rows"
    step = 1 << 18
    for b in range(0, E, step):
        want = do[dst[b:b + step]]
        want = want * v[src[b:b + step]] if binop == "mul" else (-want if binop == "sub" else want)
        assert torch.equal(torch.nan_to_num(out[b:b + step], nan=123.0), torch.nan_to_num(want, nan=123.0)), f"rows {b} ..."


def test_streamed_sums():
    n, e, d = 30000, 5000000, 61  # 1.2 GB of f_E
    g, dst, src = _graph(n, e)
    E = dst.numel()
    assert E * d * 4 >= 1200000000
    gen = torch.Generator(device=DEV)
    gen.manual_seed(d)
    v = torch.empty(n, d, device=DEV).normal_(generator=gen)
    fe = torch.empty(E, d, device=DEV).normal_(generator=gen)
    out, dv = torch.empty_like(v), torch.empty_like(v)
    gnn.gnn_ap_fwd(g.indptr, g.indices, v, fe, out, None, n, d, gnn.GNN_BIN_MUL, gnn.GNN_RED_SUM, plan=g.plan_fwd)
    gnn.gnn_ap_bwd_vertex(g.indptr_t, g.indices_t, v, fe, dv, n, d, gnn.GNN_BIN_MUL, plan=g.plan_bwd, edge_ids=g.perm)
    torch.cuda.synchronize()
    for got, to, frm in ((out, dst, src), (dv, src, dst)):
        want, scale = (torch.zeros(n, d, dtype=torch.float64, device=DEV) for _ in range(2))
        for b in range(0, E, 1 << 20):
            m = v[frm[b:b + (1 << 20)]].double() * fe[b:b + (1 << 20)].double()
            want.index_add_(0, to[b:b + (1 << 20)], m)
            scale.index_add_(0, to[b:b + (1 << 20)], m.abs())
        assert bool(((got.double() - want).abs() <= 1e-5 * scale).all())
