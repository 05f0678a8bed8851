"""Where the choice between gathering in place, from the plan's copy and with pieces changes sides, the sides agree: sizes one
percent below and above the lines of gnn_choose_layout, against the call that stays in place."""
import pytest
import torch

import paper_2104_06700_amd as gnn
import synth

pytestmark = pytest.mark.gpu

IN_PLACE = gnn.GNN_FLAG_NO_PADDED_COPY | gnn.GNN_FLAG_NO_SOURCE_BLOCKS
F32, BF16 = torch.float32, torch.bfloat16
# vertices, edges at the line, width, type, weights, backward (whose rows carry a factor)
LINES = [
    (100000, 25.0e6, 50, F32, False, False), (100000, 8.5e6, 50, F32, True, False), (100000, 8.5e6, 50, F32, False, True),
    (140000, 10.0e6, 50, F32, False, False), (140000, 8.5e6, 50, F32, False, True), (100000, 25.0e6, 100, BF16, False, False),
    (300000, 15.625e6, 64, F32, False, False), (320000, 5.0e6 * 1.024, 256, F32, False, True),
    (200000, 10.0e6, 20, F32, False, False), (200000, 0.7e9 / 128, 20, F32, True, False),
    (200000, 24.0e6, 8, F32, False, False), (200000, 28.0e6, 16, F32, False, False), (200000, 32.0e6, 32, F32, False, False),
]


@pytest.mark.parametrize("n,line,f,dtype,weights,backward", LINES)
def test_both_sides_agree(n, line, f, dtype, weights, backward):
    for e in (int(line * 0.99) // 2 * 2, int(line * 1.01) // 2 * 2):
        el = synth.rmat_symmetric(n, e, (0.57, 0.19, 0.19, 0.05), 9, device="cuda")
        w = torch.rand(e, device="cuda") + 0.5 if weights else None
        g = gnn.build_device_graph(el.dst, el.src, n, edge_w=w)
        del el
        x = torch.randn(n, f, device="cuda").to(dtype)
        op = gnn.GNN_MEAN if backward else gnn.GNN_SUM

        def call(x, flags):
            y = torch.full_like(x, float("nan"))
            if backward:
                gnn.gnn_aggregate_bwd(g.indptr_t, g.indices_t, g.edge_w_t, x, y, n, f, op, plan=g.plan_bwd, flags=flags)
            else:
                gnn.gnn_aggregate_fwd(g.indptr, g.indices, g.edge_w, x, y, n, f, op, plan=g.plan_fwd, flags=flags)
            return y.double()

        size = call(x.abs(), IN_PLACE)
        # fp32 sums in two orders; bf16 results are rounded once more on either side, to 2^-9 of the value
        bound = (2 ** -8 if dtype == BF16 else 1e-5) * size
        assert bool(((call(x, 0) - call(x, IN_PLACE)).abs() <= bound).all()), e
