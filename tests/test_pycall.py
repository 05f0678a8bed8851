"""The extension module that marshals the hot calls: argument checks that return before any device work."""
import os
import subprocess
import sys

import pytest
import torch

import paper_2104_06700_amd as gnn

I32 = torch.zeros(6, dtype=torch.int32)
X = torch.zeros(5, 4)


def _aggregate(indptr=I32, indices=I32, w=None, x=X, y=X, n=0, f=4, op=gnn.GNN_SUM, **kw):
    gnn.gnn_aggregate_fwd(indptr, indices, w, x, y, n, f, op, stream=0, **kw)


def test_calls_without_work_succeed():
    _aggregate()
    _aggregate(indptr=I32.long(), x=X.bfloat16(), y=X.bfloat16(), w=torch.zeros(3))
    gnn.gnn_aggregate_bwd(I32, I32, None, X, X, 0, 4, gnn.GNN_MEAN, stream=0)
    _aggregate(n=False, f=torch.tensor(4), flags=True)  # anything that int() takes


@pytest.mark.parametrize("kw,error", [
    (dict(y=X.double()), TypeError), (dict(x=X.half(), y=X.half()), TypeError), (dict(indptr=I32.float()), TypeError),
    (dict(indices=torch.zeros(12, dtype=torch.int32)[::2]), ValueError), (dict(w=torch.zeros(12)[::3]), ValueError),
    (dict(n=-1), gnn.GnnError), (dict(op=77), gnn.GnnError), (dict(n=5, ldx=3), gnn.GnnError), (dict(n=5, x=X[:, :2]), gnn.GnnError),
    (dict(n="five"), ValueError), (dict(x=None), AttributeError),
])
def test_rejected_arguments_of_the_aggregation(kw, error):
    with pytest.raises(error):
        _aggregate(**{"n": 5, **kw} if "op" in kw else kw)


def test_rejected_arguments_of_the_operator_table_and_the_layers():
    def fwd(fv=X, fe=None, fo=X, arg=None, ids=None):
        gnn.gnn_ap_fwd(I32, I32, fv, fe, fo, arg, 0, 4, gnn.GNN_BIN_COPY_LHS, gnn.GNN_RED_SUM, edge_ids=ids, stream=0)
    fwd()
    fwd(fe=torch.zeros(7))
    for bad in (dict(fv=X.double()), dict(fe=X.bfloat16()), dict(arg=I32.long()), dict(arg=torch.zeros(4, 5, dtype=torch.int32).t()),
                dict(ids=I32)):
        with pytest.raises(TypeError):
            fwd(**bad)
    with pytest.raises(ValueError):
        fwd(fv=torch.zeros(4, 5).t())
    w = torch.zeros(4, 3)
    with pytest.raises(ValueError):
        gnn.gnn_sage_layer_fwd(I32, I32, torch.zeros(4, 5).t(), w, torch.zeros(3), X, X, None, stream=0)
    with pytest.raises(TypeError):
        gnn.gnn_sage_layer_fwd(I32, I32, X.double(), w, torch.zeros(3), X, X, None, stream=0)
    with pytest.raises(gnn.GnnError):  # a layer needs a plan
        gnn.gnn_sage_layer_fwd(I32, I32, X, w, torch.zeros(3), X, X, None, stream=0)


def test_without_the_extension_module_the_library_loads_and_only_its_calls_fail():
    code = ("import sys; sys.modules['paper_2104_06700_amd._pycall'] = None\n"
            "import torch, paper_2104_06700_amd as gnn\n"
            "assert gnn.gnn_matmul_workspace_bytes(4, 4, 4) == 0 and gnn.status_string(0) == 'ok'\n"
            "t = torch.zeros(4, 4)\n"
            "try:\n"
            "    gnn.gnn_aggregate_fwd(t.int(), t.int(), None, t, t, 0, 4, gnn.GNN_SUM, stream=0)\n"
            "except ImportError as err:\n"
            "    assert '_pycall is missing' in str(err)\n"
            "else:\n"
            "    raise SystemExit('no error')\n")
    subprocess.run([sys.executable, "-c", code], check=True, cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
