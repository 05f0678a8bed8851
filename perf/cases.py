"""What the aggregation library is timed on: seeded synthetic graphs of the repository's own workloads and of
the ranges around them, through the public entry points, forward and backward.

A case is a dict of plain values.  "kind" names the program it stands for:
  aggregate   the aggregation stack of full-batch training: per width one forward and one backward call
  layers      a whole GraphSAGE model: the layer calls forward, then backward with every gradient
  pool        max / min pooling over the neighbours with the winners, and the gradient that goes to them
  attention   one scalar per edge that changes with every step: weighted sum, and the gradients of the
              vertices (over the transposed graph, through the edge permutation) and of the edge scalars
  messages    a full feature vector per edge: message, sum, and the gradients of vertices and edges
  sampled     mini-batch training on a new subgraph: row pointers, transposed graph and both plans are
              built, then used for one forward and one backward aggregation
Sizes: "n" vertices, "e" directed edges; "graph" is er (uniform), sym (R-MAT, both directions of every pair)
or dir (R-MAT, directed); "skew" picks the R-MAT probabilities; "widths" are the feature widths.
"""
from __future__ import annotations

import torch

import paper_2104_06700_amd as gnn
import synth

OPS = {"sum": gnn.GNN_SUM, "mean": gnn.GNN_MEAN, "gcn": gnn.GNN_GCN_SYM, "sage": gnn.GNN_SAGE_GCN}
BINOPS = {"add": gnn.GNN_BIN_ADD, "sub": gnn.GNN_BIN_SUB, "mul": gnn.GNN_BIN_MUL}
REDUCERS = {"max": gnn.GNN_RED_MAX, "min": gnn.GNN_RED_MIN}
PROBS = {"strong": (0.57, 0.19, 0.19, 0.05), "mild": (0.45, 0.22, 0.22, 0.11)}


def listed():
    return [
        # the smallest call there is in use: a graph that fits the caches many times over, launches and host path count
        dict(name="tiny_sum", kind="aggregate", graph="er", n=4096, e=65536, widths="64", op="sum", dtype="f32",
             weights=False, indptr64=False),
        # a whole model on a small graph: many short calls one after the other
        dict(name="small_layers", kind="layers", graph="sym", skew="strong", n=24490, e=1237182, widths="100,256,256,47"),
        # a step of mini-batch training: the subgraph is new every time
        dict(name="sampled_subgraph", kind="sampled", graph="sym", skew="strong", n=61226, e=3092956, widths="100", op="mean"),
        # full feature vectors on the edges, at an odd width
        dict(name="edge_messages", kind="messages", graph="sym", skew="strong", n=244903, e=12371828, widths="33", binop="mul"),
        # narrow rows with normalisation weights that belong to the graph: the index stream outweighs the features
        dict(name="weighted_narrow", kind="aggregate", graph="sym", skew="mild", n=132534, e=79000000, widths="8,64", op="sum",
             dtype="f32", weights=True, indptr64=False),
        # attention-like scalars on the same graph: new weights every step, gradients for them
        dict(name="attention", kind="attention", graph="sym", skew="mild", n=132534, e=79000000, widths="64"),
        # very many edges per vertex, wide ragged rows
        dict(name="dense_mean", kind="aggregate", graph="sym", skew="strong", n=232965, e=114615892, widths="602,256", op="mean",
             dtype="f32", weights=False, indptr64=False),
        # the two-layer model on that graph: narrow hidden rows after wide inputs
        dict(name="dense_layers", kind="layers", graph="sym", skew="strong", n=232965, e=114615892, widths="602,16,41"),
        # the headline stack: the aggregation widths of three-layer training on 2.4 million vertices
        dict(name="sparse_mean", kind="aggregate", graph="sym", skew="strong", n=2449029, e=123718280, widths="100,256", op="mean",
             dtype="f32", weights=False, indptr64=False),
        # the whole three-layer model on that graph
        dict(name="sparse_layers", kind="layers", graph="sym", skew="strong", n=2449029, e=123718280, widths="100,256,256,47"),
        # max pooling on that graph
        dict(name="sparse_pool", kind="pool", graph="sym", skew="strong", n=2449029, e=123718280, widths="100", reducer="max"),
        # the largest graph: bf16 features far beyond every cache, few edges per vertex, 64-bit row pointers
        # (a quarter of the capacity workload, so that three of them fit the card)
        dict(name="capacity_bf16", kind="aggregate", graph="dir", skew="strong", n=27764989, e=403921468, widths="128", op="mean",
             dtype="bf16", weights=False, indptr64=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    """A case of the same ranges: vertices, edges per vertex and widths over their logarithms, odd ones among them."""
    kind = rng.choice(["aggregate", "aggregate", "aggregate", "layers", "layers", "pool", "attention", "messages", "sampled"])
    n_max = {"aggregate": 2449029, "layers": 2449029, "pool": 2449029, "attention": 2449029, "messages": 244903, "sampled": 244903}[kind]
    e_max = {"aggregate": 123718280, "layers": 123718280, "pool": 123718280, "attention": 79000000, "messages": 12371828,
             "sampled": 12371828}[kind]
    n = _log_int(rng, 2000, n_max)
    # a power-law graph has no more distinct edges to offer than this
    degree = _log_int(rng, 6, min(600, max(8, n // 400)))
    graph = rng.choice(["sym", "sym", "dir"]) if n >= 20000 else rng.choice(["er", "sym", "dir"])
    e = min(e_max, n * degree + rng.randrange(n))
    if graph == "sym":
        e -= e % 2
    case = dict(kind=kind, graph=graph, n=n, e=e)
    if graph != "er":
        case["skew"] = rng.choice(["strong", "mild"])
    if kind == "layers":
        f_in, hidden, classes = _log_int(rng, 16, 602), rng.choice([16, 32, 64, 100, 128, 256]), rng.randrange(5, 65)
        # the work stays below that of the largest model above
        case["widths"] = ",".join(map(str, [f_in, hidden, classes] if rng.random() < 0.5 or f_in > 256 else [f_in, hidden, hidden, classes]))
    elif kind == "pool":
        case.update(widths=str(_log_int(rng, 4, 128)), reducer=rng.choice(["max", "min"]))
    elif kind == "attention":
        case.update(widths=str(_log_int(rng, 4, 128)))
    elif kind == "messages":
        case.update(widths=str(_log_int(rng, 2, 64)), binop=rng.choice(["add", "sub", "mul"]))
    elif kind == "sampled":
        case.update(widths=str(_log_int(rng, 8, 256)), op=rng.choice(["mean", "sage"]))
    else:
        weights = rng.random() < 0.3
        case.update(widths=str(_log_int(rng, 4, 602)), op="sum" if weights else rng.choice(["sum", "mean", "gcn", "sage"]),
                    dtype=rng.choice(["f32", "f32", "bf16"]), weights=weights, indptr64=rng.random() < 0.25)
    return case


def _widths(case):
    return [int(f) for f in case["widths"].split(",")]


def _edges(case, seed):
    if case["graph"] == "er":
        return synth.erdos_renyi_directed(case["n"], case["e"], seed, device="cuda")
    make = synth.rmat_symmetric if case["graph"] == "sym" else synth.rmat_directed
    return make(case["n"], case["e"], PROBS[case["skew"]], seed, device="cuda")


def _normal(gen, *shape, dtype=torch.float32):
    return torch.empty(shape, device="cuda", dtype=dtype).normal_(generator=gen)


def _like(t):
    return torch.empty_like(t)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    el = _edges(case, seed)
    n, e, widths, kind = el.n, el.e, _widths(case), case["kind"]
    if kind == "sampled":
        f = widths[0]
        x, dy = _normal(gen, n, f), _normal(gen, n, f)
        return dict(case=case, dst=el.dst, src=el.src, x=x, y=_like(x), dy=dy, dx=_like(x))
    w = synth.gcn_sym_edge_weights(el.dst, el.src, n) if case.get("weights") else None
    g = gnn.build_device_graph(el.dst, el.src, n, edge_w=w, indptr64=bool(case.get("indptr64")),
                               want_perm=kind in ("attention", "messages"))
    del el
    s = dict(case=case, g=g)
    if kind == "aggregate":
        dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
        if w is not None:  # the weights belong to the graph
            g.plan_fwd.bind_edge_weights(g.edge_w)
            g.plan_bwd.bind_edge_weights(g.edge_w_t)
        s["calls"] = []
        for f in widths:
            g.plan_fwd.prepare(g.indices, OPS[case["op"]], False, f, dtype)
            g.plan_bwd.prepare(g.indices_t, OPS[case["op"]], True, f, dtype)
            x, dy = _normal(gen, n, f, dtype=dtype), _normal(gen, n, f, dtype=dtype)
            s["calls"].append((f, x, _like(x), dy, _like(x)))
    elif kind == "layers":
        s["x"] = _normal(gen, n, widths[0])
        s["layers"] = []
        room = 0
        for i, (fi, fo) in enumerate(zip(widths, widths[1:])):
            relu = i + 2 < len(widths)
            f = min(fi, fo)
            g.plan_fwd.prepare(g.indices, gnn.GNN_SAGE_GCN, False, f)
            g.plan_bwd.prepare(g.indices_t, gnn.GNN_SAGE_GCN, True, f)
            room = max(room, gnn.gnn_sage_layer_workspace_bytes(n, fi, fo, relu))
            saved = torch.empty(gnn.gnn_sage_layer_saved_elems(n, fi, fo), device="cuda")
            h = torch.empty(n, fo, device="cuda")
            # The backward pass reads activations of its own and not what the forward calls of the same pass wrote:
            # a rectifier's gate jumps at zero, so two correct forward passes, equal but for their last bits,
            # would set some gates differently and hide how close the gradients are.
            act = _normal(gen, n, fo)
            s["layers"].append(dict(
                relu=relu, w=_normal(gen, fi, fo) / fi ** 0.5, b=_normal(gen, fo) * 0.1, saved=saved, h=h,
                x_bwd=s["x"] if i == 0 else s["layers"][-1]["h_bwd"], h_bwd=act.clamp_(min=0.0) if relu else act,
                saved_bwd=_normal(gen, saved.numel()), dx=None if i == 0 else torch.empty(n, fi, device="cuda"),
                dw=torch.empty(fi, fo, device="cuda"), db=torch.empty(fo, device="cuda")))
        s["dh"] = _normal(gen, n, widths[-1])
        s["workspace"] = torch.empty((room + 3) // 4, device="cuda")
    else:
        d = widths[0]
        s["v"], s["do"] = _normal(gen, n, d), _normal(gen, n, d)
        s["o"], s["dv"] = _like(s["v"]), _like(s["v"])
        if kind == "pool":
            s["arg"] = torch.empty(n, d, dtype=torch.int32, device="cuda")
        elif kind == "attention":
            s["fe"] = torch.rand(e, device="cuda", generator=gen)
            s["dfe"] = _like(s["fe"])
        else:
            s["fe"] = _normal(gen, e, d)
            s["dfe"] = _like(s["fe"])
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "sampled":
        f, op = _widths(case)[0], OPS[case["op"]]
        g = gnn.build_device_graph(s["dst"], s["src"], case["n"])
        gnn.gnn_aggregate_fwd(g.indptr, g.indices, None, s["x"], s["y"], g.n, f, op, plan=g.plan_fwd)
        gnn.gnn_aggregate_bwd(g.indptr_t, g.indices_t, None, s["dy"], s["dx"], g.n, f, op, plan=g.plan_bwd)
        return [g.indptr, g.indptr_t, g.indices_t, s["y"], s["dx"]]
    g = s["g"]
    if kind == "aggregate":
        op = OPS[case["op"]]
        out = []
        for f, x, y, dy, dx in s["calls"]:
            gnn.gnn_aggregate_fwd(g.indptr, g.indices, g.edge_w, x, y, g.n, f, op, plan=g.plan_fwd)
            gnn.gnn_aggregate_bwd(g.indptr_t, g.indices_t, g.edge_w_t, dy, dx, g.n, f, op, plan=g.plan_bwd)
            out += [y, dx]
        return out
    if kind == "layers":
        x, dh = s["x"], s["dh"]
        for l in s["layers"]:
            gnn.gnn_sage_layer_fwd(g.indptr, g.indices, x, l["w"], l["b"], l["saved"], l["h"], g.plan_fwd, relu=l["relu"])
            x = l["h"]
        for l in reversed(s["layers"]):
            gnn.gnn_sage_layer_bwd(g.indptr_t, g.indices_t, l["x_bwd"], l["w"], l["saved_bwd"], l["h_bwd"], dh, l["dx"], l["dw"],
                                   l["db"], g.plan_bwd, s["workspace"], relu=l["relu"])
            dh = l["dx"]
        return [[l["h"], l["dw"], l["db"], l["dx"]] for l in s["layers"]]
    d = _widths(case)[0]
    if kind == "pool":
        gnn.gnn_ap_fwd(g.indptr, g.indices, s["v"], None, s["o"], s["arg"], g.n, d, gnn.GNN_BIN_COPY_LHS, REDUCERS[case["reducer"]],
                       plan=g.plan_fwd)
        gnn.gnn_ap_bwd_vertex_arg(g.indices, s["arg"], s["do"], None, s["dv"], g.n, g.n, d, gnn.GNN_BIN_COPY_LHS)
        return [s["o"], s["arg"], s["dv"]]
    binop = gnn.GNN_BIN_MUL if kind == "attention" else BINOPS[case["binop"]]
    gnn.gnn_ap_fwd(g.indptr, g.indices, s["v"], s["fe"], s["o"], None, g.n, d, binop, gnn.GNN_RED_SUM, plan=g.plan_fwd)
    gnn.gnn_ap_bwd_vertex(g.indptr_t, g.indices_t, s["do"], s["fe"], s["dv"], g.n, d, binop, plan=g.plan_bwd, edge_ids=g.perm)
    gnn.gnn_ap_bwd_edge(g.indptr, g.indices, None, s["v"], s["fe"], s["do"], s["dfe"], g.n, d, binop, plan=g.plan_fwd)
    return [s["o"], s["dv"], s["dfe"]]


def work(case):
    """Every input read once and every output written once; one operation per edge and column for a plain sum, two for a
    weighted one, two per multiply-add of a dense product."""
    n, e, widths, kind = case["n"], case["e"], _widths(case), case["kind"]
    graph = 4 * e + (8 if case.get("indptr64") else 4) * (n + 1)  # indices and row pointers of one orientation
    if kind == "aggregate":
        size, weights = (2 if case["dtype"] == "bf16" else 4), 1 if case["weights"] else 0
        return dict(bytes=sum(2 * (graph + 4 * e * weights + 2 * n * f * size) for f in widths),
                    flops=sum(2 * e * f * (1 + weights) for f in widths))
    if kind == "sampled":
        f = widths[0]
        return dict(bytes=8 * e + 2 * graph + 2 * n * f * 8, flops=2 * e * f)
    if kind == "layers":
        nbytes = flops = 0
        for i, (fi, fo) in enumerate(zip(widths, widths[1:])):
            f, first = min(fi, fo), i == 0
            first_agg = fi <= fo
            # forward: features in, result out, and what the backward pass is given when aggregating first
            nbytes += graph + 4 * (n * (fi + fo) + fi * fo + (n * fi if first_agg else 0))
            flops += e * f + 2 * n * fi * fo
            # backward: output gradient, stored output (rectifier only) and stored operand in; gradients out
            relu = i + 2 < len(widths)
            nbytes += 4 * (n * fo * (2 if relu else 1) + n * fi + 2 * fi * fo + fo + (0 if first else n * fi))
            flops += 2 * n * fi * fo * (1 if first else 2)
            if not (first and first_agg):  # the gradient passes through the aggregation
                nbytes += graph
                flops += e * f
        return dict(bytes=nbytes, flops=flops)
    d = widths[0]
    if kind == "pool":  # values and winners out; then winners and gradient in, vertex gradient out
        return dict(bytes=graph + 4 * n * d * 3 + 4 * n * d * 3, flops=e * d + n * d)
    edge = 4 * e * (1 if kind == "attention" else d)
    reads_edge = kind == "attention" or case["binop"] == "mul"  # the gradients of a sum or difference need no operand
    nbytes = graph + edge + 8 * n * d                                             # forward
    nbytes += graph + (edge + 8 * e if reads_edge else 0) + 8 * n * d             # vertex gradient, through the permutation
    nbytes += graph + edge + 4 * n * d * (2 if reads_edge else 1)                 # edge gradient
    return dict(bytes=nbytes, flops=e * d * (6 if reads_edge else 4))


def tolerance(case):
    # bf16 results are rounded once at the end, fp32 sums differ by the order of their additions only
    return {"rel": 1e-2} if case.get("dtype") == "bf16" else {"rel": 1e-5}
