"""The work a user of this library has it do, as cases that can be timed and checked.

A program builds a handle for its graph once (`cbm_build`) and multiplies by it many times: the bare product `A X`, the
GCN-normalised one, the mean and GIN aggregators, the two-layer GCN, the dense `X W` beside them and, for training on a directed
graph, the product of the transpose.  `prepare` therefore makes the graph, the handle, the features and the output buffers;
`run` is one pass of the product calls.

Graphs come in the five kinds the library's workloads name, made on the GPU from the seed: `communities` (small, planted
communities), `citation` (sparse, blocks and copied neighbourhoods), `collaboration` (a union of cliques), `proximity` (nearest
neighbours of points in space) and `powerlaw` (R-MAT, undirected or directed).  Features are Gaussian, weights Glorot-uniform.
"""
import math

import numpy as np
import torch

import paper_2409_02208_amd as cbm


def listed():
    return [
        # the smallest call: a small social graph, every launch counts
        {"name": "communities_norm", "op": "normalized", "graph": "communities", "n": 1024, "k": 16},
        # raw bag-of-words features of a citation network through the normalised adjacency: wide rows, few neighbours
        {"name": "citation_norm_wide", "op": "normalized", "graph": "citation", "n": 19717, "k": 500},
        # inference of a small two-layer GCN on the citation network
        {"name": "citation_gcn", "op": "gcn", "graph": "citation", "n": 19717, "f_in": 500, "hidden": 64, "f_out": 3},
        # one hidden layer's aggregation on a co-authorship network, GCN weights
        {"name": "collaboration_norm", "op": "normalized", "graph": "collaboration", "n": 235868, "k": 128},
        # the same network, sum aggregator of a GIN layer
        {"name": "collaboration_gin", "op": "gin", "graph": "collaboration", "n": 235868, "k": 64},
        # one hidden layer's aggregation on a dense similarity graph, the format's best case
        {"name": "proximity_norm", "op": "normalized", "graph": "proximity", "n": 132534, "knn": 300, "k": 256},
        # inference of a two-layer GCN on the similarity graph: both dense products and both aggregations
        {"name": "proximity_gcn", "op": "gcn", "graph": "proximity", "n": 132534, "knn": 300, "f_in": 256, "hidden": 256, "f_out": 112},
        # label propagation (A X, no weights) of a few columns on a smaller similarity graph
        {"name": "proximity_spmm_narrow", "op": "spmm", "graph": "proximity", "n": 40000, "knn": 100, "k": 32},
        # the largest: a power-law graph of 2 M nodes and 125 M entries
        {"name": "powerlaw_norm", "op": "normalized", "graph": "powerlaw", "scale": 21, "edge_factor": 32, "k": 128},
        # mean aggregation (GraphSAGE) of class scores, an odd number of them
        {"name": "powerlaw_mean_ragged", "op": "mean", "graph": "powerlaw", "scale": 18, "edge_factor": 32, "k": 47},
        # one training step's products on a directed graph: the aggregation forward, the transpose's backward
        {"name": "directed_forward_backward", "op": "forward_backward", "graph": "directed", "scale": 17, "edge_factor": 16, "k": 100},
        # the classification layer alone: a tall product with an odd number of columns
        {"name": "matmul_classes", "op": "matmul", "m": 132534, "k": 100, "n": 47},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng):
    k = _log(rng, 8, 320)
    return k if rng.random() < 0.4 else max(8, (k + 7) // 8 * 8)  # most widths in use are multiples of eight


def draw(rng):
    op = rng.choice(["normalized", "normalized", "normalized", "spmm", "relu", "mean", "gin", "gcn", "forward_backward", "matmul"])
    if op == "matmul":
        return {"op": op, "m": _log(rng, 5000, 300000), "k": _width(rng), "n": rng.choice([rng.randint(2, 64), 8 * rng.randint(2, 32)])}
    kind = "directed" if op == "forward_backward" else rng.choice(["communities", "citation", "collaboration", "proximity", "powerlaw"])
    case = {"op": op, "graph": kind}
    if kind == "communities":
        case["n"] = _log(rng, 300, 5000)
    elif kind == "citation":
        case["n"] = _log(rng, 2500, 170000)
    elif kind == "collaboration":
        case["n"] = _log(rng, 20000, 236000)
    elif kind == "proximity":
        case["n"] = _log(rng, 6000, 132534)
        case["knn"] = _log(rng, 60, 300)
    else:
        case["scale"] = rng.randint(14, 18 if kind == "directed" else 20)
        case["edge_factor"] = rng.choice([16, 32])
    if op == "gcn":
        case["f_in"] = _width(rng)
        case["hidden"] = rng.choice([16, 32, 64, 128, 256])
        case["f_out"] = rng.choice([rng.randint(2, 64), 112])
    else:
        case["k"] = _width(rng)
    return case


# --------------------------------------------------------------------------- graphs, on the GPU, from the seed alone
def _generator(seed, salt):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 1000003 + salt)


def _csr(n, src, dst, symmetric=True):
    """(rowptr, columns) of the edges without self-loops and repetitions, as int64 tensors on the GPU."""
    keep = src != dst
    src, dst = src[keep], dst[keep]
    keys = src * n + dst
    if symmetric:
        keys = torch.cat((keys, dst * n + src))
    keys = torch.unique(keys)
    rows = keys // n
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    rowptr[1:] = torch.cumsum(torch.bincount(rows, minlength=n), 0)
    return rowptr, keys - rows * n


def _communities(n, gen):
    """Communities of 128: a node links to ten of the sixteen core members of its own and to two nodes anywhere."""
    groups = max(1, n // 128)
    mine = torch.clamp(torch.arange(n, device="cuda") // (n // groups), max=groups - 1)
    size = n // groups
    core = torch.rand(groups, size, device="cuda", generator=gen).argsort(1)[:, :16]
    pick = torch.rand(n, 16, device="cuda", generator=gen).argsort(1)[:, :10]
    near = torch.gather(core[mine], 1, pick) + (mine * size)[:, None]
    far = torch.randint(0, n, (n, 2), device="cuda", generator=gen)
    nodes = torch.arange(n, device="cuda")
    return _csr(n, nodes.repeat_interleave(12), torch.cat((near, far), 1).reshape(-1))


def _citation(n, gen):
    """Three blocks, about three links a node, most of them inside; 30 % of the nodes copy 80 % of a neighbour's links."""
    size = -(-n // 3)
    inside = int(1.31 * n)
    across = int(0.13 * n)
    u = torch.randint(0, n, (inside + across,), device="cuda", generator=gen)
    v = torch.randint(0, n, (inside + across,), device="cuda", generator=gen)
    v[:inside] = torch.clamp(u[:inside] // size * size + v[:inside] % size, max=n - 1)
    rowptr, col = _csr(n, u, v)
    who = torch.randperm(n, device="cuda", generator=gen)[:int(0.3 * n)]
    deg = rowptr[1:] - rowptr[:-1]
    who = who[deg[who] > 0]
    at = (torch.rand(len(who), device="cuda", generator=gen) * deg[who]).long()
    whom = col[rowptr[who] + torch.minimum(at, deg[who] - 1)]
    count = deg[whom]
    first = torch.cumsum(count, 0) - count
    copier = who.repeat_interleave(count)
    place = torch.arange(int(count.sum()), device="cuda") - first.repeat_interleave(count)
    taken = col[rowptr[whom].repeat_interleave(count) + place]
    keep = torch.rand(len(taken), device="cuda", generator=gen) < 0.8
    return _csr(n, torch.cat((u, copier[keep])), torch.cat((v, taken[keep])))


def _collaboration(n, gen):
    """Cliques of 2 to 50 members, sizes by a Zipf law, three memberships a node on average."""
    member = torch.poisson(torch.full((n,), 3.0, device="cuda"), generator=gen).long()
    stubs = torch.arange(n, device="cuda").repeat_interleave(member)
    stubs = stubs[torch.randperm(len(stubs), device="cuda", generator=gen)]
    support = torch.arange(2, 51, device="cuda", dtype=torch.float64)
    sizes = 2 + torch.multinomial(support ** -2.0, len(stubs) // 2, replacement=True, generator=gen)
    ends = torch.cumsum(sizes, 0)
    sizes = sizes[ends <= len(stubs)]
    starts = torch.cumsum(sizes, 0) - sizes
    src, dst = [], []
    for s in range(2, 51):
        at = starts[sizes == s]
        iu, ju = torch.triu_indices(s, s, 1, device="cuda")
        src.append(stubs[at[:, None] + iu].reshape(-1))
        dst.append(stubs[at[:, None] + ju].reshape(-1))
    return _csr(n, torch.cat(src), torch.cat(dst))


def _proximity(n, knn, gen):
    """Uniform points in the unit cube, each linked to its nearest neighbours."""
    points = torch.rand(n, 3, device="cuda", generator=gen)
    src, dst = [], []
    step = max(1, (1 << 29) // n)
    for at in range(0, n, step):
        mine = points[at:at + step]
        d = (mine[:, None, 0] - points[None, :, 0]).square_()
        d += (mine[:, None, 1] - points[None, :, 1]).square_()
        d += (mine[:, None, 2] - points[None, :, 2]).square_()
        near = torch.topk(d, min(knn + 1, n), dim=1, largest=False, sorted=False).indices
        src.append(torch.arange(at, at + len(mine), device="cuda").repeat_interleave(near.shape[1]))
        dst.append(near.reshape(-1))
    return _csr(n, torch.cat(src), torch.cat(dst))


def _powerlaw(scale, edge_factor, gen, symmetric):
    """R-MAT (0.57, 0.19, 0.19, 0.05), vertex labels shuffled."""
    n, edges = 1 << scale, edge_factor << scale
    src = torch.zeros(edges, dtype=torch.int64, device="cuda")
    dst = torch.zeros(edges, dtype=torch.int64, device="cuda")
    for _ in range(scale):
        r = torch.rand(edges, device="cuda", generator=gen)
        src = 2 * src + (r >= 0.76)
        dst = 2 * dst + (((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
    label = torch.randperm(n, device="cuda", generator=gen)
    return _csr(n, label[src], label[dst], symmetric)


def _graph(case, seed):
    gen = _generator(seed, 1)
    kind = case["graph"]
    if kind in ("powerlaw", "directed"):
        return _powerlaw(case["scale"], case["edge_factor"], gen, kind == "powerlaw")
    if kind == "proximity":
        return _proximity(case["n"], case["knn"], gen)
    return {"communities": _communities, "citation": _citation, "collaboration": _collaboration}[kind](case["n"], gen)


def _nodes(case):
    return case["n"] if "n" in case else 1 << case["scale"]


def _features(n, k, seed, salt):
    return torch.randn(n, k, device="cuda", generator=_generator(seed, salt))


def _glorot(f_in, f_out, seed, salt):
    a = math.sqrt(6.0 / (f_in + f_out))
    return torch.rand(f_in, f_out, device="cuda", generator=_generator(seed, salt)).mul_(2 * a).sub_(a)


# --------------------------------------------------------------------------- what a program has in hand, and one pass
SELF_LOOPS = ("normalized", "relu", "gcn", "forward_backward")
EPS = 0.25


def prepare(case, seed):
    op = case["op"]
    if op == "matmul":
        return {"op": op, "A": _features(case["m"], case["k"], seed, 2), "B": _glorot(case["k"], case["n"], seed, 3),
                "C": torch.empty(case["m"], case["n"], device="cuda")}
    n = _nodes(case)
    rowptr, col = _graph(case, seed)
    rowptr, col = rowptr.cpu().numpy(), col.to(torch.int32).cpu().numpy()
    state = {"op": op, "h": cbm.cbm_build(n, n, rowptr, col, add_self_loops=op in SELF_LOOPS)}
    if op == "gcn":
        f_in, hidden, f_out = case["f_in"], case["hidden"], case["f_out"]
        state.update(X=_features(n, f_in, seed, 2), W0=_glorot(f_in, hidden, seed, 3), W1=_glorot(hidden, f_out, seed, 4),
                     out=torch.empty(n, f_out, device="cuda"),
                     workspace=torch.empty(cbm.cbm_gcn2_workspace_bytes(state["h"], f_in, hidden, f_out), dtype=torch.uint8, device="cuda"))
        return state
    state.update(X=_features(n, case["k"], seed, 2), Y=torch.empty(n, case["k"], device="cuda"))
    if op == "forward_backward":
        state.update(ht=cbm.cbm_build(n, n, rowptr, col, add_self_loops=True, transpose=True), dY=_features(n, case["k"], seed, 3),
                     dX=torch.empty(n, case["k"], device="cuda"))
    return state


def run(state):
    op = state["op"]
    if op == "matmul":
        return cbm.cbm_dense_matmul(state["A"], state["B"], state["C"])
    if op == "gcn":
        return cbm.cbm_gcn2_forward(state["h"], state["X"], state["W0"], state["W1"], state["out"], state["workspace"])
    if op == "forward_backward":
        return (cbm.cbm_spmm_normalized(state["h"], state["X"], state["Y"]),
                cbm.cbm_spmm_normalized(state["ht"], state["dY"], state["dX"]))
    if op == "gin":
        return cbm.cbm_spmm_gin(state["h"], EPS, state["X"], state["Y"])
    call = {"normalized": cbm.cbm_spmm_normalized, "relu": cbm.cbm_spmm_normalized_relu, "mean": cbm.cbm_spmm_mean, "spmm": cbm.cbm_spmm}[op]
    return call(state["h"], state["X"], state["Y"])


# --------------------------------------------------------------------------- what a pass cannot do without
def _degree(case):
    """Mean entries of a row of the graph, as the generators give them."""
    kind = case["graph"]
    if kind == "proximity":
        return 1.07 * case["knn"]
    if kind in ("powerlaw", "directed"):
        return (1.85 if kind == "powerlaw" else 0.97) * case["edge_factor"]
    return {"communities": 23.0, "citation": 4.2, "collaboration": 39.2}[kind]


def work(case):
    op = case["op"]
    if op == "matmul":
        m, k, n = case["m"], case["k"], case["n"]
        return {"bytes": 4 * (m * k + k * n + m * n), "flops": 2 * m * k * n}
    n = _nodes(case)
    entries = n * (_degree(case) + (op in SELF_LOOPS))
    pattern = 4 * entries + 8 * n  # a column index each, an offset a row
    if op == "gcn":
        f, h, o = case["f_in"], case["hidden"], case["f_out"]
        return {"bytes": 2 * pattern + 4 * (n * f + f * h + 3 * n * h + h * o + 3 * n * o), "flops": 2 * n * h * (f + o) + entries * (h + o)}
    passes = 2 if op == "forward_backward" else 1
    return {"bytes": passes * (pattern + 8 * n * case["k"]), "flops": passes * entries * case["k"]}


def tolerance(case):
    # sums of up to a hundred thousand 32-bit terms: four times the worst seen against 64 bits, 4.3e-7 in the 2-norm (two layers)
    # and 4e-5 at one value (the bare sum of a power-law graph's largest row, against the root mean square of all rows)
    return {"rel": 2e-6, "max": 1.6e-4}


# --------------------------------------------------------------------------- the same in 64 bits, in plain torch
def _sum_rows(rowptr, col, X, weight=None):
    """sum over each row's entries j of weight[j] X[j], in 64 bits."""
    n, k = len(rowptr) - 1, X.shape[1]
    if weight is not None:
        X = X * weight[:, None]
    out = torch.zeros(n, k, dtype=torch.float64, device="cuda")
    room = max(1 << 20, (1 << 29) // k)  # entries at a time
    ends = rowptr.cpu().numpy()
    at = 0
    while at < n:
        to = max(at + 1, int(np.searchsorted(ends, ends[at] + room, side="right")) - 1)
        part = X[col[ends[at]:ends[to]]]
        out[at:to] = torch.segment_reduce(part, "sum", lengths=rowptr[at + 1:to + 1] - rowptr[at:to], axis=0, unsafe=True, initial=0.0)
        at = to
    return out


def _with_self(rowptr, col):
    n = len(rowptr) - 1
    rows = torch.repeat_interleave(torch.arange(n, device="cuda"), rowptr[1:] - rowptr[:-1])
    nodes = torch.arange(n, device="cuda")
    keys = torch.unique(torch.cat((rows * n + col, nodes * n + nodes)))
    rows = keys // n
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    rowptr[1:] = torch.cumsum(torch.bincount(rows, minlength=n), 0)
    return rowptr, keys - rows * n


def _transposed(rowptr, col):
    n = len(rowptr) - 1
    rows = torch.repeat_interleave(torch.arange(n, device="cuda"), rowptr[1:] - rowptr[:-1])
    keys = torch.sort(col * n + rows).values
    turned = keys // n
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    rowptr[1:] = torch.cumsum(torch.bincount(turned, minlength=n), 0)
    return rowptr, keys - turned * n


def exact(case, seed):
    op = case["op"]
    if op == "matmul":
        return _features(case["m"], case["k"], seed, 2).double() @ _glorot(case["k"], case["n"], seed, 3).double()
    n = _nodes(case)
    rowptr, col = _graph(case, seed)
    if op in SELF_LOOPS:
        rowptr, col = _with_self(rowptr, col)
        d = (rowptr[1:] - rowptr[:-1]).double().rsqrt()

    def normalized(X, turned=False):
        return _sum_rows(*(_transposed(rowptr, col) if turned else (rowptr, col)), X, d).mul_(d[:, None])

    if op == "gcn":
        X = _features(n, case["f_in"], seed, 2).double()
        W0, W1 = _glorot(case["f_in"], case["hidden"], seed, 3).double(), _glorot(case["hidden"], case["f_out"], seed, 4).double()
        return normalized(normalized(X @ W0).relu_() @ W1)
    X = _features(n, case["k"], seed, 2).double()
    if op == "forward_backward":
        return normalized(X), normalized(_features(n, case["k"], seed, 3).double(), turned=True)
    if op == "normalized":
        return normalized(X)
    if op == "relu":
        return normalized(X).relu_()
    total = _sum_rows(rowptr, col, X)
    if op == "gin":
        return total.add_(X, alpha=1 + EPS)
    if op == "mean":
        return total / torch.clamp(rowptr[1:] - rowptr[:-1], min=1).double()[:, None]
    return total
