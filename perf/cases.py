"""What the sampling library is used for, as cases that can be timed.

A case is one sampling call (with what its consumer calls next, where that is a
call of this library too) on a synthetic graph: k-hop neighbourhoods for GNN
mini-batches and for whole graphs, random walks for embeddings, layer-wise
importance samples with their adjacency matrices.  Graphs have the shapes of the
workloads of `bench.py` (R-MAT and Chung-Lu power-law graphs, symmetrised,
vertices relabelled at random) and are generated on the GPU from the seed.

`listed()` is the fixed list, `draw(rng)` one more case of the same ranges,
`prepare` builds what a program holds before the call (graph handle, roots,
output arrays, workspace), `run` is one call, `work` the bytes it cannot do
without, `tolerance` how exact the outputs are.
"""
from __future__ import annotations

import math

import torch

from paper_2009_06693_amd import binding as B

DEVICE = "cuda:0"
APPS = {"deepwalk": B.ND_DEEPWALK, "ppr": B.ND_PPR, "node2vec": B.ND_NODE2VEC, "khop": B.ND_KHOP,
        "layer": B.ND_LAYER, "multirw": B.ND_MULTIRW}


def _case(**kw):
    """All fields of a case.

    graph "rmat" (V a power of two) or "power" (Chung-Lu, degree exponent `gamma`, largest
    expected degree `cap`); `pairs` undirected pairs are drawn before loops and repeats go.
    offsets 32 or 64 (bits); weights "none", "uniform" in [1, 5) or "symmetric" = 2^14 / (deg deg).
    samples: number of samples (k-hop and walks: one root each); everywhere: True = vertex 0, 1, 2,
    ... is sample 0's, 1's, 2's root, False = roots in random order without repeats.
    fanout (k-hop, layer) as text; steps (walks); unique: rounds of unique-neighbour sampling;
    records: the walks are gathered into one row per walk; edges: the edges between consecutive
    layers are recorded; static: the entry point that brings its own scratch."""
    c = dict(app="khop", graph="power", V=233000, pairs=59_600_000, gamma=2.1, cap=26000.0, offsets=32,
             weights="none", samples=1024, per_sample=1, everywhere=False, fanout="", steps=0, unique=0,
             records=False, edges=False, static=False)
    unknown = set(kw) - set(c) - {"name"}
    if unknown:
        raise KeyError(unknown)
    c.update(kw)
    return c


_RMAT22 = dict(graph="rmat", V=1 << 22, pairs=35_800_000, offsets=64)
_RMAT12 = dict(graph="rmat", V=1 << 12, pairs=65_536)
_PPI = dict(graph="power", V=57_000, pairs=826_000, gamma=2.3, cap=1280.0)
_DENSE = dict(graph="power", V=233_000, pairs=59_600_000, gamma=2.1, cap=26000.0)
_ORKUT = dict(graph="power", V=3_000_000, pairs=58_800_000, gamma=2.1, cap=10800.0)


def listed():
    return [
        # Inference for a few requested vertices: the neighbourhood of a handful of roots, three hops,
        # scratch from the library (a serving loop that allocates nothing).  Latency only.
        _case(name="khop_serve_37", app="khop", **_DENSE, samples=37, fanout="15,10,5", static=True),
        # GraphSAGE training: one mini-batch of 1,024 roots on the dense 233 K-vertex graph.
        _case(name="khop_batch_1024", app="khop", **_DENSE, samples=1024, fanout="25,10"),
        # The same epoch in one call: every vertex of the dense graph a root (its adjacency does not fit the
        # last-level cache).
        _case(name="khop_dense_all", app="khop", **_DENSE, samples=233_000, everywhere=True, fanout="25,10"),
        # Every vertex of a skewed 4.2 M-vertex graph with 64-bit offsets, half of the vertices isolated.
        _case(name="khop_rmat22_all", app="khop", **_RMAT22, samples=1 << 22, everywhere=True, fanout="25,10"),
        # Neighbours without repeats within a sample (GraphSAGE without replacement).
        _case(name="khop_unique_rmat22", app="khop", **_RMAT22, samples=1 << 22, everywhere=True, fanout="25,10",
              unique=4),
        # DeepWalk corpora: a small graph (few walks, a chain of short dependent steps) ...
        _case(name="deepwalk_rmat12", app="deepwalk", **_RMAT12, samples=1 << 12, everywhere=True, steps=100,
              records=True),
        # ... and a large one; the walks leave as one row per walk, as a skip-gram trainer reads them.
        _case(name="deepwalk_rmat22", app="deepwalk", **_RMAT22, samples=1 << 22, everywhere=True, steps=100,
              records=True),
        # Second-order and terminating walks over edge weights on a protein-interaction-sized graph.
        _case(name="node2vec_57k", app="node2vec", **_PPI, weights="uniform", samples=57_000, everywhere=True,
              steps=100),
        _case(name="ppr_57k", app="ppr", **_PPI, weights="uniform", samples=57_000, everywhere=True, steps=100),
        # LADIES-style training: 4,096 mini-batches of 64 roots, two layers of 2,048 vertices, and the adjacency
        # matrices between the layers.
        _case(name="layer_edges_3m", app="layer", **_ORKUT, samples=4096, per_sample=64, fanout="2048,2048",
              edges=True),
        # Layer sampling over symmetrically normalised edge weights, 257 mini-batches of 512 roots.
        _case(name="layer_symmetric_3m", app="layer", **_ORKUT, weights="symmetric", samples=257, per_sample=512,
              fanout="512,512"),
        # Multi-dimensional random walk (frontier sampling): 100 roots per sample, 100 steps.
        _case(name="multirw_rmat22", app="multirw", **_RMAT22, samples=41_943, per_sample=100, steps=100),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case: an application, a graph between the smallest and the largest listed one, and a
    number of samples over its whole range, none with more output than the largest listed ones."""
    kind = rng.choice(["khop", "khop", "khop", "khop_unique", "deepwalk", "deepwalk", "node2vec", "ppr", "layer",
                       "layer_edges", "multirw"])
    wide = rng.random() < 0.3
    if rng.random() < 0.4:
        scale = rng.randint(12, 22)
        V, g = 1 << scale, dict(graph="rmat", gamma=2.1, cap=1000.0)
    else:
        V, g = _log_int(rng, 4096, 3_000_000), dict(graph="power", gamma=round(rng.uniform(2.05, 2.6), 2))
    degree = math.exp(rng.uniform(math.log(8), math.log(60 if V > 300_000 else 400)))
    pairs = max(2 * V, min(int(V * degree / 2), 58_800_000 if V <= 3_000_000 else 35_800_000, V * (V // 64)))
    if g["graph"] == "power":
        g["cap"] = float(min(V // 8, int(40 * 2 * pairs / V)))
    g = dict(g, V=V, pairs=pairs, offsets=64 if wide else 32)
    weights = rng.choice(["none", "uniform"])
    everywhere = rng.random() < 0.5
    if kind in ("khop", "khop_unique"):
        fanout = rng.choice(["25,10", "25,10", "10,25", "15,10,5", "10,10", "5,5", "20", "7,13", "8,8,4"])
        slots = math.prod(int(x) for x in fanout.split(","))
        n = _log_int(rng, 16, min(V, 600_000_000 // slots))
        static = kind == "khop" and n * slots <= 1_000_000 and rng.random() < 0.5
        return _case(app="khop", **g, samples=n, everywhere=everywhere, fanout=fanout, static=static,
                     unique=rng.choice([2, 4, 8]) if kind == "khop_unique" else 0)
    if kind in ("deepwalk", "node2vec", "ppr"):
        steps = rng.choice([10, 40, 80, 100])
        most = {"deepwalk": 200_000_000, "ppr": 60_000_000, "node2vec": 12_000_000}[kind]
        n = _log_int(rng, 64, min(V, most // steps))
        return _case(app=kind, **g, weights=weights if V * degree < 40_000_000 else "none", samples=n,
                     everywhere=everywhere, steps=steps, records=kind == "deepwalk" and rng.random() < 0.5)
    if kind in ("layer", "layer_edges"):
        per = rng.choice([16, 64, 500, 512])
        fanout = rng.choice(["256,256", "512,512", "1000,300", "2048,2048"])
        n = _log_int(rng, 1, max(1, min(V // per, (1 << 22) // max(int(x) for x in fanout.split(",")))))
        symmetric = kind == "layer" and V * degree < 40_000_000 and rng.random() < 0.5
        return _case(app="layer", **g, weights="symmetric" if symmetric else "none", samples=n, per_sample=per,
                     fanout=fanout, edges=kind == "layer_edges")
    per = rng.choice([4, 30, 100])
    n = _log_int(rng, 16, max(16, min(V // per, 42_000)))
    return _case(app="multirw", **g, samples=n, per_sample=per, steps=rng.choice([20, 100]))


# ---------------------------------------------------------------------------- graphs
def _rmat_pairs(scale, n, gen):
    a, b, c = (0.57, 0.19, 0.19) if scale < 16 else (0.6, 0.15, 0.15)
    u = torch.zeros(n, dtype=torch.int64, device=DEVICE)
    v = torch.zeros(n, dtype=torch.int64, device=DEVICE)
    for _ in range(scale):
        r = torch.rand(n, generator=gen, device=DEVICE)
        down = r >= a + b
        right = torch.logical_or(torch.logical_and(r >= a, ~down), r >= a + b + c)
        u = u * 2 + down
        v = v * 2 + right
    return u, v


def _power_pairs(V, n, gamma, cap, gen):
    """Endpoints with probability proportional to (i + i0)^-alpha, through the inverse of the integral;
    i0 makes the largest expected degree `cap`."""
    alpha = 1.0 / (gamma - 1.0)
    k = 1.0 - alpha

    def largest(i0):
        return 2.0 * n * i0 ** -alpha / (((V + i0) ** k - i0 ** k) / k)

    lo, hi = 0.0, math.log(64.0 * V)
    for _ in range(60):
        mid = (lo + hi) / 2
        lo, hi = (mid, hi) if largest(math.exp(mid)) > cap else (lo, mid)
    i0 = math.exp(hi)
    base, span = i0 ** k, (V + i0) ** k - i0 ** k
    ends = []
    for _ in range(2):
        r = torch.rand(n, generator=gen, device=DEVICE, dtype=torch.float64)
        ends.append(((r * span + base) ** (1.0 / k) - i0).to(torch.int64).clamp_(0, V - 1))
    return ends


def _graph(case, gen):
    """(row offsets, columns, weights or None): symmetric, no loops, rows ascending without repeats."""
    V = case["V"]
    if case["graph"] == "rmat":
        u, v = _rmat_pairs(V.bit_length() - 1, case["pairs"], gen)
    else:
        u, v = _power_pairs(V, case["pairs"], case["gamma"], case["cap"], gen)
    keep = u != v
    label = torch.randperm(V, generator=gen, device=DEVICE)
    u, v = label[u[keep]], label[v[keep]]
    key = torch.unique(torch.cat([(u << 32) | v, (v << 32) | u]))
    del u, v, keep
    rows = torch.arange(V + 1, device=DEVICE, dtype=torch.int64) << 32
    off = torch.searchsorted(key, rows)
    col = (key & 0x7FFFFFFF).to(torch.int32)
    w = None
    if case["weights"] != "none":
        src, dst = key >> 32, key & 0x7FFFFFFF
        if case["weights"] == "uniform":  # the same in both directions
            h = (torch.minimum(src, dst) * 2654435761 + torch.maximum(src, dst) * 40503 + 12345) & 0xFFFFFFFF
            h = (h ^ (h >> 15)) * 2246822519 & 0xFFFFFFFF
            w = 1.0 + 4.0 * ((h >> 8).to(torch.float32) / float(1 << 24))
        else:
            deg = (off[1:] - off[:-1]).to(torch.float32)
            w = 16384.0 / (deg[src] * deg[dst])
    return off.to(torch.int64 if case["offsets"] == 64 else torch.int32), col, w


# ---------------------------------------------------------------------------- the contract
def _fanout(case):
    return [int(x) for x in case["fanout"].split(",")] if case["fanout"] else []


def _layers(case):
    """(transit slots, new slots) per sample at every step of a layer case."""
    f = _fanout(case)
    return list(zip([case["per_sample"]] + f[:-1], f))


def _matrix_buffers(S, n_prev, m):
    """What a training loop keeps for one layer's adjacency matrices: row pointers, scratch, and room for
    the edges (a place beyond the last edge stays -1), so that no step waits for the host."""
    pairs = S * n_prev * m
    room = max(min(pairs, 1 << 26), pairs // 24)
    return dict(row_ptr=torch.empty(S * n_prev + 1, dtype=torch.int64, device=DEVICE),
                workspace=torch.empty(max(B.nd_layer_edges_workspace_bytes(S, n_prev), 256), dtype=torch.uint8,
                                      device=DEVICE),
                slots=torch.full((room,), -1, dtype=torch.int32, device=DEVICE))


def prepare(case, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    off, col, w = _graph(case, gen)
    graph = B.nd_graph_create(off, col, w)
    n = case["samples"] * case["per_sample"]
    if case["everywhere"]:
        roots = torch.arange(n, dtype=torch.int32, device=DEVICE)
    else:
        roots = torch.randperm(case["V"], generator=gen, device=DEVICE)[:n].to(torch.int32)
    kw = {}
    app = APPS[case["app"]]
    if case["app"] in ("khop", "layer"):
        kw = dict(num_steps=len(_fanout(case)), fanout=_fanout(case))
    else:
        kw = dict(num_steps=case["steps"])
    if case["app"] in ("layer", "multirw"):
        kw["roots_per_sample"] = case["per_sample"]
    if case["app"] == "node2vec":
        kw.update(p=2.0, q=0.5)
    if case["app"] == "ppr":
        kw["term_prob"] = 0.01
    if case["weights"] != "none":
        kw["use_weights"] = 1
    if case["unique"]:
        kw["unique_rounds"] = case["unique"]
    params = B.nd_params_init(**kw)
    state = dict(case=case, graph=graph, app=app, params=params, roots=roots, seed=seed + 1)
    if case["app"] in ("khop", "layer") and not case["static"]:
        state["sampler"] = B.Sampler(graph, app, params, n)
        if case["edges"]:
            state["matrices"] = [_matrix_buffers(case["samples"], p, f) for p, f in _layers(case)]
        return state
    # walks keep their steps as the rows of one array; the serving loop brings its own outputs as well
    lens, ws_bytes = B.nd_sample_query(graph, app, params, n)
    if case["static"]:
        state["out"] = [torch.empty(k, dtype=torch.int32, device=DEVICE) for k in lens]
        state["status"] = torch.zeros(1, dtype=torch.int32, device=DEVICE)
        return state
    state["steps"] = torch.empty((len(lens), case["samples"]), dtype=torch.int32, device=DEVICE)
    state["out"] = [state["steps"][i] for i in range(len(lens))]
    state["workspace"] = torch.empty(ws_bytes, dtype=torch.uint8, device=DEVICE)
    if case["records"]:
        state["rows"] = torch.empty((case["samples"], len(lens)), dtype=torch.int32, device=DEVICE)
    return state


def run(state):
    case, graph, roots = state["case"], state["graph"], state["roots"]
    if case["static"]:
        B.nd_sample_static(graph, state["app"], state["params"], roots, state["seed"], state["out"],
                           state["status"])
        return {"steps": state["out"], "status": state["status"]}
    if "sampler" not in state:  # walks
        B.nd_sample(graph, state["app"], state["params"], roots, state["seed"], state["out"], state["workspace"])
        if case["records"]:
            return B.nd_samples_pack(state["out"], case["samples"], state["rows"])
        return state["steps"]
    out = state["sampler"].run(roots, state["seed"])
    if not case["edges"]:
        return out
    S = case["samples"]
    layers = [roots.view(S, -1)] + [o.view(S, -1) for o in out]
    for before, after, m in zip(layers, layers[1:], state["matrices"]):
        B.nd_layer_edges_count(graph, before, after, m["row_ptr"], m["workspace"])
        B.nd_layer_edges_fill(graph, before, after, m["row_ptr"], m["slots"])
    return {"layers": out, "matrices": [(m["row_ptr"], m["slots"]) for m in state["matrices"]]}


def work(case):
    """Bytes only (the arithmetic is integer and small): roots and outputs once; of the graph, an adjacency
    entry per draw and a row's two offsets per transit, but no more of either than the graph has.
    Weighted draws read a weight with every entry; recorded edges read the transits' lists, which
    between them hold the whole graph when there are many samples."""
    E = 2 * case["pairs"] * 0.97
    S, b_off = case["samples"], case["offsets"] // 8
    per_entry = 4 + (4 if case["weights"] != "none" else 0)
    if case["app"] in ("khop", "layer"):
        width, widths, transits = 1, [], S * case["per_sample"]
        for f in _fanout(case):
            width = f if case["app"] == "layer" else width * f
            widths.append(width)
        transits += S * sum(widths[:-1])
        outputs = S * sum(widths)
    else:
        outputs = S * case["steps"]
        transits = outputs
    total = 4.0 * S * case["per_sample"] + 4.0 * outputs
    total += per_entry * min(E, outputs) + 2.0 * b_off * min(case["V"], transits)
    if case["records"]:
        total += 8.0 * outputs - 4.0 * outputs  # the steps are read once more to become records
    if case["edges"]:
        total += 4.0 * E * min(1.0, S * sum(p for p, _ in _layers(case)) / case["V"])
        # row pointers, and an edge between about one in sixty (transit, new vertex) pairs
        total += sum(8.0 * S * p + 4.0 * S * p * f / 60 for p, f in _layers(case))
    return {"bytes": total, "flops": 0.0}


def tolerance(case):
    """Vertex numbers and slots are whole numbers and exactly one output is right."""
    return "exact"
