"""The routes that run all steps of a sample in one launch (k-hop, unique neighbours, walks, layer
samples), at the sizes where their kernels change shape, against the oracle: one draw or two per
lane, several samples per workgroup or several workgroups per sample, rows in LDS up to the last
that fit, launches of 128 steps, 64 or 256 walks and 4 or 16 samples per workgroup, weighted links,
rows whose weights all quantise to zero, calls of more walks than one launch has counters for."""
import numpy as np
import pytest
import torch

import oracle
from paper_2009_06693_amd import binding as B
from paper_2009_06693_amd import inputs

from gpu_util import assert_steps_equal, gpu_sample

pytestmark = pytest.mark.gpu


def _graph(weighted, int64_offsets, zeros=True):
    """Skewed, with dead ends, one row that holds nearly every vertex, and (weighted) rows and
    entries whose weights quantise to zero."""
    rng = np.random.default_rng(7)
    V = 700
    pairs = set(zip(rng.integers(0, V, 6000).tolist(), (rng.random(6000) ** 2 * V).astype(int).tolist()))
    pairs |= {(3, v) for v in range(0, V, 2)} | {(v, 3) for v in range(0, V, 3)}
    pairs = sorted((a, b) for a, b in pairs if a % 11 != 5)    # rows 5, 16, ... are empty
    w = None
    if weighted:
        w = (1.0 + 4.0 * rng.random(len(pairs))).astype(np.float32)
        if zeros:
            w[rng.random(len(pairs)) < 0.1] = 1e-6
            w[[a % 13 == 1 for a, _ in pairs]] = 1e-6
    g = inputs.from_edges(V, pairs, weights=w, int64_offsets=int64_offsets)
    return g, B.nd_graph_create(g.row_offsets, g.col_indices, g.weights), \
        oracle.OracleGraph(g.row_offsets, g.col_indices, g.weights)


@pytest.fixture(scope="module", params=[(False, False), (True, False), (False, True), (True, True)],
                ids=["plain32", "weighted32", "plain64", "weighted64"])
def graph(request):
    return _graph(*request.param)


def _roots(V, n, seed):
    r = np.random.default_rng(seed).integers(0, V, size=n, dtype=np.int32)
    r[::17] = -1
    return r


@pytest.mark.parametrize("fanout,S", [([1], 1), ([7], 9000), ([2], 9000), ([2, 3], 9000), ([3, 2, 1, 2], 3000),
                                      ([15, 10, 5], 37), ([25, 10], 2049), ([4096, 2], 3), ([63, 64, 2], 2),
                                      ([64, 64, 2], 2), ([300000], 2)])
def test_khop(graph, fanout, S):
    g, dg, og = graph
    roots = _roots(g.V, S, 1)
    want = oracle.khop(og, roots, fanout, seed=5, sample_id_base=9)
    got, stats = gpu_sample(dg, B.ND_KHOP, roots, 5, num_steps=len(fanout), fanout=fanout, sample_id_base=9)
    assert_steps_equal(got, want, f"khop {fanout} S={S}")
    live = [(roots >= 0).sum()] + [(w >= 0).sum() for w in want[:-1]]
    assert stats[:, 0].tolist() == live


def test_khop_into_outputs_of_any_alignment(graph):
    g, dg, og = graph
    roots = _roots(g.V, 333, 2)
    want = oracle.khop(og, roots, [3, 4], seed=6)
    p = B.nd_params_init(num_steps=2, fanout=[3, 4])
    lens, ws = B.nd_sample_query(dg, B.ND_KHOP, p, 333)
    for skip in (0, 1, 2, 3):
        flat = [torch.full((n + 8,), -7, dtype=torch.int32, device="cuda:0") for n in lens]
        out = [f[skip:skip + n] for f, n in zip(flat, lens)]
        B.nd_sample(dg, B.ND_KHOP, p, torch.as_tensor(roots, device="cuda:0"), 6, out,
                    torch.empty(ws, dtype=torch.uint8, device="cuda:0"))
        torch.cuda.synchronize()
        assert_steps_equal([o.cpu().numpy() for o in out], want, f"skip={skip}")
        for f, n in zip(flat, lens):
            assert (f[:skip] == -7).all() and (f[skip + n:] == -7).all()


@pytest.mark.parametrize("fanout,rounds", [([1], 1), ([32], 64), ([33], 3), ([16, 2], 4), ([5, 7, 3], 5), ([255, 1], 2),
                                           ([2, 1024], 2), ([1024, 2], 3)])
def test_unique_neighbours(graph, fanout, rounds):
    g, dg, og = graph
    roots = _roots(g.V, 257, 3)
    want = oracle.khop(og, roots, fanout, seed=8, unique_rounds=rounds)
    got, _ = gpu_sample(dg, B.ND_KHOP, roots, 8, num_steps=len(fanout), fanout=fanout, unique_rounds=rounds)
    assert_steps_equal(got, want, f"unique {fanout} rounds={rounds}")


@pytest.mark.parametrize("steps,S", [(1, 1), (127, 63), (128, 64), (129, 65), (257, 130), (3, 65536), (3, 65537)])
def test_walks(graph, steps, S):
    g, dg, og = graph
    roots = _roots(g.V, S, 4)
    for weighted in ((0, 1) if g.weights is not None else (0,)):
        kw = dict(num_steps=steps, use_weights=weighted)
        want = oracle.deepwalk(og, roots, steps, seed=9, use_weights=bool(weighted))
        got, stats = gpu_sample(dg, B.ND_DEEPWALK, roots, 9, **kw)
        assert_steps_equal(got, list(want), "deepwalk")
        assert stats[:, 0].tolist() == [(roots >= 0).sum()] + [(w >= 0).sum() for w in want[:-1]]
        want = oracle.ppr(og, roots, steps, 0.02, seed=10, use_weights=bool(weighted))
        got, _ = gpu_sample(dg, B.ND_PPR, roots, 10, term_prob=0.02, **kw)
        assert_steps_equal(got, list(want), "ppr")


@pytest.mark.parametrize("steps,S", [(1, 15), (15, 16), (16, 17), (17, 255), (33, 257), (144, 1000), (31, 8192),
                                     (31, 8193)])
def test_walks_of_sixteen_lanes(graph, steps, S):
    """Up to 8,192 walks: blocks of 16 steps, walks that end at any place inside one, empty rows at the graph's end."""
    g, dg, og = graph
    roots = _roots(g.V, S, 14)
    roots[-1] = g.V - 1
    for weighted in ((0, 1) if g.weights is not None else (0,)):
        kw = dict(num_steps=steps, use_weights=weighted, sample_id_base=77)
        want = oracle.deepwalk(og, roots, steps, seed=15, use_weights=bool(weighted), sample_id_base=77)
        got, stats = gpu_sample(dg, B.ND_DEEPWALK, roots, 15, **kw)
        assert_steps_equal(got, list(want), "deepwalk")
        assert stats[:, 0].tolist() == [(roots >= 0).sum()] + [(w >= 0).sum() for w in want[:-1]]
        for p in (0.0, 0.1, 1.0):
            want = oracle.ppr(og, roots, steps, p, seed=16, use_weights=bool(weighted), sample_id_base=77)
            got, stats = gpu_sample(dg, B.ND_PPR, roots, 16, term_prob=p, **kw)
            assert_steps_equal(got, list(want), f"ppr {p}")
            assert stats[:, 0].tolist() == [(roots >= 0).sum()] + [(w >= 0).sum() for w in want[:-1]]


@pytest.mark.parametrize("int64_offsets", [False, True])
@pytest.mark.parametrize("steps,S", [(1, 1), (127, 63), (129, 65), (257, 130), (3, 65537)])
def test_node2vec(int64_offsets, steps, S):
    g, dg, og = _graph(True, int64_offsets, zeros=False)
    roots = _roots(g.V, S, 4)
    for weighted in (0, 1):
        for attempts in (0, 1, 64):
            want = oracle.node2vec(og, roots, steps, 2.0, 0.5, seed=11, use_weights=bool(weighted),
                                   max_attempts=attempts)
            got, stats = gpu_sample(dg, B.ND_NODE2VEC, roots, 11, num_steps=steps, p=2.0, q=0.5,
                                    n2v_max_attempts=attempts, use_weights=weighted)
            assert_steps_equal(got, list(want), f"node2vec attempts={attempts} weighted={weighted}")
            assert stats[:, 0].tolist() == [(roots >= 0).sum()] + [(w >= 0).sum() for w in want[:-1]]


@pytest.mark.parametrize("int64_offsets", [False, True])
@pytest.mark.parametrize("steps,S", [(1, 15), (40, 17), (130, 33), (5, 16384), (5, 16385)])
def test_node2vec_with_several_attempts_at_once(int64_offsets, steps, S):
    """Four attempts per round up to 16,384 walks where most are refused; budgets that end inside a round or at its
    end, whichever bias is the highest."""
    g, dg, og = _graph(True, int64_offsets, zeros=False)
    roots = _roots(g.V, S, 41)
    for p, q, weighted in ((2.0, 0.5, 1), (0.25, 4.0, 0), (4.0, 4.0, 1), (1.0, 1.0, 0), (8.0, 0.125, 0)):
        for attempts in (1, 4, 5, 64) if S < 1000 else (6,):
            want = oracle.node2vec(og, roots, steps, p, q, seed=42, use_weights=bool(weighted), max_attempts=attempts,
                                   sample_id_base=5)
            got, stats = gpu_sample(dg, B.ND_NODE2VEC, roots, 42, num_steps=steps, p=p, q=q, sample_id_base=5,
                                    n2v_max_attempts=attempts, use_weights=weighted)
            assert_steps_equal(got, list(want), f"node2vec p={p} q={q} attempts={attempts} weighted={weighted}")
            assert stats[:, 0].tolist() == [(roots >= 0).sum()] + [(w >= 0).sum() for w in want[:-1]]


def test_node2vec_without_membership_tables():
    """The tables are made when the scratch of a node2vec call is asked for; without them rows are searched."""
    g, dg, og = _graph(True, False, zeros=False)
    roots = _roots(g.V, 500, 5)
    want = oracle.node2vec(og, roots, 20, 0.5, 4.0, seed=12, use_weights=True)
    lens, ws = B.nd_sample_query(dg, B.ND_DEEPWALK, B.nd_params_init(num_steps=20), 500)  # the same scratch
    out = [torch.empty(n, dtype=torch.int32, device="cuda:0") for n in lens]
    B.nd_sample(dg, B.ND_NODE2VEC, B.nd_params_init(num_steps=20, p=0.5, q=4.0, use_weights=1),
                torch.as_tensor(roots, device="cuda:0"), 12, out, torch.empty(ws, dtype=torch.uint8, device="cuda:0"))
    torch.cuda.synchronize()
    assert_steps_equal([o.cpu().numpy() for o in out], list(want), "node2vec")


@pytest.mark.parametrize("R,steps,S", [(1, 64, 15), (2, 129, 17), (100, 65, 16), (256, 70, 33), (257, 130, 5),
                                       (1024, 300, 4), (1025, 300, 3), (4096, 64, 1)])
def test_multi_dimensional_walk(graph, R, steps, S):
    g, dg, og = graph
    roots = _roots(g.V, R * S, 6)
    want = oracle.multirw(og, roots, R, steps, seed=13)
    got, _ = gpu_sample(dg, B.ND_MULTIRW, roots, 13, num_steps=steps, roots_per_sample=R)
    assert_steps_equal(got, list(want), f"multirw R={R}")


@pytest.mark.parametrize("app,steps,S,R", [(B.ND_DEEPWALK, 2100, 800_000, 1), (B.ND_MULTIRW, 2100, 60_000, 3)])
def test_more_walks_than_one_launch_counts_for_fit_the_static_scratch(app, steps, S, R):
    """Counters for every workgroup of these calls would take 26 and 32 MB; samples beyond what the scratch
    has room for go to further launches.  The bad roots are the first launch's and the last launch's."""
    g, dg, og = _graph(False, False)
    roots = np.random.default_rng(8).integers(0, g.V, size=S * R, dtype=np.int32)
    roots[[5, S * R - 2]] = g.V
    p = B.nd_params_init(num_steps=steps, roots_per_sample=R) if R > 1 else B.nd_params_init(num_steps=steps)
    lens, ws = B.nd_sample_query(dg, app, p, S * R)
    assert ws <= B.ND_STATIC_SCRATCH_BYTES
    flat = torch.empty((steps, S), dtype=torch.int32, device="cuda:0")
    status = torch.zeros(1, dtype=torch.int32, device="cuda:0")
    out = [flat[i] for i in range(steps)]
    r = torch.as_tensor(roots, device="cuda:0")
    B.nd_sample_static(dg, app, p, r, 21, out, status)
    torch.cuda.synchronize()
    assert int(status) == 1
    clean = roots.copy()
    clean[[5, S * R - 2]] = -1
    for a, n in ((0, 200), (S // 2, 200), (S - 200, 200)):
        part = clean[a * R:(a + n) * R]
        want = (oracle.multirw(og, part, R, steps, seed=21, sample_id_base=a) if R > 1
                else oracle.deepwalk(og, part, steps, seed=21, sample_id_base=a))
        assert np.array_equal(flat[:, a:a + n].cpu().numpy(), np.stack(list(want)))
    if R == 1:
        workspace = torch.empty(ws, dtype=torch.uint8, device="cuda:0")
        B.nd_sample(dg, app, p, r, 21, out, workspace)
        live = B.nd_sample_stats(workspace, steps)[:, 0]
        assert live[0] == S - 2 and live[1:].tolist() == (flat[:-1] >= 0).sum(dim=1).tolist()
        with pytest.raises(B.NdError):
            B.nd_sample_status(workspace)


@pytest.mark.parametrize("per,fanout,S", [(1, [1], 1), (64, [512], 513), (64, [513, 7], 512), (3, [513, 600], 513),
                                          (512, [4096, 512], 2), (4096, [9, 4096], 2), (2, [3], 16_500),
                                          (63, [64], 5), (65, [3, 64], 5), (128, [2, 1], 3), (4, [129], 3),
                                          (256, [5], 3), (257, [256], 3), (1, [513, 512], 300), (4096, [514], 257)])
def test_layer(graph, per, fanout, S):
    g, dg, og = graph
    roots = _roots(g.V, per * S, 7)
    for weighted in ((0, 1) if g.weights is not None else (0,)):
        want = oracle.layer(og, roots, per, fanout, seed=14, use_weights=bool(weighted))
        got, _ = gpu_sample(dg, B.ND_LAYER, roots, 14, num_steps=len(fanout), fanout=fanout, roots_per_sample=per,
                            use_weights=weighted)
        assert_steps_equal(got, want, f"layer per={per} {fanout} weighted={weighted}")


@pytest.mark.parametrize("graph", [(True, False), (True, True)], ids=["weighted32", "weighted64"], indirect=True)
@pytest.mark.parametrize("per,fanout", [(4096, [4096, 30]), (1, [700, 4096]), (65, [64, 63, 5])])
def test_layer_over_weights_with_and_without_the_rows_totals(graph, per, fanout):
    """They are made when the sizes of a weighted layer call are asked for."""
    g, dg, og = graph
    roots = _roots(g.V, per * 7, 51)
    want = oracle.layer(og, roots, per, fanout, seed=52, use_weights=True)
    kw = dict(num_steps=len(fanout), fanout=fanout, roots_per_sample=per)
    fresh = B.nd_graph_create(g.row_offsets, g.col_indices, g.weights)
    for asked in (0, 1):
        lens, ws = B.nd_sample_query(fresh, B.ND_LAYER, B.nd_params_init(use_weights=asked, **kw), roots.size)
        out = [torch.empty(n, dtype=torch.int32, device="cuda:0") for n in lens]
        B.nd_sample(fresh, B.ND_LAYER, B.nd_params_init(use_weights=1, **kw), torch.as_tensor(roots, device="cuda:0"), 52,
                    out, torch.empty(ws, dtype=torch.uint8, device="cuda:0"))
        torch.cuda.synchronize()
        assert_steps_equal([o.cpu().numpy() for o in out], want, f"asked={asked}")


@pytest.mark.parametrize("heavy_first", [False, True])
def test_layer_rows_whose_guide_cells_hold_many_entries(heavy_first):
    """A few heavy entries beside hundreds of light ones: all light ones of a stretch fall into one or two cells
    of the row's guide table, so the search inside the row goes on by halves."""
    V = 900
    pairs = [(a, b) for a in range(V) for b in range(0, V, 1 if a < 8 else 90)]
    w = np.full(len(pairs), 0.5, np.float32)
    w[np.arange(len(pairs)) % 450 == (0 if heavy_first else 449)] = 3000.0
    g = inputs.from_edges(V, pairs, weights=w, int64_offsets=heavy_first)
    dg, og = B.nd_graph_create(g.row_offsets, g.col_indices, g.weights), \
        oracle.OracleGraph(g.row_offsets, g.col_indices, g.weights)
    roots = np.arange(40, dtype=np.int32) % 8
    want = oracle.layer(og, roots, 4, [2000, 700], seed=3, use_weights=True)
    light = np.asarray(want[0]) % 450 != (0 if heavy_first else 449)
    assert light.sum() > 100   # some draws do end among the light entries
    got, _ = gpu_sample(dg, B.ND_LAYER, roots, 3, num_steps=2, fanout=[2000, 700], roots_per_sample=4, use_weights=1)
    assert_steps_equal(got, want, f"heavy_first={heavy_first}")


@pytest.mark.parametrize("heavy_first", [False, True])
def test_weighted_walks_where_one_entry_outweighs_a_long_row(heavy_first):
    """A hub whose light entries all fall into two cells of its row's guide table: a draw that ends among them takes
    the looks of a search by halves, not one look per light entry (14,000 of them: milliseconds, where the whole
    call takes a tenth of one), so the call takes about as long as with equal weights."""
    V, S, steps = 20_001, 65_536, 8
    pairs = [(0, b) for b in range(1, V)] + [(a, 0) for a in range(1, V)]
    heavy = 0 if heavy_first else V - 2
    w = np.ones(len(pairs), np.float32)
    w[:V - 1] = 1e-4
    w[heavy] = 30_000.0
    g = inputs.from_edges(V, pairs, weights=w)
    og = oracle.OracleGraph(g.row_offsets, g.col_indices, g.weights)
    roots = np.zeros(S, np.int32)
    want = oracle.deepwalk(og, roots, steps, seed=19, use_weights=True)
    assert sum((np.asarray(want[i]) != heavy + 1).sum() for i in range(0, steps, 2)) > 5  # light entries are drawn
    times = []
    for weights in (np.ones_like(w), g.weights):
        dg = B.nd_graph_create(g.row_offsets, g.col_indices, weights)
        s = B.Sampler(dg, B.ND_DEEPWALK, B.nd_params_init(num_steps=steps, use_weights=1), S)
        r = torch.as_tensor(roots, device="cuda:0")
        s.run(r, 19)
        marks = [torch.cuda.Event(enable_timing=True) for _ in range(8)]
        for m in marks:
            m.record()
            out = s.run(r, 19)
        torch.cuda.synchronize()
        times.append(min(a.elapsed_time(b) for a, b in zip(marks, marks[1:])))
    assert_steps_equal([o.cpu().numpy() for o in out], list(want), f"heavy_first={heavy_first}")
    got, _ = gpu_sample(dg, B.ND_PPR, roots, 20, num_steps=steps, use_weights=1, term_prob=0.02)
    assert_steps_equal(got, list(oracle.ppr(og, roots, steps, 0.02, seed=20, use_weights=True)), "ppr")
    print(f"[times] equal weights {times[0]:.4f} ms, one heavy entry {times[1]:.4f} ms", flush=True)
    assert times[1] < 8.0 * times[0] + 0.05  # 0.0129 and 0.0154 ms; entry by entry 2.4 ms


@pytest.mark.parametrize("weighted,int64_offsets", [(False, False), (False, True), (True, False), (True, True)])
@pytest.mark.parametrize("p,q,attempts", [(0.05, 20.0, 64), (0.05, 20.0, 2), (2.0, 0.5, 0), (20.0, 0.05, 1)])
def test_node2vec_draws_that_end_in_the_exact_one(weighted, int64_offsets, p, q, attempts):
    """Few lanes of a wavefront at a time (its lanes share a row then) and all of them; rows around one and two
    wavefronts long; samples in workgroups of 64 and 256."""
    V = 701
    pairs = [(a, (31 * a + 7 * j) % V) for a in range(V) for j in range((1, 63, 64, 65, 3, 0, 129, 500)[a % 8])]
    pairs = sorted(pairs)
    w = 1.0 + 4.0 * np.random.default_rng(5).random(len(pairs), dtype=np.float32) if weighted else None
    g = inputs.from_edges(V, pairs, weights=w, int64_offsets=int64_offsets)
    dg, og = B.nd_graph_create(g.row_offsets, g.col_indices, g.weights), \
        oracle.OracleGraph(g.row_offsets, g.col_indices, g.weights)
    for steps, S in ((9, 700), (2, 65_600)):
        roots = _roots(g.V, S, 9)
        for use in ((0, 1) if weighted else (0,)):
            want = oracle.node2vec(og, roots, steps, p, q, seed=22, use_weights=bool(use), max_attempts=attempts)
            got, _ = gpu_sample(dg, B.ND_NODE2VEC, roots, 22, num_steps=steps, p=p, q=q, n2v_max_attempts=attempts,
                                use_weights=use)
            assert_steps_equal(got, list(want), f"node2vec p={p} q={q} attempts={attempts} weighted={use}")


def test_node2vec_with_biases_far_apart_takes_no_longer_than_in_windows():
    """Most candidates are rejected 64 times and a row is gone through for the draw: by one lane each where the lanes
    come together (windows), by the wavefront where they come one by one."""
    g = inputs.config2_graph()
    dg = B.nd_graph_create(g.row_offsets, g.col_indices, g.weights)
    r = torch.as_tensor(inputs.all_vertices_roots(g)[:20_000], device="cuda:0")
    times, outs = [], []
    for window in (0, 256):
        s = B.Sampler(dg, B.ND_NODE2VEC, B.nd_params_init(num_steps=10, p=0.05, q=20.0, use_weights=1,
                                                          sched_window=window), r.numel())
        outs.append([o.clone() for o in s.run(r, 19)])
        marks = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
        for m in marks:
            m.record()
            s.run(r, 19)
        torch.cuda.synchronize()
        times.append(min(a.elapsed_time(b) for a, b in zip(marks, marks[1:])))
    assert all(torch.equal(a, b) for a, b in zip(*outs))
    print(f"[times] over links {times[0]:.2f} ms, in windows {times[1]:.2f} ms", flush=True)
    assert times[0] < 1.1 * times[1]


@pytest.mark.parametrize("weighted,int64_offsets", [(False, True), (True, False)])
@pytest.mark.parametrize("attempts", [0, 3])
def test_node2vec_exact_draws_in_long_rows(weighted, int64_offsets, attempts):
    """Rows whose entries one pass of the wavefront covers, just not, and those that are cut into stretches of one
    and of several passes; rows of one entry, which need no draw; weights of zero beside others."""
    lengths = [1, 2, 5, 255, 256, 257, 512, 16_383, 16_385, 33_000]
    V = 33_100
    pairs = sorted({(a, (17 + j) % V) for a, n in enumerate(lengths) for j in range(n)} |
                   {(b, b % len(lengths)) for b in range(len(lengths), V)} | {(b, b // 3) for b in range(30, V, 7)})
    w = None
    if weighted:
        w = 1.0 + 4.0 * np.random.default_rng(5).random(len(pairs), dtype=np.float32)
        first = np.array([i == 0 or pairs[i - 1][0] != a for i, (a, _) in enumerate(pairs)])
        w[(np.arange(len(pairs)) % 3 == 0) & ~first] = 1e-6  # quantises to zero; no row of nothing else
    g = inputs.from_edges(V, pairs, weights=w, int64_offsets=int64_offsets)
    dg, og = B.nd_graph_create(g.row_offsets, g.col_indices, g.weights), \
        oracle.OracleGraph(g.row_offsets, g.col_indices, g.weights)
    for S in (60, 65_700):   # workgroups of 64 and of 256; few walks live
        roots = np.full(S, -1, np.int32)
        roots[:60] = np.arange(60) % 23
        if S > 60:
            roots[-60:] = np.arange(60) % 12
        for use in ((0, 1) if weighted else (0,)):
            for p, q in ((20.0, 0.05), (0.05, 20.0)):
                want = oracle.node2vec(og, roots, 6, p, q, seed=23, use_weights=bool(use), max_attempts=attempts)
                got, _ = gpu_sample(dg, B.ND_NODE2VEC, roots, 23, num_steps=6, p=p, q=q, n2v_max_attempts=attempts,
                                    use_weights=use)
                assert_steps_equal(got, list(want), f"node2vec S={S} p={p} q={q} weighted={use}")


def _least_time(dg, app, params, r, seed=19):
    """Milliseconds of the fastest of a few calls, and the outputs."""
    s = B.Sampler(dg, app, params, r.numel())
    out = [o.clone() for o in s.run(r, seed)]
    marks = [torch.cuda.Event(enable_timing=True) for _ in range(5)]
    for m in marks:
        m.record()
        s.run(r, seed)
    torch.cuda.synchronize()
    return min(a.elapsed_time(b) for a, b in zip(marks, marks[1:])), out


def test_node2vec_over_a_hub_takes_no_longer_than_in_windows():
    """Every other step stands on a row of 200,000 entries one of which outweighs the rest, so every draw from it
    is an exact one, of many walks at once."""
    V = 200_001
    pairs = [(0, b) for b in range(1, V)] + [(a, 0) for a in range(1, V)]
    w = np.full(len(pairs), 0.01, np.float32)
    w[V // 2] = 30_000.0
    g = inputs.from_edges(V, pairs, weights=w)
    dg = B.nd_graph_create(g.row_offsets, g.col_indices, g.weights)
    r = torch.arange(64, dtype=torch.int32, device="cuda:0") * 3000
    (links, a), (windows, b) = (_least_time(dg, B.ND_NODE2VEC, B.nd_params_init(
        num_steps=2, p=2.0, q=0.5, use_weights=1, sched_window=window), r) for window in (0, 256))
    assert all(torch.equal(x, y) for x, y in zip(a, b))
    print(f"[times] over links {links:.2f} ms, in windows {windows:.2f} ms", flush=True)
    assert links < 1.1 * windows


@pytest.mark.parametrize("fanout,S", [([257], 2048), ([512], 2047), ([32, 16], 2048), ([5, 171], 2048),
                                      ([1024], 8191), ([10, 10, 10], 8192), ([1, 1025], 8192)])
def test_unique_neighbours_of_many_samples(graph, fanout, S):
    """Two wavefronts per sample up to 1,024 slots, four above and for few samples; rounds that one wavefront ends."""
    g, dg, og = graph
    roots = _roots(g.V, S, 3)
    want = oracle.khop(og, roots, fanout, seed=8, unique_rounds=6)
    got, _ = gpu_sample(dg, B.ND_KHOP, roots, 8, num_steps=len(fanout), fanout=fanout, unique_rounds=6)
    assert_steps_equal(got, want, f"unique {fanout} S={S}")


@pytest.mark.parametrize("fanout,rounds,S", [([10, 10, 10], 64, 30_000), ([25, 20], 4, 57_000)])
def test_unique_neighbours_take_no_longer_than_hop_by_hop(fanout, rounds, S):
    """On a ring most slots find nothing that is not held and stay open for all rounds."""
    if rounds == 64:
        V = 100_000
        g = inputs.from_edges(V, sorted({(v, (v + d) % V) for v in range(V) for d in (1, V - 1)}))
    else:
        g = inputs.config2_graph()
    dg = B.nd_graph_create(g.row_offsets, g.col_indices, None)
    r = torch.as_tensor(inputs.all_vertices_roots(g)[:S], device="cuda:0")
    (links, a), (hops, b) = (_least_time(dg, B.ND_KHOP, B.nd_params_init(
        num_steps=len(fanout), fanout=fanout, unique_rounds=rounds, sched_window=window), r) for window in (0, -1))
    assert all(torch.equal(x, y) for x, y in zip(a, b))
    print(f"[times] all hops {links:.3f} ms, hop by hop {hops:.3f} ms", flush=True)
    assert links < 1.1 * hops


@pytest.mark.parametrize("int64_offsets", [False, True])
def test_weighted_draws_from_rows_whose_weights_span_decades(int64_offsets):
    """Guide cells of every length, first, last and only ones of a row among them: what two looks do not find is
    searched for up to the next cell's guide."""
    V = 2100
    rng = np.random.default_rng(15)
    pairs = [(a, (a + j) % V) for a in range(V) for j in range((1, 2, 3, 40, 700, 2000)[a % 6] if a < 60 else 5)]
    pairs = sorted(pairs)
    w = np.minimum(10.0 ** (6.5 * rng.random(len(pairs)) - 4.0), 30_000.0).astype(np.float32)
    g = inputs.from_edges(V, pairs, weights=w, int64_offsets=int64_offsets)
    dg, og = B.nd_graph_create(g.row_offsets, g.col_indices, g.weights), \
        oracle.OracleGraph(g.row_offsets, g.col_indices, g.weights)
    roots = (np.arange(6000) % 60).astype(np.int32)
    got, _ = gpu_sample(dg, B.ND_DEEPWALK, roots, 24, num_steps=4, use_weights=1)
    assert_steps_equal(got, list(oracle.deepwalk(og, roots, 4, seed=24, use_weights=True)), "deepwalk")
    for per, fanout in ((1, [600, 30]), (60, [900])):
        want = oracle.layer(og, roots[:600], per, fanout, seed=25, use_weights=True)
        got, _ = gpu_sample(dg, B.ND_LAYER, roots[:600], 25, num_steps=len(fanout), fanout=fanout,
                            roots_per_sample=per, use_weights=1)
        assert_steps_equal(got, want, f"layer {per} {fanout}")


@pytest.mark.parametrize("S", [40, 8192, 8193])
@pytest.mark.parametrize("int64_offsets", [False, True])
def test_weighted_walks_with_and_without_cells(int64_offsets, S):
    """The cells are made when the sizes of a weighted walk are asked for; rows of one to 400 entries whose cells
    hold none, four and hundreds of them, rows and ends of rows without weight."""
    rng = np.random.default_rng(31)
    V, pairs, w = 500, [], []
    for v in range(V):
        deg = (1, 2, 3, 4, 5, 9, 64, 400, 0)[v % 9]
        row = np.sort(rng.choice(V, size=deg, replace=False)).tolist()
        pairs += [(v, u) for u in row]
        kind = v % 5
        x = np.ones(deg) if kind == 0 else 1.0 + 4.0 * rng.random(deg) if kind == 1 else 10.0 ** rng.uniform(-4, 4, deg)
        if kind == 3 and deg > 2:
            x[deg // 2:] = 1e-6
        if kind == 4 and v % 3 == 0:
            x[:] = 1e-6
        w += x.tolist()
    g = inputs.from_edges(V, pairs, weights=np.array(w, dtype=np.float32), int64_offsets=int64_offsets)
    roots = _roots(V, S, 32)
    og = oracle.OracleGraph(g.row_offsets, g.col_indices, g.weights)
    want = oracle.ppr(og, roots, 40, 0.01, seed=33, use_weights=True)
    for asked in (False, True):
        dg = B.nd_graph_create(g.row_offsets, g.col_indices, g.weights)
        p = B.nd_params_init(num_steps=40, term_prob=0.01, use_weights=1)
        lens, ws = B.nd_sample_query(dg, B.ND_PPR, p if asked else B.nd_params_init(num_steps=40), S)  # the same scratch
        out = [torch.empty(n, dtype=torch.int32, device="cuda:0") for n in lens]
        B.nd_sample(dg, B.ND_PPR, p, torch.as_tensor(roots, device="cuda:0"), 33, out,
                    torch.empty(ws, dtype=torch.uint8, device="cuda:0"))
        torch.cuda.synchronize()
        assert_steps_equal([o.cpu().numpy() for o in out], list(want), f"asked={asked}")


@pytest.mark.parametrize("below", [False, True])
@pytest.mark.parametrize("S", [1, 8193])
def test_weighted_draw_whose_high_word_is_that_of_a_threshold(S, below):
    """The cells hold the thresholds' high words: where the draw's is the same, the low words decide."""
    seed = 5
    r0, r1, *_ = (int(x) for x in oracle.philox4x32_10([0, 0, 0, 0], [seed, 0]))
    word = (r0 << 32) + r1
    # a threshold ceil(c 2^64 / total) beside the word, on the side that is asked for
    total, c = next((t, c) for t in range(2**32 - 2**16, 2**32 - 2**20, -256)
                    for c in range(word * t // 2**64 - 1, word * t // 2**64 + 3)
                    if -(-c * 2**64 // t) >> 32 == r0 and (word < -(-c * 2**64 // t)) == below)

    def parts(x):  # x as weights that float32 holds exactly
        half = x // 2 // 256 * 256
        return [y for y in (half, (x - half) // 256 * 256, (x - half) % 256) if y > 0]
    first, second = parts(c), parts(total - c)
    q = first + second
    assert sum(q) == total and all(float(np.float32(y)) == y and y < 2**31 for y in q)
    V = len(q) + 1
    pairs = [(0, 1 + i) for i in range(len(q))] + [(1 + i, 0) for i in range(len(q))]
    w = np.array([x / 65536.0 for x in q] + [1.0] * len(q), dtype=np.float32)
    g = inputs.from_edges(V, pairs, weights=w)
    dg = B.nd_graph_create(g.row_offsets, g.col_indices, g.weights)
    og = oracle.OracleGraph(g.row_offsets, g.col_indices, g.weights)
    roots = np.zeros(S, dtype=np.int32)
    want = oracle.deepwalk(og, roots, 2, seed=seed, use_weights=True)
    assert (want[0][0] <= len(first)) == below
    got, _ = gpu_sample(dg, B.ND_DEEPWALK, roots, seed, num_steps=2, use_weights=1)
    assert_steps_equal(got, list(want), "deepwalk")


@pytest.mark.parametrize("degree,fanout,grouped", [(120, [10, 100], True), (119, [10, 100], False), (120, [7, 143], False),
                                                   (130, [10, 99], False), (80, [16, 44], True), (79, [16, 44], False),
                                                   (80, [16, 43], False)])
def test_khop_groups_where_the_graph_is_dense_and_pairs_are_many(degree, fanout, grouped):
    """Both sides of the rule's lines (20 and 14 M draws, 8 and 16 pairs per vertex); the routes agree."""
    V = 20_000
    v = torch.arange(V, device="cuda:0")
    col = ((v[:, None] + 3 * torch.arange(1, degree + 1, device="cuda:0")) % V).sort(dim=1).values
    dg = B.nd_graph_create(torch.arange(V + 1, device="cuda:0") * degree, col.reshape(-1).to(torch.int32))
    r = torch.randperm(V, device="cuda:0").to(torch.int32)
    outs = []
    for window in (0, -1):
        s = B.Sampler(dg, B.ND_KHOP, B.nd_params_init(num_steps=2, fanout=fanout, sched_window=window), V)
        outs.append(s.run(r, 26))
        torch.cuda.synchronize()
        assert (s.stats()[1, 1] > 0) == (grouped or window == -1)
    assert all(torch.equal(a, b) for a, b in zip(*outs))


@pytest.mark.parametrize("int64_offsets", [False, True])
@pytest.mark.parametrize("S", [20_000, 20_001])
def test_dense_khop_whose_first_hop_is_not_grouped(int64_offsets, S):
    """At most a root per vertex: the first hop is drawn in order; roots that are none, out of range or repeated."""
    V, degree, fanout = 20_000, 130, [11, 95]
    v = torch.arange(V, device="cuda:0")
    col = ((v[:, None] + 3 * torch.arange(1, degree + 1, device="cuda:0")) % V).sort(dim=1).values
    off = torch.arange(V + 1, device="cuda:0") * degree
    col = col[:V - 1].reshape(-1)                              # the last row is empty
    off[V] = off[V - 1]
    dg = B.nd_graph_create(off if int64_offsets else off.to(torch.int32), col.to(torch.int32))
    r = torch.arange(S, device="cuda:0").flip(0).to(torch.int32) % V
    r[5], r[6], r[300], r[S - 1] = -1, r[7], V, -5
    outs = []
    for window in (0, -1):
        s = B.Sampler(dg, B.ND_KHOP, B.nd_params_init(num_steps=2, fanout=fanout, sched_window=window, sample_id_base=9), S)
        outs.append([o.clone() for o in s.run(r, 61)])
        torch.cuda.synchronize()
        with pytest.raises(B.NdError):
            s.status()
        stats = s.stats()
        assert stats[0, 0] == S - 3 and stats[1, 0] == int((outs[-1][0] >= 0).sum()) and stats[1, 1] > 0
        assert (stats[0, 1] == 0) == (window == 0 and S <= V)
    assert all(torch.equal(a, b) for a, b in zip(*outs))


def _whole_and_halves(dg, app, S, roots, **kw):
    """The outputs of a call, and of two calls for its halves, step by step."""
    def call(first, last):
        p = B.nd_params_init(sample_id_base=first, **kw)
        return [o.reshape(-1) for o in B.Sampler(dg, app, p, last - first).run(roots[first:last], 33)]

    return zip(call(0, S), zip(call(0, S // 2), call(S // 2, S)))


@pytest.mark.parametrize("fanout", [[3, 6], [9, 4], [9, 3]])
def test_outputs_of_large_khop_calls(graph, fanout):
    """From 64 M draws of the last hop on outputs leave past the caches, in pairs or one by one: the first such call
    against its two halves, which are below the line."""
    g, dg, _ = graph
    S = -(-(64 << 20) // (fanout[0] * fanout[1]))
    r = torch.from_numpy(_roots(g.V, S, 3)).cuda()
    for whole, halves in _whole_and_halves(dg, B.ND_KHOP, S, r, num_steps=2, fanout=fanout):
        assert torch.equal(whole, torch.cat(halves))


@pytest.mark.parametrize("fanout", [[9, 3], [3, 6]])
def test_large_khop_calls_with_unique_neighbours(fanout):
    """64 M slots of the last hop against their two halves."""
    g, dg, _ = _graph(False, False)
    S = -(-(64 << 20) // (fanout[0] * fanout[1]))
    r = torch.from_numpy(_roots(g.V, S, 3)).cuda()
    for whole, halves in _whole_and_halves(dg, B.ND_KHOP, S, r, num_steps=2, fanout=fanout, unique_rounds=3):
        assert torch.equal(whole, torch.cat(halves))


@pytest.mark.parametrize("n", [2100, 2920, 3400])
def test_layer_samples_over_weights_that_leave_the_totals(n):
    """More samples than units hold with the rows' totals in LDS: against a graph that has none, and the oracle."""
    g, dg, og = _graph(True, False)
    S = 513 if n == 2100 else 257
    roots = _roots(g.V, n * S, 61)
    r = torch.as_tensor(roots, device="cuda:0")
    kw = dict(num_steps=2, fanout=[n, n], roots_per_sample=n)
    outs = []
    for asked in (1, 0):
        d = B.nd_graph_create(g.row_offsets, g.col_indices, g.weights)
        lens, ws = B.nd_sample_query(d, B.ND_LAYER, B.nd_params_init(use_weights=asked, **kw), r.numel())
        outs.append([torch.empty(k, dtype=torch.int32, device="cuda:0") for k in lens])
        B.nd_sample(d, B.ND_LAYER, B.nd_params_init(use_weights=1, **kw), r, 62, outs[-1],
                    torch.empty(ws, dtype=torch.uint8, device="cuda:0"))
        torch.cuda.synchronize()
    want = oracle.layer(og, roots[n * (S - 2):], n, [n, n], seed=62, use_weights=True, sample_id_base=S - 2)
    for a, b, w in zip(*outs, want):
        assert torch.equal(a, b)
        assert np.array_equal(a[n * (S - 2):].cpu().numpy(), np.asarray(w).reshape(-1))


@pytest.mark.parametrize("weighted,int64_offsets", [(False, False), (False, True), (True, False)])
@pytest.mark.parametrize("V", [128, 129, 256, 257, 1025, 4096])
def test_khop_over_packed_columns(V, weighted, int64_offsets):
    """Dense graphs, whose columns are read in as many bits as a vertex takes (7 to 12): rows that start at any bit, a
    last row that ends with the array, the largest vertex in it; one draw or two per lane, one hop to three."""
    rng = np.random.default_rng(V)
    rows = [np.unique(np.append(rng.integers(0, V, 4000 if V < 300 else 190), [V - 1, 0][:1 + v % 2])) for v in range(V)]
    off = np.concatenate([[0], np.cumsum([r.size for r in rows])]).astype(np.int64 if int64_offsets else np.int32)
    col = np.concatenate(rows).astype(np.int32)
    assert col.size >= 128 * V
    w = (1.0 + rng.random(col.size)).astype(np.float32) if weighted else None
    dg, og = B.nd_graph_create(off, col, w), oracle.OracleGraph(off, col, w)
    for fanout, S in (([25, 10], 900), ([7, 13], 2300), ([211], 1000), ([15, 10, 5], 300)):
        roots = _roots(V, S, 3)
        want = oracle.khop(og, roots, fanout, seed=8, sample_id_base=4)
        got, _ = gpu_sample(dg, B.ND_KHOP, roots, 8, num_steps=len(fanout), fanout=fanout, sample_id_base=4)
        assert_steps_equal(got, want, f"khop {fanout} V={V}")


@pytest.mark.parametrize("int64_offsets", [False, True])
@pytest.mark.parametrize("V", [2, 3, 4, 5, 9, 17, 33, 64])
def test_khop_over_packed_columns_of_few_bits(V, int64_offsets):
    """1 to 6 bits, of which up to 32 entries lie in a word: every row but one holds every vertex, 6 M draws, as many per parent
    as such rows allow; against the sample-parallel kernel, which reads the columns as they are."""
    rows = [np.arange(V)] * (V - 1) + [np.array([V - 1])]
    off = np.concatenate([[0], np.cumsum([r.size for r in rows])]).astype(np.int64 if int64_offsets else np.int32)
    dg = B.nd_graph_create(off, np.concatenate(rows).astype(np.int32))
    last = max(1, 5 * int(off[-1]) // (6 * V))
    r = torch.from_numpy(_roots(V, -(-6_000_000 // (3 * last)), 5)).cuda()
    outs = []
    for mode in (B.ND_MODE_TRANSIT_PARALLEL, B.ND_MODE_SAMPLE_PARALLEL):
        s = B.Sampler(dg, B.ND_KHOP, B.nd_params_init(num_steps=2, fanout=[3, last], mode=mode), r.numel())
        outs.append([o.clone() for o in s.run(r, 14)])
        torch.cuda.synchronize()
        s.status()
    for a, b in zip(*outs):
        assert torch.equal(a, b)
    assert int(outs[0][1].max()) == V - 1 and int(outs[0][1][outs[0][1] >= 0].min()) == 0


@pytest.mark.parametrize("V", [1 << 25, (1 << 25) + 1])
def test_khop_at_the_widest_packed_columns(V):
    """25 bits, the most that one load of four bytes holds at every bit of a byte, and a vertex more, where the columns
    stay as they are: against the sample-parallel kernel, which reads those."""
    v = torch.arange(V, device="cuda:0")
    other = (v * 2654435761 + 12345) % V
    other = torch.where(other == v, (v + 1) % V, other)
    col = torch.stack([torch.minimum(v, other), torch.maximum(v, other)], 1).view(-1).to(torch.int32)
    off = (torch.arange(V + 1, device="cuda:0") * 2).to(torch.int32)
    del v, other
    dg = B.nd_graph_create(off, col)
    r = torch.randint(0, V, (6_000_000,), device="cuda:0", dtype=torch.int32)
    r[:1000] = torch.arange(V - 1000, V, device="cuda:0", dtype=torch.int32)
    outs = []
    for mode in (B.ND_MODE_TRANSIT_PARALLEL, B.ND_MODE_SAMPLE_PARALLEL):
        s = B.Sampler(dg, B.ND_KHOP, B.nd_params_init(num_steps=2, fanout=[1, 1], mode=mode), r.numel())
        outs.append([o.clone() for o in s.run(r, 13)])
        torch.cuda.synchronize()
        s.status()
    for a, b in zip(*outs):
        assert torch.equal(a, b)
        assert int(a.min()) >= 0


@pytest.mark.parametrize("fanout", [[200], [60], [25, 9]])
def test_unique_neighbours_whose_vertices_share_one_bucket(fanout):
    """Rows of vertices that the kernels' hash sends to one bucket in 512: a pass for every one of them."""
    v = np.arange(200_000, dtype=np.uint32)
    same = v[((v * np.uint32(2654435761)) >> 15) & 511 == 77][:300].astype(np.int32)
    V, n = 200_000, same.size
    assert n == 300
    rows = {int(r): np.sort(same[r % 7:]) for r in range(40)}
    rows.update({int(s): np.sort(same[i % 5::2]) for i, s in enumerate(same) if int(s) >= 40})
    off = np.zeros(V + 1, dtype=np.int64)
    for r, c in rows.items():
        off[r + 1] = c.size
    off = np.cumsum(off)
    col = np.concatenate([rows[r] for r in sorted(rows)]).astype(np.int32)
    dg, og = B.nd_graph_create(off, col), oracle.OracleGraph(off, col)
    roots = np.arange(40, dtype=np.int32)
    want = oracle.khop(og, roots, fanout, seed=3, unique_rounds=6)
    got, _ = gpu_sample(dg, B.ND_KHOP, roots, 3, num_steps=len(fanout), fanout=fanout, unique_rounds=6)
    assert_steps_equal(got, want, f"{fanout}")


@pytest.mark.parametrize("fanout,rounds", [([3, 6], 0), ([9, 4], 0), ([32], 3), ([20, 3], 3), ([11, 11], 3), ([25, 10], 3)])
@pytest.mark.parametrize("wide", [False, True])
def test_first_calls_whose_outputs_leave_past_the_caches(fanout, rounds, wide):
    """24 M draws in pairs, and as many unique neighbours (half a wavefront and whole ones), over 44 M entries, with which they
    are more than the last-level cache holds: against halves, which are below the line."""
    V, degree = 2_000_000, 22
    v = torch.arange(V, device="cuda:0")
    col = (v[:, None] + 1 + 977 * torch.arange(degree, device="cuda:0")) % V
    col = col.sort(1).values.view(-1).to(torch.int32)
    off = torch.arange(V + 1, device="cuda:0") * degree
    dg = B.nd_graph_create(off if wide else off.to(torch.int32), col)
    S = -(-24_000_000 // int(np.prod(fanout)))
    r = torch.from_numpy(_roots(V, S, 3)).cuda()
    for whole, halves in _whole_and_halves(dg, B.ND_KHOP, S, r, num_steps=len(fanout), fanout=fanout, unique_rounds=rounds):
        assert torch.equal(whole, torch.cat(halves))


@pytest.mark.parametrize("app,S,kw", [(B.ND_KHOP, 30_000, dict(num_steps=2, fanout=[25, 10])),
                                      (B.ND_KHOP, 30_000, dict(num_steps=2, fanout=[25, 57])),
                                      (B.ND_KHOP, 30_000, dict(num_steps=2, fanout=[25, 3], sched_sub_max=64)),
                                      (B.ND_DEEPWALK, 800_001, dict(num_steps=2, use_weights=1)),
                                      (B.ND_NODE2VEC, 800_001, dict(num_steps=3, p=0.5, q=2.0))])
def test_many_pairs_are_shared_out_by_neighbourhoods(graph, app, S, kw):
    """More pairs than 256 for each group of lanes: whole pairs per round, draws that cross a round's end (57), some
    transits in the other classes; against the sample-parallel kernel."""
    g, dg, _ = graph
    kw = dict(kw, use_weights=int(bool(kw.get("use_weights")) and g.weights is not None))
    if "sched_sub_max" not in kw:
        kw["sched_force_class"] = B.ND_CLASS_SUBWAVE
    r = torch.from_numpy(_roots(g.V, S, 3)).cuda()
    outs = []
    for mode in (dict(mode=B.ND_MODE_SAMPLE_PARALLEL), {}):
        use = {k: v for k, v in kw.items() if not (mode and k.startswith("sched"))}
        s = B.Sampler(dg, app, B.nd_params_init(**use, **mode), S)
        outs.append([o.clone() for o in s.run(r, 17)])
        torch.cuda.synchronize()
        s.status()
    for a, b in zip(*outs):
        assert torch.equal(a, b)
    if app == B.ND_KHOP:
        assert int((outs[0][0] >= 0).sum()) >= 2048 * 256


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("V,int64_offsets,S,R", [((1 << 20) + 37, True, 8200, 9), (1 << 21, False, 8192, 5)])
def test_multi_dimensional_walk_where_rows_are_empty(V, int64_offsets, S, R, weighted):
    """Half of the rows are empty, the last one as well as the one before, and which they are is looked up in bits: many
    samples of 100 steps, whose roots are picked before and after step 64, against the oracle."""
    rng = np.random.default_rng(V)
    deg = rng.integers(1, 4, V)
    deg[rng.random(V) < 0.5] = 0
    deg[:3], deg[-2:] = (0, 1, 0), (2, 0)
    off = np.concatenate([[0], np.cumsum(deg)])
    n = int(off[-1])
    # ascending within a row: a start and steps of at least one
    start, gap = rng.integers(0, V - 8, V), rng.integers(1, 4, V)
    row = np.repeat(np.arange(V), deg)
    col = (start[row] + gap[row] * (np.arange(n) - off[:-1][row])).astype(np.int32)
    off = off.astype(np.int64 if int64_offsets else np.int32)
    w = (1.0 + rng.random(n)).astype(np.float32) if weighted else None
    dg, og = B.nd_graph_create(off, col, w), oracle.OracleGraph(off, col, w)
    roots = rng.integers(0, V, S * R, dtype=np.int32)
    roots[::13] = -1
    roots[1::17], roots[2::17] = V - 1, V - 2
    want = oracle.multirw(og, roots, R, 100, seed=5)
    got, _ = gpu_sample(dg, B.ND_MULTIRW, roots, 5, num_steps=100, roots_per_sample=R)
    assert_steps_equal(got, list(want), f"V={V}")


@pytest.mark.parametrize("V,int64_offsets,R,steps", [((1 << 20) + 37, True, 30, 100), (1 << 21, False, 100, 70),
                                                     (1 << 21, False, 100, 200)])
def test_multi_dimensional_walk_of_many_roots_where_rows_are_empty(V, int64_offsets, R, steps):
    """As many roots as it takes for the bits of empty rows to be read (the routes are pinned on the host): one launch whose
    second round is short, and two of which the second has both rounds."""
    rng = np.random.default_rng(V + R)
    deg = rng.integers(1, 4, V)
    deg[rng.random(V) < 0.5] = 0
    deg[:3], deg[-2:] = (0, 1, 0), (2, 0)
    off = np.concatenate([[0], np.cumsum(deg)])
    start, gap = rng.integers(0, V - 8, V), rng.integers(1, 4, V)
    row = np.repeat(np.arange(V), deg)
    col = (start[row] + gap[row] * (np.arange(off[-1]) - off[:-1][row])).astype(np.int32)
    off = off.astype(np.int64 if int64_offsets else np.int32)
    dg, og = B.nd_graph_create(off, col), oracle.OracleGraph(off, col)
    roots = rng.integers(0, V, 8192 * R, dtype=np.int32)
    roots[::13] = -1
    roots[1::17], roots[2::17] = V - 1, V - 2
    want = oracle.multirw(og, roots, R, steps, seed=6)
    got, _ = gpu_sample(dg, B.ND_MULTIRW, roots, 6, num_steps=steps, roots_per_sample=R)
    assert_steps_equal(got, list(want), f"V={V}")


@pytest.mark.parametrize("V", [1, 63, 64, 65, 257])
def test_offsets_of_few_rows(V):
    """Errors in the offsets, and none, where rows fill a wavefront or a workgroup and where they do not."""
    col = np.zeros(1, np.int32)
    for v in {0, V // 2, V - 1}:  # the only entry is of row v
        off = (np.arange(V + 1) > v).astype(np.int64)
        dg = B.nd_graph_create(off, col)
        got, _ = gpu_sample(dg, B.ND_DEEPWALK, np.arange(V, dtype=np.int32), 1, num_steps=1)
        assert got[0].tolist() == [0 if i == v else -1 for i in range(V)]
        for at, by in ((V, 1), (0, 1), (v, 2), (v + 1, -2)):
            bad = off.copy()
            bad[at] += by
            with pytest.raises(B.NdError):
                B.nd_graph_create(bad, col)
