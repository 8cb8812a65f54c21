"""GPU parity for the edges between consecutive layers (Section 4.2, importance
sampling): the C ABI's count + fill against the oracle, entry by entry."""
import numpy as np
import pytest
import torch

import oracle
from paper_2009_06693_amd import binding as B
from paper_2009_06693_amd import inputs

from gpu_util import device_graph

pytestmark = pytest.mark.gpu


def _compare(g, transits, sampled):
    dg, og = device_graph(g)
    t = torch.as_tensor(np.ascontiguousarray(transits, dtype=np.int32), device="cuda:0")
    v = torch.as_tensor(np.ascontiguousarray(sampled, dtype=np.int32), device="cuda:0")
    print(f"[edges] S={t.shape[0]} n_prev={t.shape[1]} m={v.shape[1]}", flush=True)
    row_ptr, slots = B.layer_edges(dg, t, v)
    torch.cuda.synchronize()
    want_ptr, want_slots = oracle.layer_edges(og, transits, sampled)
    assert np.array_equal(row_ptr.cpu().numpy(), want_ptr)
    assert np.array_equal(slots.cpu().numpy(), want_slots)
    return want_ptr


_small = inputs.small_graph()
_small64 = inputs.small_graph(scale=9, edges=9000, seed=17, int64_offsets=True)


@pytest.mark.parametrize("n_prev,m,S", [(1, 1, 1), (64, 64, 7), (64, 2048, 5), (2048, 2048, 3), (100, 777, 9),
                                        (3, 65, 300), (513, 1, 4),
                                        (2049, 2048, 2), (4200, 64, 2)])   # more than one chunk of transit slots
def test_edges_between_random_layers(n_prev, m, S):
    g = _small
    rng = np.random.default_rng(n_prev * 7919 + m)
    transits = rng.integers(-1, g.V, (S, n_prev)).astype(np.int32)
    # new vertices drawn from the transits' neighbourhoods so that edges are plentiful, with repeats
    deg = np.diff(g.row_offsets)
    pool = g.col_indices[: max(1, g.E // 3)]
    sampled = pool[rng.integers(0, pool.size, (S, m))].astype(np.int32)
    sampled[rng.random((S, m)) < 0.05] = -1
    ptr = _compare(g, transits, sampled)
    if n_prev >= 64 and m >= 64:
        assert ptr[-1] > 0


def test_edges_of_a_sampled_layer_call_with_int64_offsets():
    g = _small64
    dg, og = device_graph(g)
    S, R = 6, 16
    roots = inputs.permutation(g.V, 3)[:S * R].copy()
    p = B.nd_params_init(num_steps=2, fanout=[300, 500], roots_per_sample=R)
    r = torch.as_tensor(roots, device="cuda:0")
    s = B.Sampler(dg, B.ND_LAYER, p, S * R)
    out = s.run(r, 9)
    torch.cuda.synchronize()
    layers = [roots.reshape(S, R), out[0].cpu().numpy().reshape(S, 300), out[1].cpu().numpy().reshape(S, 500)]
    for i in range(2):
        ptr = _compare(g, layers[i], layers[i + 1])
        assert ptr[-1] >= layers[i + 1].shape[1] * S   # every drawn vertex is some transit's neighbour


def test_every_vertex_once_reads_back_the_adjacency_rows():
    g = inputs.small_graph(scale=8, edges=2500, seed=4)
    dg, _ = device_graph(g)
    V = g.V
    ids = torch.arange(V, dtype=torch.int32, device="cuda:0").reshape(1, V)
    row_ptr, slots = B.layer_edges(dg, ids, ids.clone())
    assert np.array_equal(row_ptr.cpu().numpy(), g.row_offsets.astype(np.int64))
    assert np.array_equal(slots.cpu().numpy(), g.col_indices)


@pytest.mark.parametrize("copies", [2, 9, 70, 2048])
def test_a_vertex_held_by_many_slots_gives_one_edge_per_slot(copies):
    """Runs of equal vertices of every length class: written lane by lane up to 8, by the search over
    running sums above, and more than one 64-wide group of outputs per queue drain at 70 and 2,048."""
    g = _small
    deg = np.diff(g.row_offsets)
    hub = int(np.argmax(deg))
    nbrs = g.col_indices[g.row_offsets[hub]:g.row_offsets[hub + 1]]
    m = 2048
    rng = np.random.default_rng(copies)
    sampled = rng.integers(0, g.V, (2, m)).astype(np.int32)
    sampled[0, rng.choice(m, copies, replace=False)] = nbrs[0]          # one neighbour of the hub, many times
    sampled[1, :] = nbrs[rng.integers(0, nbrs.size, m)] if copies == 2048 else sampled[1]
    transits = np.full((2, 40), hub, dtype=np.int32)
    transits[:, 1::2] = rng.integers(0, g.V, (2, 20))
    ptr = _compare(g, transits, sampled)
    assert ptr[1] - ptr[0] >= copies


@pytest.mark.parametrize("int64_offsets", [False, True])
def test_adjacency_lists_that_end_at_and_around_the_kernels_step_sizes(int64_offsets):
    """A wavefront streams a list in steps of 256 or 512 entries, 64 at a time: lists one short of,
    equal to and one past the multiples, with the vertices looked for at their very ends."""
    lengths = [1, 63, 64, 65, 255, 256, 257, 511, 512, 513, 767, 768, 1023, 1024, 1025, 1536, 2047, 2048, 2049, 4097]
    V = 5000
    rng = np.random.default_rng(77)
    edges = []
    for u, n in enumerate(lengths):
        edges += [(u, int(v)) for v in np.sort(rng.choice(V, n, replace=False))]
    g = inputs.from_edges(V, edges, int64_offsets=int64_offsets)
    transits = np.array([np.arange(len(lengths)), np.arange(len(lengths))[::-1]], dtype=np.int32)
    ends = [int(g.col_indices[g.row_offsets[u + 1] - 1]) for u in range(len(lengths))]   # the last entry of each list
    firsts = [int(g.col_indices[g.row_offsets[u]]) for u in range(len(lengths))]
    sampled = np.array([ends + firsts, rng.integers(0, V, 2 * len(lengths)).tolist()], dtype=np.int32)
    ptr = _compare(g, transits, sampled)
    assert ptr[len(lengths)] >= 2 * len(lengths) - 1     # every list holds its own first and last entry


def test_empty_and_error_cases():
    g = _small
    dg, _ = device_graph(g)
    e = torch.empty((0, 5), dtype=torch.int32, device="cuda:0")
    row_ptr, slots = B.layer_edges(dg, e, torch.empty((0, 9), dtype=torch.int32, device="cuda:0"))
    assert row_ptr.cpu().tolist() == [0] and slots.numel() == 0
    t = torch.zeros((2, 4), dtype=torch.int32, device="cuda:0")
    with pytest.raises(B.NdError) as err:
        B.layer_edges(dg, t, torch.zeros((2, B.ND_MAX_EDGE_SLOTS + 1), dtype=torch.int32, device="cuda:0"))
    assert err.value.code == B.ND_ERR_TOO_LARGE
    bad = torch.full((2, 4), g.V, dtype=torch.int32, device="cuda:0")
    with pytest.raises(B.NdError) as err:
        B.layer_edges(dg, bad, t)
    assert err.value.code == B.ND_ERR_BAD_ROOT
    # a short edge buffer is filled up to its capacity and not beyond
    rng = np.random.default_rng(1)
    tr = torch.as_tensor(rng.integers(0, g.V, (3, 50)).astype(np.int32), device="cuda:0")
    sv = torch.as_tensor(g.col_indices[rng.integers(0, g.E, (3, 400))].astype(np.int32), device="cuda:0")
    row_ptr, full = B.layer_edges(dg, tr, sv)
    assert full.numel() > 10
    short = torch.full((full.numel(),), -7, dtype=torch.int32, device="cuda:0")
    B.nd_layer_edges_fill(dg, tr, sv, row_ptr, short[: full.numel() // 2])
    torch.cuda.synchronize()
    half = full.numel() // 2
    assert torch.equal(short[:half], full[:half]) and bool((short[half:] == -7).all())


def test_edges_among_the_vertices_of_one_step():
    """Cluster-style use (Section 4.2, "Cluster Sampling": an edge is recorded when it joins two
    transits of the same step): the same array on both sides."""
    g = _small
    rng = np.random.default_rng(77)
    hubs = np.argsort(-np.diff(g.row_offsets))[:400].astype(np.int32)
    members = hubs[rng.integers(0, hubs.size, (6, 300))]
    members[rng.random(members.shape) < 0.03] = -1
    ptr = _compare(g, members, members)
    assert ptr[-1] > 0


@pytest.mark.parametrize("n_prev", [150, 2300])
def test_an_edge_array_that_ends_anywhere_is_filled_up_to_there(n_prev):
    """Rows are stored as offsets inside the rows of a chunk of slots: arrays that end before, in and after rows of
    transits that one slot holds, or 70 slots do, in the first chunk and (2,300 slots) in the second."""
    g = _small
    dg, _ = device_graph(g)
    rng = np.random.default_rng(5)
    tr = rng.integers(0, g.V, (2, n_prev)).astype(np.int32)
    hub = int(np.argmax(np.diff(g.row_offsets)))
    tr[:, rng.permutation(n_prev)[:70]] = hub
    sv = np.concatenate([g.col_indices[rng.integers(0, g.E, (2, 300))], g.col_indices[g.row_offsets[hub]:][:40][None].repeat(2, 0)], 1)
    tr, sv = (torch.as_tensor(x.astype(np.int32), device="cuda:0") for x in (tr, sv))
    row_ptr, full = B.layer_edges(dg, tr, sv)
    ends = [0, 1, 2, 63, 64, 65] + [int(row_ptr[i]) + d for i in (n_prev // 2, n_prev - 1, n_prev, n_prev + 1) for d in (-1, 0, 1, 30)]
    if n_prev > 2048:
        ends += [int(row_ptr[i]) + d for i in (2047, 2048, n_prev + 2048) for d in (-1, 0, 1)]
    for end in sorted({e for e in ends if 0 <= e <= full.numel()} | {full.numel() - 1}):
        short = torch.full((full.numel(),), -7, dtype=torch.int32, device="cuda:0")
        B.nd_layer_edges_fill(dg, tr, sv, row_ptr, short[:end])
        torch.cuda.synchronize()
        assert torch.equal(short[:end], full[:end]) and bool((short[end:] == -7).all()), end


def test_lists_that_start_beyond_four_billion_entries():
    """The places of lists are kept as 32 bits and five more: 4.3 G entries, rows on both sides of 2^32."""
    V, degree = 70_000, 62_000
    if torch.cuda.mem_get_info()[0] < 60 << 30:
        pytest.skip("needs 60 GB of free device memory")
    col = torch.arange(degree, dtype=torch.int32, device="cuda:0").repeat(V)
    for shift in range(1, 8):                                # row v holds the vertices from v % 8 on
        col.view(V, degree)[shift::8] += shift
    dg = B.nd_graph_create(torch.arange(V + 1, device="cuda:0") * degree, col)
    del col
    last = (1 << 32) // degree
    rng = np.random.default_rng(9)
    tr = np.array([[0, last - 1, last, last + 1, V - 1, last, 5], [V - 1, V - 2, 3, last, -1, 7, last + 8]], dtype=np.int32)
    sv = rng.integers(0, 9, (2, 40)).astype(np.int32)
    sv[:, 20:] = rng.integers(degree - 4, degree + 9, (2, 20))
    row_ptr, slots = B.layer_edges(dg, torch.as_tensor(tr, device="cuda:0"), torch.as_tensor(sv, device="cuda:0"))
    row_ptr, slots = row_ptr.cpu().numpy(), slots.cpu().numpy()
    for i, t in enumerate(tr.reshape(-1)):
        row = sv[i // tr.shape[1]]
        first = t % 8
        want = [j for j in np.lexsort((np.arange(row.size), row)) if t >= 0 and first <= row[j] < degree + first]
        assert slots[row_ptr[i]:row_ptr[i + 1]].tolist() == want, (i, t)


def _fill_time(dg, transits, sampled):
    """The least time of a filling pass, ms."""
    S, n = transits.shape
    row_ptr = torch.empty(S * n + 1, dtype=torch.int64, device="cuda:0")
    ws = torch.empty(max(B.nd_layer_edges_workspace_bytes(S, n), 256), dtype=torch.uint8, device="cuda:0")
    B.nd_layer_edges_count(dg, transits, sampled, row_ptr, ws)
    assert int(row_ptr[-1]) == 0
    slots = torch.empty(1, dtype=torch.int32, device="cuda:0")
    marks = [torch.cuda.Event(enable_timing=True) for _ in range(12)]
    for m in marks:
        B.nd_layer_edges_fill(dg, transits, sampled, row_ptr, slots)
        m.record()
    torch.cuda.synchronize()
    return min(a.elapsed_time(b) for a, b in zip(marks, marks[1:]))


def test_a_vertex_in_every_slot_is_ordered_about_as_fast_as_different_ones():
    """Leaves of a star and no edges between them, so that a filling pass is its preparation: each slot that looks at
    every other one of its vertex took 167 us where different vertices take 19 and a bitmap per vertex 32.  Three times
    is between."""
    V = 4001
    g = inputs.from_edges(V, [(0, v) for v in range(1, V)] + [(v, 0) for v in range(1, V)])
    dg, _ = device_graph(g)
    S = 512
    tr = (1 + torch.arange(S * 64, device="cuda:0") % (V - 1)).to(torch.int32).view(S, 64)
    different = _fill_time(dg, tr, torch.arange(1, 2049, device="cuda:0", dtype=torch.int32).repeat(S, 1))
    one = _fill_time(dg, tr, torch.full((S, 2048), 7, device="cuda:0", dtype=torch.int32))
    print(f"[times] different vertices {different:.4f} ms, one {one:.4f} ms", flush=True)
    assert one < 3 * different


@pytest.mark.parametrize("runs", [[2048], [65, 64, 63, 66], [1023, 1025], [65] * 31 + [33], [128, 129, 1, 64, 700, 2]])
def test_slots_of_a_vertex_leave_in_order_whatever_their_number(runs):
    """Runs around 64 slots, up to which each slot looks at the others, as many longer ones as there can be, and all slots."""
    g = _small
    hub = int(np.argmax(np.diff(g.row_offsets)))
    nbrs = g.col_indices[g.row_offsets[hub]:g.row_offsets[hub + 1]]
    assert nbrs.size >= len(runs)
    rng = np.random.default_rng(len(runs))
    sampled = np.full((3, 2048), -1, dtype=np.int32)
    for row in sampled:
        row[rng.permutation(2048)[:sum(runs)]] = np.repeat(rng.permutation(nbrs)[:len(runs)], runs)
    transits = rng.integers(0, g.V, (3, 2100)).astype(np.int32)
    transits[:, ::700] = hub
    ptr = _compare(g, transits, sampled)
    assert ptr[1] - ptr[0] == sum(runs)
