"""Graphs that have no links, because a quarter of the free device memory does not hold them: the check of
their rows, and the routes that look rows up instead - walks in windows, k-hop grouped by transit, layer
sampling step by step - as a call without scheduling parameters takes them, against the oracle.  The rest
of the device's memory is taken while the graphs are made, and given back before they are used."""
import gc

import numpy as np
import pytest
import torch

import oracle
from paper_2009_06693_amd import binding as B

from gpu_util import assert_steps_equal, gpu_sample

pytestmark = pytest.mark.gpu

V = 120_000
LEFT = 1 << 30   # bytes that stay free: the graphs below take 0.1 to 0.25 GB each without their links, 0.3 GB of links


class _TakenMemory:
    """All but about LEFT bytes of the device's memory, in pieces of 16 GB and less."""

    def __enter__(self):
        gc.collect()
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        self.pieces = []
        size = 16 << 30
        while size >= 64 << 20:
            if torch.cuda.mem_get_info()[0] - size >= LEFT:
                self.pieces.append(torch.empty(size, dtype=torch.uint8, device="cuda:0"))
            else:
                size //= 2
        print(f"[memory] {torch.cuda.mem_get_info()[0] >> 20} MB left", flush=True)
        return self

    def __exit__(self, *_):
        self.pieces.clear()
        torch.cuda.empty_cache()


def _csr(entries):
    """Skewed columns, some empty rows, one row that holds half of the vertices."""
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(entries)
    u = torch.randint(0, V, (entries,), generator=gen, device="cuda:0")
    v = (torch.rand(entries, generator=gen, device="cuda:0", dtype=torch.float64) ** 2 * V).to(torch.int64)
    u[u % 11 == 5] = 0
    key = torch.unique(torch.cat([(u << 32) | v, (3 << 32) | torch.arange(0, V, 2, device="cuda:0")]))
    off = torch.searchsorted(key, torch.arange(V + 1, device="cuda:0") << 32)
    return off.to(torch.int64).cpu().numpy(), (key & 0x7FFFFFFF).to(torch.int32).cpu().numpy()


def _refused(off, col, w):
    """Creates graphs with one bad entry each; [(what is said, the error)]."""
    last = int(np.flatnonzero(np.diff(off) > 1)[-1])
    at = int(off[last]) + 1
    got = []
    for place, value, say in ((at, col[at - 1], "ascending"), (at, col[at - 1] - 1, "ascending"),
                              (col.size - 1, V, "column"), (0, -1, "column")):
        bad = col.copy()
        bad[place] = value
        try:
            B.nd_graph_create(off, bad, w)
            got.append((say, None))
        except B.NdError as e:
            got.append((say, e))
    return got


@pytest.fixture(scope="module")
def graphs():
    """All of them while the memory is taken once (it takes seconds)."""
    made = {}
    for name, weighted, wide in (("plain32", False, False), ("weighted64", True, True), ("plain64", False, True)):
        off, col = _csr(10_000_000 if weighted else 20_000_000)
        if not wide:
            off = off.astype(np.int32)
        w = 1.0 + 4.0 * np.random.default_rng(3).random(col.size, dtype=np.float32) if weighted else None
        made[name] = [off, col, w]
    with _TakenMemory():
        for m in made.values():
            off, col, w = m
            assert col.size * (32 if w is not None else 16) > torch.cuda.mem_get_info()[0] // 4
            m.append(B.nd_graph_create(off, col, w))
            m.append(_refused(off, col, w))
            m.append(oracle.OracleGraph(off, col, w))
    yield made
    for m in made.values():
        m[3].destroy()


@pytest.fixture(params=["plain32", "weighted64", "plain64"])
def graph(request, graphs):
    off, col, w, dg, _, og = graphs[request.param]
    return off, col, w, dg, og


def _roots(n, seed):
    r = np.random.default_rng(seed).integers(0, V, size=n, dtype=np.int32)
    r[::17] = -1
    return r


@pytest.mark.parametrize("steps,S", [(1, 1), (129, 300), (2, (1 << 21) + 5)])
def test_walks(graph, steps, S):
    _, _, w, dg, og = graph
    roots = _roots(S, 1)
    for weighted in ((0, 1) if w is not None else (0,)):
        kw = dict(num_steps=steps, use_weights=weighted)
        want = oracle.deepwalk(og, roots, steps, seed=2, use_weights=bool(weighted))
        got, stats = gpu_sample(dg, B.ND_DEEPWALK, roots, 2, **kw)
        assert_steps_equal(got, list(want), "deepwalk")
        # only routes that group count distinct transits
        assert [bool(x) for x in stats[:, 1]] == [bool((x >= 0).any()) for x in [roots] + list(want[:-1])]
        got, _ = gpu_sample(dg, B.ND_PPR, roots, 3, term_prob=0.02, **kw)
        assert_steps_equal(got, list(oracle.ppr(og, roots, steps, 0.02, seed=3, use_weights=bool(weighted))), "ppr")
        if S < 1000:
            got, _ = gpu_sample(dg, B.ND_NODE2VEC, roots, 4, p=2.0, q=0.5, **kw)
            assert_steps_equal(got, list(oracle.node2vec(og, roots, steps, 2.0, 0.5, seed=4,
                                                         use_weights=bool(weighted))), "node2vec")


@pytest.mark.parametrize("R,steps,S", [(1, 130, 70), (100, 65, 300)])
def test_multi_dimensional_walk(graph, R, steps, S):
    _, _, _, dg, og = graph
    roots = _roots(R * S, 5)
    got, stats = gpu_sample(dg, B.ND_MULTIRW, roots, 6, num_steps=steps, roots_per_sample=R)
    assert_steps_equal(got, list(oracle.multirw(og, roots, R, steps, seed=6)), "multirw")
    assert stats[0, 1] > 0


@pytest.mark.parametrize("fanout,S,rounds", [([25, 10], 1000, 0), ([3, 2, 1, 2], 3000, 0), ([16, 2], 257, 4)])
def test_khop(graph, fanout, S, rounds):
    _, _, _, dg, og = graph
    roots = _roots(S, 7)
    got, stats = gpu_sample(dg, B.ND_KHOP, roots, 8, num_steps=len(fanout), fanout=fanout, unique_rounds=rounds)
    assert_steps_equal(got, oracle.khop(og, roots, fanout, seed=8, unique_rounds=rounds), "k-hop")
    assert stats[0, 1] > 0


@pytest.mark.parametrize("per,fanout,S", [(1, [1], 1), (64, [512], 513), (64, [513, 7], 64), (512, [4096, 512], 2),
                                          (4096, [9, 4096], 2)])
def test_layer(graph, per, fanout, S):
    _, _, w, dg, og = graph
    roots = _roots(per * S, 9)
    for weighted in ((0, 1) if w is not None else (0,)):
        got, _ = gpu_sample(dg, B.ND_LAYER, roots, 10, num_steps=len(fanout), fanout=fanout, roots_per_sample=per,
                            use_weights=weighted)
        assert_steps_equal(got, oracle.layer(og, roots, per, fanout, seed=10, use_weights=bool(weighted)),
                           f"layer per={per} {fanout} weighted={weighted}")


@pytest.mark.parametrize("name", ["plain32", "weighted64", "plain64"])
def test_bad_rows_are_refused(graphs, name):
    """Without links the check of the rows is a pass of its own, for unweighted graphs too."""
    refused = graphs[name][4]
    assert len(refused) == 4
    for say, e in refused:
        assert e is not None and e.code == B.ND_ERR_BAD_GRAPH and say in str(e)
