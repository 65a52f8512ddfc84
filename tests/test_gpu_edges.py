"""Hyperedge samples and profiles from groups of neighbours, against the oracle:
at the sizes where rows, groups, work items and node lists are cut."""
import random

import numpy as np
import pytest

from oracle import native
from workloads import from_edge_lists, powerlaw_hypergraph

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2310_15668_amd as M
    c = M.Context(0)
    yield c
    c.close()


def _lists(degrees, seed, small=700):
    """64 heavy nodes in many hyperedges, and light nodes of the given degrees,
    two of them in some hyperedges (a pair then shares one or several)."""
    rng = random.Random(seed)
    edges = {tuple(sorted(rng.sample(range(64), rng.choice((1, 2, 3, 4))))) for _ in range(small)}
    v = 64
    for d in degrees:
        while d > 0:
            e = set(rng.sample(range(64), rng.choice((1, 2, 5, 18)))) | {v}
            if rng.random() < 0.4:
                e |= {u for u in (v - 1, v - 2) if u >= 64}
            e = tuple(sorted(e))
            if e not in edges:
                edges.add(e)
                d -= 1
        v += 1
    edges = sorted(edges)
    rng.shuffle(edges)
    return from_edge_lists(edges, v)


def _star(d, seed):
    """One node in d + 1 hyperedges: rows of exactly d entries."""
    rng = random.Random(seed)
    edges = [(0,)] + [tuple([0] + sorted(rng.sample(range(1, 40), rng.choice((1, 2, 3)))) + [40 + x]) for x in range(d)]
    return from_edge_lists(edges, 40 + d)


CASES = {
    "star-1": lambda: _star(1, 1),
    "star-255": lambda: _star(255, 2),
    "star-257": lambda: _star(257, 3),
    "star-513": lambda: _star(513, 4),
    "star-1025": lambda: _star(1025, 5),
    # lists of 2 to 200 members, 63 to 65 and 128 at the edges of what is held
    "lists": lambda: _lists([2, 3, 31, 63, 64, 65, 66, 127, 128, 129, 200], 6),
    # short rows: few neighbours for each light node
    "sparse": lambda: powerlaw_hypergraph(4000, 3000, 1, 6, 2.5, 0.3, seed=7),
    "wide": lambda: powerlaw_hypergraph(500, 900, 1, 32, 1.2, 0.5, seed=8),
    "all-heavy": lambda: powerlaw_hypergraph(60, 700, 1, 12, 2.0, 0.8, seed=9),
}


@pytest.mark.parametrize("name", list(CASES))
def test_profiles(ctx, name):
    import paper_2310_15668_amd as M
    h = CASES[name]()
    print(f"[gpu] {name}: |E|={h.num_edges} nnz={h.nnz}", flush=True)
    g = M.mochy_project(ctx, h.edge_ptr, h.edge_nodes, h.num_nodes)
    try:
        rows = h.num_edges if h.num_edges < 1000 else 48  # the oracle's pairs are quadratic in the degree
        p26, p431 = M.mochy_hyperedge_profiles(ctx, g, 0, rows)
        o26, o431, inv = native.hyperedge_profiles(h, 0, rows, nthreads=8)
        assert (inv == 0).all()
        assert (p431 == o431).all(), np.argwhere(p431 != o431)[:5]
        assert (p26 == o26).all()
        _, _, raw431, _ = M.mochy_count_sampled_edges(ctx, g, 31, 3)
        s26, s431, sinv, _ = native.mochy_a_raw(h, s=31, seed=3, nthreads=8)
        assert sinv == 0 and (raw431 == s431).all()
    finally:
        g.close()


def test_several_batches(ctx):
    """More samples than one batch of scratch holds (here by its row limit):
    the sum over two calls is the one call's."""
    import paper_2310_15668_amd as M
    h = powerlaw_hypergraph(40, 60, 1, 5, 2.0, 0.6, seed=10)
    print(f"[gpu] batches: |E|={h.num_edges}", flush=True)
    g = M.mochy_project(ctx, h.edge_ptr, h.edge_nodes, h.num_nodes)
    try:
        n = 32768 + 100
        raw431 = M.mochy_count_sampled_edges(ctx, g, n, 4)[2]
        a = M.mochy_count_sampled_edges(ctx, g, 32768, 4)[2]
        b = M.mochy_count_sampled_edges(ctx, g, 100, 4, 32768)[2]
        assert (np.asarray(a) + np.asarray(b) == np.asarray(raw431)).all()
        _, o431, inv, _ = native.mochy_a_raw(h, s=n, seed=4, nthreads=8)
        assert inv == 0 and (raw431 == o431).all()
    finally:
        g.close()


@pytest.mark.parametrize("a,b", [(16000, 17000), (23000, 24000)])
def test_large_groups(ctx, a, b):
    """All hyperedges share one node: a of two nodes and b of three.  A row has
    two groups, whose pairs fill 4-byte counters over several samples (33,000
    hyperedges) or at once (47,000)."""
    import paper_2310_15668_amd as M
    nodes, sizes, v = [], [], 1
    for x in range(a + b):
        c = 1 if x < a else 2
        nodes += [0] + list(range(v, v + c))
        sizes.append(1 + c)
        v += c
    ptr = np.zeros(a + b + 1, dtype=np.int64)
    ptr[1:] = np.cumsum(sizes)
    print(f"[gpu] large groups: |E|={a + b}", flush=True)
    g = M.mochy_project(ctx, ptr, np.array(nodes, dtype=np.int32), v)
    try:
        pairs = lambda n: n * (n - 1) // 2
        of = {2: sorted([pairs(a - 1), (a - 1) * b, pairs(b)]), 3: sorted([pairs(a), a * (b - 1), pairs(b - 1)])}
        p431 = M.mochy_hyperedge_profiles(ctx, g, a - 3, a + 3)[1]
        for x, row in enumerate(p431):
            assert sorted(row[row > 0].tolist()) == of[2 if x < 3 else 3]
        raw431 = np.asarray(M.mochy_count_sampled_edges(ctx, g, 23, 3)[2])
        assert raw431.sum() == 23 * pairs(a + b - 1)
    finally:
        g.close()
