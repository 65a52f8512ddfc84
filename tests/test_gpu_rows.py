"""Line-graph rows and records at the sizes where they are cut: words and tiles
of the row bitmap, lists taken as bitmaps or walked, entries put off, graphs of
a batch that start inside a word."""
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


def _sparse(E, seed):
    """E hyperedges, few neighbours each; 64 nodes in about E / 40 of them, on
    both sides of what is taken as a bitmap."""
    rng = random.Random(seed)
    edges = set()
    while len(edges) < E:
        e = {64 + rng.randrange(3 * E)}
        if rng.random() < 0.6:
            e.add(min(63, int(rng.expovariate(0.05))))
        if rng.random() < 0.3:
            e.add(64 + rng.randrange(3 * E))
        edges.add(tuple(sorted(e)))
    edges = sorted(edges)
    rng.shuffle(edges)
    return from_edge_lists(edges, 64 + 3 * E)


def _wide(E, seed):
    """Hyperedges of 25 to 32 of 80 nodes: nearly all share light nodes."""
    rng = random.Random(seed)
    edges = set()
    while len(edges) < E:
        edges.add(tuple(sorted(rng.sample(range(80), rng.randint(25, 32)))))
    return from_edge_lists(sorted(edges), 80)


CASES = {
    "31": lambda: _sparse(31, 1), "32": lambda: _sparse(32, 2), "33": lambda: _sparse(33, 3),
    "8191": lambda: _sparse(8191, 4), "8192": lambda: _sparse(8192, 5), "8193": lambda: _sparse(8193, 6),
    "16385": lambda: _sparse(16385, 7),
    "wide-511": lambda: _wide(511, 8), "wide-700": lambda: _wide(700, 9),
    "flat": lambda: powerlaw_hypergraph(3000, 9000, 1, 4, 2.5, 0.0, seed=10),
}


@pytest.mark.parametrize("name", list(CASES))
def test_counts(ctx, name):
    import paper_2310_15668_amd as M
    h = CASES[name]()
    print(f"[gpu] rows {name}: |E|={h.num_edges} nnz={h.nnz}", flush=True)
    deg, w = native.line_graph_degrees(h, 8)
    g = M.mochy_project(ctx, h.edge_ptr, h.edge_nodes, h.num_nodes)
    try:
        st = M.mochy_graph_stats(ctx, g)
        assert g.num_hyperwedges == w and st["max_line_degree"] == deg.max()
        assert st["sum_deg_sq"] == int((deg * deg).sum())
        c26, c431 = M.mochy_count_exact(ctx, g)
        r26, r431, _ = native.mochy_e(h, nthreads=8)
        assert (np.asarray(c431) == r431).all() and (np.asarray(c26) == r26).all()
        if w:  # the records' masks and the hyperwedges' order
            raw431 = M.mochy_count_sampled(ctx, g, 2000, 3)[2]
            o431 = native.aplus_raw(h, r=2000, seed=3, nthreads=8)[1]
            assert (np.asarray(raw431) == o431).all()
    finally:
        g.close()


def test_graphs_of_a_batch(ctx):
    import paper_2310_15668_amd as M
    hs = [_sparse(n, 20 + n) for n in (33, 1, 64, 95, 31)] + [_wide(100, 30), powerlaw_hypergraph(50, 300, 1, 8, 2.0, 0.9, seed=31)]
    print("[gpu] rows of a batch", flush=True)
    counts = M.mochy_profile(ctx, [(h.edge_ptr, h.edge_nodes, h.num_nodes) for h in hs])[0]
    for h, row in zip(hs, counts):
        r26, r431, _ = native.mochy_e(h, nthreads=8)
        assert (row[:26] == r26).all() and (row[26:] == r431).all()


@pytest.mark.parametrize("extra", [[0, 1], [0, 70], [70, 71]])
def test_repeats(ctx, extra):
    """A repeated hyperedge of heavy nodes, of both, and of light nodes."""
    import paper_2310_15668_amd as M
    h = powerlaw_hypergraph(200, 900, 2, 6, 2.0, 0.9, seed=40)
    rows = {tuple(h.edge_nodes[h.edge_ptr[x]:h.edge_ptr[x + 1]].tolist()) for x in range(h.num_edges)}
    rows = [list(r) for r in sorted(rows | {tuple(extra)})] + [extra]
    ptr = np.zeros(len(rows) + 1, dtype=np.int64)
    ptr[1:] = np.cumsum([len(r) for r in rows])
    print(f"[gpu] repeat {extra}", flush=True)
    with pytest.raises(M.MochyError) as e:
        M.mochy_project(ctx, ptr, np.array([v for r in rows for v in r], dtype=np.int32), 200)
    assert e.value.status == -2
