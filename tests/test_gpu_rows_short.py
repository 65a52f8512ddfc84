"""Line-graph rows and records of hypergraphs with more hyperedges than one tile
of the row bitmap (8,192): rows on either side of the short-row kernel (256
neighbours) and of a single sweep (4,096), against the oracle."""
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


def _stars(degrees, E, seed, heavy=90):
    """A centre with rows of exactly d for each d: nodes of its own shared by d
    hyperedges.  The other hyperedges hold one of `heavy` nodes and nodes of
    their own, up to E in all, in any order."""
    rng = random.Random(seed)
    edges, v = [], heavy
    for d in degrees:
        centre = list(range(v, v + 3))
        edges.append(centre)
        edges += [sorted({centre[x % 3], v + 3 + x // 2, v + 3 + d + x}) for x in range(d)]
        v += 3 + 2 * d
    while len(edges) < E:
        edges.append([min(heavy - 1, int(rng.expovariate(0.02))), v] + ([v + 1] if rng.random() < 0.5 else []))
        v += 2
    rng.shuffle(edges)
    return from_edge_lists(edges, v + 2)


CASES = {
    "8192": (lambda: _stars([0, 1, 255, 256, 257], 8192, 1), 1500),
    "8193": (lambda: _stars([0, 1, 2, 31, 63, 64, 255, 256, 257, 258], 8193, 2), 1500),
    "20000": (lambda: _stars([255, 256, 257, 600], 20000, 3), 250),
    "4096": (lambda: _stars([4095], 8300, 4), 40), "4097": (lambda: _stars([4097, 4096], 9300, 5), 40),
    "flat": (lambda: powerlaw_hypergraph(9000, 12000, 1, 4, 2.5, 0.0, seed=10), None),
    "skewed": (lambda: powerlaw_hypergraph(9000, 14000, 1, 12, 2.2, 0.6, seed=11), 200),
}


@pytest.mark.parametrize("name", list(CASES))
def test_counts(ctx, name):
    import paper_2310_15668_amd as M
    make, some = CASES[name]
    h = make()
    print(f"[gpu] rows {name}: |E|={h.num_edges} nnz={h.nnz}", flush=True)
    deg, w = native.line_graph_degrees(h, 8)
    g = M.mochy_project(ctx, h.edge_ptr, h.edge_nodes, h.num_nodes)
    try:
        st = M.mochy_graph_stats(ctx, g)
        assert g.num_hyperwedges == w and st["max_line_degree"] == deg.max()
        assert st["sum_deg_sq"] == int((deg * deg).sum())
        for c0 in (0,) if some is None else (0, h.num_edges // 2, h.num_edges - some):
            c1 = h.num_edges if some is None else c0 + some
            c26, c431 = M.mochy_count_exact_range(ctx, g, c0, c1)
            r26, r431, inv = native.mochy_e(h, c0, c1, nthreads=8)
            assert inv == 0 and (c431 == r431).all() and (c26 == r26).all(), (c0, c1)
        # the records' masks and the hyperwedges' order, from the stored rows and without
        o431 = native.aplus_raw(h, r=3000, seed=3, nthreads=8)[1]
        for rows in (1, 0):
            ctx.set_option(M.MOCHY_OPT_APLUS_ROWS, rows)
            assert (np.asarray(M.mochy_count_sampled(ctx, g, 3000, 3)[2]) == o431).all()
    finally:
        ctx.set_option(M.MOCHY_OPT_APLUS_ROWS, 0)
        g.close()


def test_batch(ctx):
    import paper_2310_15668_amd as M
    hs = [_stars([1, 300], 700, 6), _stars([255, 257], 8200, 7), from_edge_lists([[0, 1]], 2), _stars([256], 8193, 8),
          powerlaw_hypergraph(50, 300, 1, 8, 2.0, 0.9, seed=31)]
    print(f"[gpu] rows of a batch, |E|={[h.num_edges for h in hs]}", flush=True)
    counts = M.mochy_profile(ctx, [(h.edge_ptr, h.edge_nodes, h.num_nodes) for h in hs])[0]
    for h, row in zip(hs, counts):
        r26, r431, _ = native.mochy_e(h, nthreads=8)
        assert (row[:26] == r26).all() and (row[26:] == r431).all()


@pytest.mark.parametrize("d", [2, 256, 257, 5000])
def test_repeats(ctx, d):
    """Two hyperedges alike, in rows of d."""
    import paper_2310_15668_amd as M
    edges = [[0, 1], *([0, 2 + x] for x in range(d - 1)), *([5002 + 2 * x, 5003 + 2 * x] for x in range(8200)), [0, 1]]
    ptr = np.zeros(len(edges) + 1, dtype=np.int64)
    ptr[1:] = np.cumsum([len(e) for e in edges])
    print(f"[gpu] repeat in rows of {d}", flush=True)
    with pytest.raises(M.MochyError) as e:
        M.mochy_project(ctx, ptr, np.array([v for e in edges for v in e], dtype=np.int32), 5004 + 2 * 8200)
    assert e.value.status == -2
