"""Line-graph degrees and hyperwedge order of the line-graph-free mode where
part of the neighbours is counted from bitmaps of the dense node lists."""
import random

import numpy as np
import pytest

from oracle import native
from workloads import from_edge_lists, powerlaw_hypergraph

pytestmark = pytest.mark.gpu

LG_FREE = 4


@pytest.fixture(scope="module")
def ctx():
    import paper_2310_15668_amd as M
    c = M.Context(0)
    yield c
    c.close()


def _stars(E, n_dense, seed):
    """E hyperedges: a few nodes in many of them, nodes in one in 100 to one in
    2000 of them (on both sides of what counts as dense), nodes in one or two."""
    rng = random.Random(seed)
    edges = set()
    top = n_dense + 40
    while len(edges) < E:
        e = set(rng.sample(range(n_dense), rng.choice((0, 1, 1, 2, 3) if n_dense > 2 else (0, 1))))
        if rng.random() < 0.5:
            e.add(n_dense + min(39, int(rng.expovariate(0.15))))
        if rng.random() < 0.5 or not e:
            e.add(top + rng.randrange(2 * E))
        edges.add(tuple(sorted(e)))
    edges = sorted(edges)
    rng.shuffle(edges)
    return from_edge_lists(edges, top + 2 * E)


CASES = {  # words of 64 hyperedges, loads of 128, turns of 8192; no dense, all dense
    "1": lambda: from_edge_lists([[0, 1]], 2),
    "63": lambda: _stars(63, 3, 1),
    "64": lambda: _stars(64, 3, 2),
    "65": lambda: _stars(65, 1, 3),
    "128": lambda: _stars(128, 5, 4),
    "129": lambda: _stars(129, 70, 5),
    "8191": lambda: _stars(8191, 70, 6),
    "8193": lambda: _stars(8193, 4, 7),
    "20001": lambda: _stars(20001, 30, 8),
    "flat": lambda: powerlaw_hypergraph(60000, 30000, 1, 5, 2.5, 0.0, seed=9),
    "skewed": lambda: powerlaw_hypergraph(9000, 30000, 1, 25, 2.5, 1.0, seed=10),
}


@pytest.mark.parametrize("name", list(CASES))
def test_degrees_and_order(ctx, name):
    import paper_2310_15668_amd as M
    h = CASES[name]()
    print(f"[gpu] {name}: |E|={h.num_edges} nnz={h.nnz}", flush=True)
    deg, w = native.line_graph_degrees(h, 8)
    g = M.mochy_project(ctx, h.edge_ptr, h.edge_nodes, h.num_nodes, LG_FREE)
    try:
        st = M.mochy_graph_stats(ctx, g)
        assert g.num_hyperwedges == w
        assert st["max_line_degree"] == deg.max()
        assert st["candidates"] == int((deg * (deg - 1) // 2).sum())
        assert st["sum_deg_sq"] == int((deg * deg).sum())
        if w:  # the samples' hyperwedges follow the upper degrees, row by row
            _, _, raw431, _ = M.mochy_count_sampled(ctx, g, 3000, 5)
            _, o431, inv, ow = native.aplus_raw(h, r=3000, seed=5, nthreads=8)
            assert inv == 0 and ow == w
            assert (np.asarray(raw431) == o431).all()
    finally:
        g.close()


def _repeat(kind):
    rng = random.Random(3)
    edges = {tuple(sorted(rng.sample(range(12), rng.choice((2, 3))) + [12 + rng.randrange(4000)])) for _ in range(3000)}
    edges |= {(0, 1), (0, 1, 2), (0, 12 + 4000), (12 + 4001, 12 + 4002), (0, 1, 12 + 4003)}
    again = {"dense": (0, 1), "dense3": (0, 1, 2), "mixed": (0, 12 + 4000), "sparse": (12 + 4001, 12 + 4002),
             "mixed3": (0, 1, 12 + 4003), "none": None}[kind]
    edges = [list(e) for e in sorted(edges)]
    rng.shuffle(edges)
    if again:
        edges.append(list(again))
    ptr = np.zeros(len(edges) + 1, dtype=np.int64)
    ptr[1:] = np.cumsum([len(e) for e in edges])
    return ptr, np.array([v for e in edges for v in e], dtype=np.int32)


@pytest.mark.parametrize("kind", ["dense", "dense3", "mixed", "mixed3", "sparse", "none"])
def test_repeats(ctx, kind):
    import paper_2310_15668_amd as M
    ptr, nodes = _repeat(kind)
    print(f"[gpu] repeat {kind}: |E|={len(ptr) - 1}", flush=True)
    if kind == "none":
        M.mochy_project(ctx, ptr, nodes, 12 + 4004, LG_FREE).close()
        return
    with pytest.raises(M.MochyError) as e:
        M.mochy_project(ctx, ptr, nodes, 12 + 4004, LG_FREE)
    assert e.value.status == -2


@pytest.mark.parametrize("E", [131071, 131073, 262145, 524289, 1048700])
def test_selection_tiles(ctx, E):
    """Rows drawn from one tile of all hyperedges, at the sizes where the tile
    and its block grow, and from several tiles."""
    import paper_2310_15668_amd as M
    rng = np.random.default_rng(E)
    top = np.minimum((rng.pareto(0.5, size=E) * 3).astype(np.int64), 1999)  # a few nodes in many hyperedges
    own = 2000 + np.arange(E)
    nodes = np.stack([top, own], axis=1).astype(np.int32).reshape(-1)
    ptr = np.arange(E + 1, dtype=np.int64) * 2
    print(f"[gpu] selection |E|={E}", flush=True)
    g = M.mochy_project(ctx, ptr, nodes, 2000 + E, LG_FREE)
    try:
        held = np.bincount(top)
        pairs = held * (held - 1) // 2
        assert g.num_hyperwedges == pairs.sum()
        # each sample {i, j} of a node in n hyperedges meets the n - 2 others, all in one class
        raw431 = np.asarray(M.mochy_count_sampled(ctx, g, 4000, 7)[2])
        assert (raw431 > 0).sum() == 1
        order = np.argsort(top, kind="stable")
        first = np.concatenate([[0], np.cumsum(held)])
        place = np.empty(E, dtype=np.int64)
        place[order] = np.arange(E) - first[top[order]]
        up = held[top] - 1 - place  # neighbours above each row
        ends = np.cumsum(up)
        want = sum(int(held[top[int(np.searchsorted(ends, w, side="right"))]]) - 2
                   for w in (sample_wedge(n, 7, int(pairs.sum())) for n in range(4000)))
        assert raw431.sum() == want
    finally:
        g.close()


def sample_wedge(n, seed, W):
    x = native.philox4x32_10([n & 0xffffffff, n >> 32, 0, 0], [seed & 0xffffffff, seed >> 32])
    return ((x[1] << 32 | x[0]) * W) >> 64
