"""Hyperedge samples and profiles by scanning rows (rows of up to 64 neighbours,
or no memory for the groups), against the oracle: rows on either side of the
line, lists of work items, and the scan where the groups are the usual way."""
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


def _star(d):
    """One node in d + 1 hyperedges (rows of d entries) that share others."""
    return from_edge_lists([(0,)] + [(0, 1 + x % 3, 4 + x // 2, 4 + d + x) for x in range(d)], 4 + 2 * d)


CASES = {
    "none": (lambda: from_edge_lists([[0, 1], [2, 3], [4]], 5), 0),
    "star-1": (lambda: _star(1), 0),
    "star-63": (lambda: _star(63), 0),
    "star-64": (lambda: _star(64), 0),
    "star-65": (lambda: _star(65), 0),
    "flat": (lambda: powerlaw_hypergraph(6000, 3000, 2, 4, 2.5, 0.0, seed=1), 0),
    # bit 0: the scratch is refused; items of 256 neighbours at their edges
    "star-256-scan": (lambda: _star(256), 1),
    "star-257-scan": (lambda: _star(257), 1),
    "wide-scan": (lambda: powerlaw_hypergraph(500, 900, 1, 32, 1.2, 0.5, seed=8), 1),
    "all-heavy-scan": (lambda: powerlaw_hypergraph(60, 700, 1, 12, 2.0, 0.8, seed=9), 1),
}


@pytest.mark.parametrize("name", list(CASES))
def test_scan(ctx, name):
    import paper_2310_15668_amd as M
    make, faults = CASES[name]
    h = make()
    print(f"[gpu] {name}: |E|={h.num_edges} nnz={h.nnz}", flush=True)
    g = M.mochy_project(ctx, h.edge_ptr, h.edge_nodes, h.num_nodes)
    ctx.set_option(M.MOCHY_OPT_TEST_FAULTS, faults)
    try:
        rows = min(h.num_edges, 900)
        p26, p431 = M.mochy_hyperedge_profiles(ctx, g, 0, rows)
        o26, o431, inv = native.hyperedge_profiles(h, 0, rows, nthreads=8)
        assert (inv == 0).all()
        assert (p431 == o431).all() and (p26 == o26).all()
        for s, begin in ((1, 0), (300, 7), (5000, 1 << 33)):
            raw431 = M.mochy_count_sampled_edges(ctx, g, s, 3, begin)[2]
            _, s431, sinv, _ = native.mochy_a_raw(h, s=s, seed=3, n0=begin, nthreads=8)
            assert sinv == 0 and (raw431 == s431).all()
    finally:
        ctx.set_option(M.MOCHY_OPT_TEST_FAULTS, 0)
        g.close()


def test_several_batches(ctx):
    """More samples than one batch: the oracle's hits, by how often each
    hyperedge is drawn."""
    import paper_2310_15668_amd as M
    h = powerlaw_hypergraph(40, 60, 1, 5, 2.0, 0.3, seed=10)
    n = (1 << 20) + 77
    print(f"[gpu] scan batches: |E|={h.num_edges}", flush=True)
    g = M.mochy_project(ctx, h.edge_ptr, h.edge_nodes, h.num_nodes)
    try:
        raw431 = M.mochy_count_sampled_edges(ctx, g, n, 4)[2]
        _, o431, inv, _ = native.mochy_a_raw(h, s=n, seed=4, nthreads=8)
        assert inv == 0 and (raw431 == o431).all()
    finally:
        g.close()


@pytest.mark.parametrize("faults", [0, 1])
@pytest.mark.parametrize("name,E", [("group", 146000), ("group", 148000), ("group", 200000), ("flat", 190000)])
def test_many_hyperedges(ctx, name, E, faults):
    """Bitmaps of a row over 146,000 to 200,000 hyperedges: with their own LDS the
    kernels' blocks take up to 74 KB.  `group`: one row longer than is scanned."""
    import paper_2310_15668_amd as M
    rng = np.random.default_rng(E)
    a = rng.integers(0, E, size=E).astype(np.int64)
    a[:90] = E
    nodes = np.stack([a, E + 1 + np.arange(E) % (E - 7), 2 * E + 1 + np.arange(E)], axis=1)
    if name == "flat":
        nodes = nodes[90:]
    n = len(nodes)
    h = from_edge_lists(nodes.tolist(), 3 * E + 1)
    print(f"[gpu] {name} {E}, faults {faults}: |E|={h.num_edges}", flush=True)
    g = M.mochy_project(ctx, h.edge_ptr, h.edge_nodes, h.num_nodes)
    ctx.set_option(M.MOCHY_OPT_TEST_FAULTS, faults)
    try:
        for lo, hi in ((0, 200), (n - 200, n)):
            p26, p431 = M.mochy_hyperedge_profiles(ctx, g, lo, hi)
            o26, o431, inv = native.hyperedge_profiles(h, lo, hi, nthreads=8)
            assert (inv == 0).all() and int(o431.sum()) > 0
            assert (p431 == o431).all() and (p26 == o26).all()
        raw431 = M.mochy_count_sampled_edges(ctx, g, 20000, 3)[2]
        _, s431, sinv, _ = native.mochy_a_raw(h, s=20000, seed=3, nthreads=8)
        assert sinv == 0 and (raw431 == s431).all()
        if faults == 0:  # rows, records and the correction of as many
            c431 = M.mochy_count_exact(ctx, g)[1]
            assert (c431 == native.mochy_e(h, nthreads=8)[1]).all()
    finally:
        ctx.set_option(M.MOCHY_OPT_TEST_FAULTS, 0)
        g.close()
