"""Exact counts where the choice of the 64 heavy nodes is at its edges: fewer
than 64 nodes in two hyperedges, ties for the last place, nodes in one to three
levels of blocks.  A node given two bits, or a bit given twice, shows as wrong
overlaps."""
import random

import numpy as np
import pytest

from oracle import cp, native
from workloads import from_edge_lists, powerlaw_hypergraph

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2310_15668_amd as M
    c = M.Context(0)
    yield c
    c.close()


def _spread(V, E, seed, smax=5):
    """E hyperedges over a few hundred of V nodes spread over all of them, so that
    the nodes in most hyperedges lie in different blocks; many of one degree."""
    rng = random.Random(seed)
    pool = sorted(rng.sample(range(V), min(V, 300)) if V > 300 else range(V))
    pool = sorted(set(pool) | {0, V - 1})
    edges = set()
    for _ in range(50 * E):
        if len(edges) == E:
            break
        edges.add(tuple(sorted(rng.sample(pool, min(len(pool), rng.randint(1, smax))))))
    return from_edge_lists(sorted(edges), V)


CASES = {
    "few": lambda: _spread(20, 200, 1),
    "63": lambda: _spread(63, 400, 2),
    "64": lambda: _spread(64, 400, 3),
    "65": lambda: _spread(65, 400, 4),
    "pairs": lambda: from_edge_lists([[x, (x + 1) % 500] if x < 499 else [0, 499] for x in range(500)], 500),
    "1025": lambda: _spread(1025, 500, 5),
    "8192": lambda: _spread(8192, 500, 6),
    "8193": lambda: _spread(8193, 500, 7),
    "70001": lambda: _spread(70001, 500, 8),
    "1048577": lambda: _spread(1048577, 500, 9),
}


@pytest.mark.parametrize("name", list(CASES))
def test_exact_counts(ctx, name):
    import paper_2310_15668_amd as M
    h = CASES[name]()
    print(f"[gpu] heavy {name}: |V|={h.num_nodes} |E|={h.num_edges}", flush=True)
    g = M.mochy_project(ctx, h.edge_ptr, h.edge_nodes, h.num_nodes)
    try:
        c26, c431 = M.mochy_count_exact(ctx, g)
    finally:
        g.close()
    r26, r431, _ = native.mochy_e(h, nthreads=8)
    assert (np.asarray(c431) == r431).all()
    assert (np.asarray(c26) == r26).all()


@pytest.mark.parametrize("copies", [1, 15, 16, 17, 33])
def test_profile_of_many_copies(ctx, copies):
    """As many graphs as the profile kernel reads at a time, one more, one less."""
    import paper_2310_15668_amd as M
    hs = [powerlaw_hypergraph(60 + 7 * x, 80 + x, 1, 6, 2.0, 0.7, seed=20 + x) for x in range(copies + 1)]
    print(f"[gpu] profile of {copies} copies", flush=True)
    counts, sig26, cp26, sig431, cp431 = M.mochy_profile(ctx, [(h.edge_ptr, h.edge_nodes, h.num_nodes) for h in hs])
    for h, row in zip(hs, counts):
        r26, r431, _ = native.mochy_e(h, nthreads=8)
        assert (row[:26] == r26).all() and (row[26:] == r431).all()
    for lo, hi, sig, prof in ((0, 26, sig26, cp26), (26, 457, sig431, cp431)):
        d = cp.significance(counts[0, lo:hi].tolist(), [r[lo:hi].tolist() for r in counts[1:]], 1.0)
        np.testing.assert_allclose(sig, d, rtol=1e-12, atol=1e-300)
        np.testing.assert_allclose(prof, cp.characteristic_profile(d), rtol=1e-12, atol=1e-300)
