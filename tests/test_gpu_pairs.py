"""Pairs of neighbour groups of long rows (the matrix-core pair kernels).

Rows of at least 512 groups take them; each hypergraph here has such rows at a
place where they can go wrong, and the counts are compared with every-pair
counting (no groups) and with the oracle.
"""
import itertools
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


def _star(count, extra, centre_size=25):
    """A centre whose `count` neighbours all have distinct records: a node of
    the centre and a distinct set of `extra` of 60 nodes that are all heavy."""
    sets = itertools.islice(itertools.combinations(range(100, 160), extra), -(-count // 4))
    edges = [list(range(centre_size))] + [[a, *s] for s in sets for a in range(4)][:count]
    return from_edge_lists(edges, 160)


def _wide(seed):
    """Large hyperedges: centres of 29 to 32 nodes (31 and 32 leave no mask bit
    for a window's slot), neighbours sharing more than 3 nodes with them and
    holding more than 7 heavy ones."""
    rng = random.Random(seed)
    edges = set()
    for n in (29, 30, 31, 32):
        for _ in range(2):
            edges.add(tuple(sorted(rng.sample(range(40), n))))
    while len(edges) < 3000:
        n = rng.choice((2, 3, 3, 4, 4, 5, 6, 9, 14))
        edges.add(tuple(sorted({min(299, int(rng.expovariate(1 / 45))) for _ in range(n)} | {rng.randrange(300)})))
    edges = [e for e in edges if len(e) > 1]
    rng.shuffle(edges)
    return from_edge_lists(edges, 300)


CASES = {
    # 511, 512 and 513 groups above the centre: either side of the row limit
    "511-groups": (lambda: _star(511, 2), (0, 1)),
    "512-groups": (lambda: _star(512, 2), (0, 40)),
    "513-groups": (lambda: _star(513, 2), (0, 40)),
    # two hash parts: the groups are sorted after the grouping
    "two-parts": (lambda: _star(7080, 2), (0, 12)),
    # more groups above the centre than the sort holds
    "14000-groups": (lambda: _star(14000, 3), (0, 4)),
    "large-hyperedges": (lambda: _wide(5), (0, None)),
    "hub-heavy": (lambda: powerlaw_hypergraph(400, 5000, 1, 25, 2.2, 0.8, seed=31), (0, None)),
    # the range's centres in the middle: groups with and without members above
    "middle": (lambda: powerlaw_hypergraph(2000, 9000, 2, 25, 2.5, 0.9, seed=32), (4000, 4400)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_pairs_against_every_pair(ctx, name):
    import paper_2310_15668_amd as M
    make, (c0, c1) = CASES[name]
    h = make()
    c1 = h.num_edges if c1 is None else c1
    print(f"[gpu] {name}: |E|={h.num_edges}, centres [{c0}, {c1})", flush=True)
    g = M.mochy_project(ctx, h.edge_ptr, h.edge_nodes, h.num_nodes)
    try:
        a26, a431 = M.mochy_count_exact_range(ctx, g, c0, c1)
        st = M.mochy_exact_stats(ctx)
        ctx.set_option(M.MOCHY_OPT_GROUP_CAPACITY, 0)
        b26, b431 = M.mochy_count_exact_range(ctx, g, c0, c1)
        ctx.set_option(M.MOCHY_OPT_GROUPS, 0)
        e26, e431 = M.mochy_count_exact_range(ctx, g, c0, c1)
    finally:
        ctx.set_option(M.MOCHY_OPT_GROUPS, 1)
        ctx.set_option(M.MOCHY_OPT_GROUP_CAPACITY, 144 << 30)
        g.close()
    assert st["groups"] > 0 and int(e431.sum()) > 0
    assert (a431 == e431).all() and (a26 == e26).all()
    assert (b431 == e431).all() and (b26 == e26).all()
    some = list(range(c0, c1, max(1, (c1 - c0) // 8)))[:8] if c1 - c0 > 8 else list(range(c0, c1))
    if name != "14000-groups":
        o26, o431, inv = native.mochy_e_centers(h, some)
        g = M.mochy_project(ctx, h.edge_ptr, h.edge_nodes, h.num_nodes)
        s431 = np.zeros(431, np.int64)
        try:
            for c in some:
                s431 += M.mochy_count_exact_range(ctx, g, c, c + 1)[1]
        finally:
            g.close()
        assert inv == 0 and (s431 == o431).all()
