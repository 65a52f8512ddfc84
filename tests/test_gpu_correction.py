"""The light-pair correction from the table of overlaps, against the oracle and
against the path that takes the pairs owner by owner (two listing passes)."""
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


def _light_degrees(degrees, seed):
    """64 heavy nodes in many hyperedges, and one light node of each degree: a
    unit of the candidate list holds 4 owners, so the degrees stand at its
    edges."""
    rng = random.Random(seed)
    edges = {tuple(sorted(rng.sample(range(64), rng.choice((2, 3, 4))))) for _ in range(900)}
    v = 64
    for d in degrees:
        while d:
            e = tuple(sorted(rng.sample(range(64), rng.choice((1, 2, 5, 18))) + [v]))
            if e not in edges:
                edges.add(e)
                d -= 1
        v += 1
    edges = sorted(edges)
    rng.shuffle(edges)
    return from_edge_lists(edges, v)


CASES = {
    "degrees": (lambda: _light_degrees([2, 3, 4, 5, 6, 8, 9, 10, 13, 16, 17, 33], 1), (None, (0, 1), (100, 517))),
    "one-light-pair": (lambda: _light_degrees([2], 2), (None,)),
    "many-light": (lambda: powerlaw_hypergraph(3000, 2500, 1, 25, 2.2, 0.4, seed=3), (None, (700, 1300))),
    # 40,000 hyperedges: rows of the table long enough for a queue per XCD
    "long-rows": (lambda: powerlaw_hypergraph(30000, 40000, 2, 6, 2.5, 0.35, seed=4), (None, (39000, 39999))),
}


@pytest.mark.parametrize("name", list(CASES))
def test_correction_paths(ctx, name):
    import paper_2310_15668_amd as M
    make, ranges = CASES[name]
    h = make()
    g = M.mochy_project(ctx, h.edge_ptr, h.edge_nodes, h.num_nodes)
    try:
        for c0, c1 in [(0, h.num_edges) if r is None else r for r in ranges]:
            print(f"[gpu] {name}: |E|={h.num_edges}, centres [{c0}, {c1})", flush=True)
            a26, a431 = M.mochy_count_exact_range(ctx, g, c0, c1)
            sa = M.mochy_exact_stats(ctx)
            ctx.set_option(M.MOCHY_OPT_TEST_FAULTS, 8)
            b26, b431 = M.mochy_count_exact_range(ctx, g, c0, c1)
            sb = M.mochy_exact_stats(ctx)
            ctx.set_option(M.MOCHY_OPT_TEST_FAULTS, 0)
            r26, r431, inv = native.mochy_e(h, c0, c1)
            assert inv == 0 and sa["light_pairs"] > 0
            assert (a431 == r431).all() and (a26 == r26).all(), np.nonzero(a431 != r431)
            assert (b431 == r431).all() and (b26 == r26).all()
            for k in ("light_pairs", "fix_scanned", "fix_centres", "fix_changed"):
                assert sa[k] == sb[k], k
    finally:
        ctx.set_option(M.MOCHY_OPT_TEST_FAULTS, 0)
        g.close()


def test_correction_of_a_batch(ctx):
    # graphs of different sizes, one without a light pair, in one set
    import paper_2310_15668_amd as M
    graphs = [_light_degrees(list(range(2, 20)), 5), _light_degrees([], 6),
              powerlaw_hypergraph(2000, 1500, 1, 12, 2.2, 0.5, seed=7), _light_degrees([2, 40], 8)]
    print(f"[gpu] batch |E|={[h.num_edges for h in graphs]}", flush=True)
    counts = M.mochy_profile(ctx, [(h.edge_ptr, h.edge_nodes, h.num_nodes) for h in graphs])[0]
    for x, h in enumerate(graphs):
        r26, r431, inv = native.mochy_e(h)
        assert inv == 0
        assert (counts[x, :26] == r26).all() and (counts[x, 26:] == r431).all(), x
