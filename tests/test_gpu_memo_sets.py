"""Memoized keys whose neighbours hold many of the heavy-node sets that are
counted: few and many sets, as many as overflow them, neighbours with singles
and pairs of a set but not the triple."""
import random

import numpy as np
import pytest

from oracle import native
from workloads import from_edge_lists

pytestmark = pytest.mark.gpu


def _heavy(heavy, sizes, seed, E=500):
    """Hyperedges of a few of `heavy` common nodes and a light one or two."""
    rng = random.Random(seed)
    edges = set()
    while len(edges) < E:
        e = set(rng.sample(range(heavy), min(heavy, rng.choice(sizes))))
        e |= {heavy + rng.randrange(400) for _ in range(rng.randint(1, 2))}
        edges.add(tuple(sorted(e)))
    edges = sorted(edges)
    rng.shuffle(edges)
    return from_edge_lists(edges, heavy + 400)


CASES = {"2": (2, (1, 2)), "3": (3, (1, 2, 3)), "singles": (40, (1,)), "pairs": (40, (1, 2)), "12": (12, (1, 2, 3, 5)),
         "64": (64, (1, 2, 3)), "wide": (64, (4, 9, 15))}


@pytest.mark.parametrize("pool", [0, 1])
@pytest.mark.parametrize("name", list(CASES))
def test_sets(name, pool):
    import paper_2310_15668_amd as M
    heavy, sizes = CASES[name]
    h = _heavy(heavy, sizes, 60 + heavy)
    print(f"[gpu] memo sets {name}, pool {pool}: |E|={h.num_edges}", flush=True)
    o431 = native.aplus_raw(h, r=20000, seed=9, nthreads=8)[1]
    with M.Context(0) as c:
        c.set_option(M.MOCHY_OPT_MEMO_ALL, 1)
        c.set_option(M.MOCHY_OPT_MEMO_POOL, pool)
        for flags in (0, 4):  # stored rows, and none
            g = M.mochy_project(c, h.edge_ptr, h.edge_nodes, h.num_nodes, flags)
            try:
                raw431 = M.mochy_count_sampled(c, g, 20000, 9)[2]
                assert (np.asarray(raw431) == o431).all()
                if flags:
                    assert M.mochy_memo_stats(c)["memo_samples"] > 0
            finally:
                g.close()
