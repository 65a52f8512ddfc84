"""Small buffers kept by the context: calls of changing sizes give the same
counts with and without, and a limit of 0 gives everything back."""
import numpy as np
import pytest

from oracle import native
from workloads import powerlaw_hypergraph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("limit", [None, 0, 3000, 1 << 20])
def test_small_buffers(limit):
    import paper_2310_15668_amd as M
    hs = [powerlaw_hypergraph(40 + 90 * x, 60 + 130 * x, 1, 8, 2.2, 0.8, seed=50 + x) for x in range(5)]
    refs = [native.mochy_e(h, nthreads=8)[1] for h in hs]
    a431 = native.mochy_a_raw(hs[2], s=40, seed=2, nthreads=8)[1]
    with M.Context(0) as c:
        if limit is not None:
            c.set_option(M.MOCHY_OPT_CACHE_BYTES, limit)
        for turn, order in enumerate(([0, 1, 2, 3, 4], [4, 3, 2, 1, 0], [2, 0, 4, 1, 3])):
            print(f"[gpu] cache limit {limit}, turn {turn}", flush=True)
            kept = []
            for x in order:  # two graphs alive at a time
                h = hs[x]
                kept.append((x, M.mochy_project(c, h.edge_ptr, h.edge_nodes, h.num_nodes)))
                for y, g in kept:
                    assert (np.asarray(M.mochy_count_exact(c, g)[1]) == refs[y]).all()
                    if y == 2:
                        assert (np.asarray(M.mochy_count_sampled_edges(c, g, 40, 2)[2]) == a431).all()
                if len(kept) == 2:
                    kept.pop(0)[1].close()
            for _, g in kept:
                g.close()
            if turn == 1:
                c.set_option(M.MOCHY_OPT_CACHE_BYTES, 0)  # gives back what is kept
