"""Rows of 127 to 129 neighbour groups, on either side of the line between the
lane-per-pair kernel and the matrix-core kernels, with and without a row long
enough in the hypergraph for the latter to be launched at all."""
import itertools

import numpy as np
import pytest

from oracle import native
from workloads import from_edge_lists

pytestmark = pytest.mark.gpu


def _star(count, first):
    """A centre of 8 nodes from `first` on, and `count` neighbours of distinct
    records: one of its nodes and a distinct pair of 16 others."""
    sets = itertools.islice(itertools.combinations(range(first + 8, first + 24), 2), -(-count // 8))
    return [list(range(first, first + 8))] + [[a, *s] for s in sets for a in range(first, first + 8)][:count]


@pytest.mark.parametrize("count", [127, 128, 129, 255, 257])
@pytest.mark.parametrize("long_row", [0, 511, 512])
def test_row_limit(count, long_row):
    import paper_2310_15668_amd as M
    edges = _star(count, 0) + ([[100], *[[100, 101 + x] for x in range(long_row)]] if long_row else [])
    h = from_edge_lists([sorted(e) for e in edges], 101 + long_row)
    print(f"[gpu] {count} groups, row of {long_row}: |E|={h.num_edges}", flush=True)
    with M.Context(0) as ctx:
        g = M.mochy_project(ctx, h.edge_ptr, h.edge_nodes, h.num_nodes)
        try:
            c26, c431 = M.mochy_count_exact(ctx, g)
        finally:
            g.close()
    r26, r431, _ = native.mochy_e(h, nthreads=8)
    assert (np.asarray(c431) == r431).all() and (np.asarray(c26) == r26).all()
