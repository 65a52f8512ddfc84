"""Batches of many graphs through the lane-per-pair kernel: as many graphs as are
looked at together, more than the launch has blocks, empty ones, and one that
every block has to help with."""
import numpy as np
import pytest

from oracle import native
from workloads import from_edge_lists, powerlaw_hypergraph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("groups", [1, 0])
@pytest.mark.parametrize("blocks", [1, 8])
@pytest.mark.parametrize("n", [2, 7, 8, 9, 17, 200, 1500])
def test_counts(n, blocks, groups):
    import paper_2310_15668_amd as M
    kinds = [powerlaw_hypergraph(20 + 3 * x, 30 + 7 * x, 1, 6, 2.2, 0.6, seed=x) for x in range(13)]
    kinds += [from_edge_lists([[0, 1], [2]], 3), from_edge_lists([], 0)]
    big = powerlaw_hypergraph(700, 2000, 2, 9, 2.5, 0.5, seed=77)  # no row of 512 neighbours
    refs = [native.mochy_e(h, nthreads=8) for h in kinds + [big]]
    order = [(4 * x + x // 15) % 15 for x in range(n)]
    order[n // 2] = 15
    hs = [(kinds + [big])[k] for k in order]
    print(f"[gpu] {n} graphs, blocks {blocks}, groups {groups}", flush=True)
    with M.Context(0) as ctx:
        ctx.set_option(M.MOCHY_OPT_PAIR_BLOCKS, blocks)
        ctx.set_option(M.MOCHY_OPT_GROUPS, groups)
        counts = M.mochy_profile(ctx, [(h.edge_ptr, h.edge_nodes, h.num_nodes) for h in hs])[0]
    for x, k in enumerate(order):
        r26, r431, inv = refs[k]
        assert inv == 0 and (counts[x, :26] == r26).all() and (counts[x, 26:] == r431).all(), x
