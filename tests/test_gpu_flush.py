"""The kernels with 32-bit counters, made to empty them every few additions while
other waves add (fault bit 4; otherwise after 2^24 entries or 2^26 visits of a
wave): the every-pair kernel and the light-pair correction on its table."""
import numpy as np
import pytest

from oracle import native
from workloads import powerlaw_hypergraph

pytestmark = pytest.mark.gpu

CASES = {
    "skewed": lambda: powerlaw_hypergraph(900, 2500, 2, 12, 2.5, 0.9, seed=4),
    "many-light": lambda: powerlaw_hypergraph(3000, 2500, 1, 25, 2.2, 0.4, seed=3),
}


@pytest.mark.parametrize("name", list(CASES))
def test_counts(name):
    import paper_2310_15668_amd as M
    h = CASES[name]()
    print(f"[gpu] {name}: |E|={h.num_edges}", flush=True)
    with M.Context(0) as ctx:
        g = M.mochy_project(ctx, h.edge_ptr, h.edge_nodes, h.num_nodes)
        ctx.set_option(M.MOCHY_OPT_TEST_FAULTS, 16)
        for c0, c1 in [(0, h.num_edges), (300, 800)]:
            r26, r431, inv = native.mochy_e(h, c0, c1, nthreads=8)
            for groups in (1, 0):
                ctx.set_option(M.MOCHY_OPT_GROUPS, groups)
                c26, c431 = M.mochy_count_exact_range(ctx, g, c0, c1)
                st = M.mochy_exact_stats(ctx)
                assert inv == 0 and st["fix_changed"] > 0
                assert (c431 == r431).all() and (c26 == r26).all(), (groups, np.nonzero(c431 != r431))
        g.close()


def _scanned(h):
    """(candidate pairs of the light nodes, row entries they scan)."""
    deg = np.bincount(h.edge_nodes, minlength=h.num_nodes)
    rows = native.line_graph_degrees(h, 8)[0]
    owner = np.repeat(np.arange(h.num_edges), np.diff(h.edge_ptr))
    order = np.argsort(h.edge_nodes, kind="stable")
    ends = np.cumsum(deg)
    pairs = entries = 0
    for v in np.argsort(-deg, kind="stable")[64:]:
        d = np.sort(rows[owner[order[ends[v] - deg[v]:ends[v]]]])[::-1].astype(np.int64)
        pairs += len(d) * (len(d) - 1) // 2
        entries += int((np.arange(len(d)) * d).sum())
    return pairs, entries


def test_long_rows_of_the_table():
    """36,000 hyperedges: rows of the table above 32,768 bytes, whose units the
    waves pull from a queue for each XCD.  The same counts as owner by owner,
    from the list and from two listings, and with the counters emptied early."""
    import paper_2310_15668_amd as M
    h = powerlaw_hypergraph(2500, 42000, 2, 12, 2.5, 0.9, seed=5)
    pairs, entries = _scanned(h)
    # as many pairs as have such queues, of rows that the table is made for
    assert h.num_edges > 32768 and pairs > 4 * 65536
    assert entries > h.num_edges ** 2 and entries * 25 > pairs * h.num_edges
    print(f"[gpu] long rows: |E|={h.num_edges}", flush=True)
    with M.Context(0) as ctx:
        g = M.mochy_project(ctx, h.edge_ptr, h.edge_nodes, h.num_nodes)
        got = {}
        for faults in (0, 1, 8, 16):
            ctx.set_option(M.MOCHY_OPT_TEST_FAULTS, faults)
            got[faults] = M.mochy_count_exact(ctx, g)[1], M.mochy_exact_stats(ctx)
        g.close()
    assert got[0][1]["fix_changed"] > 0
    for f in (1, 8, 16):
        assert (got[f][0] == got[0][0]).all(), f
        assert got[f][1]["fix_changed"] == got[0][1]["fix_changed"]
