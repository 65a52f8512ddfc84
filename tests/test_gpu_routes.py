"""Which kernels the rules choose, on either side of each line: the counts of
both sides are compared with the oracle elsewhere."""
import numpy as np
import pytest

from workloads import from_edge_lists, powerlaw_hypergraph

pytestmark = pytest.mark.gpu


def _flat(E, V, size, seed=5):
    rows = np.unique(np.sort(np.random.default_rng(seed).integers(0, V, size=(E, size)), axis=1), axis=0)
    rows = rows[(np.diff(rows, axis=1) > 0).all(axis=1)]
    return from_edge_lists(rows[np.random.default_rng(seed + 1).permutation(len(rows))].tolist(), V)


def _star(d):
    return from_edge_lists([(0,)] + [(0, 1 + x % 3, 4 + x // 2, 4 + d + x) for x in range(d)], 4 + 2 * d)


GRAPHS = {
    "star-64": lambda: _star(64), "star-65": lambda: _star(65), "star-511": lambda: _star(511),
    "star-512": lambda: _star(512), "flat-0.48GB": lambda: _flat(22000, 9000, 3),
    "flat-0.67GB": lambda: _flat(26000, 9000, 3),
    "long-rows": lambda: powerlaw_hypergraph(2500, 42000, 2, 12, 2.5, 0.9, seed=5),
    "small": lambda: powerlaw_hypergraph(300, 400, 2, 6, 2.5, 0.4, seed=1),
}
G, E, MX, T, O, L = "groups", "every_pair", "matrix", "table", "owners", "listed"
EXACT = [
    ("small", 0, 1, {G, T, L}), ("small", 1, 1, {G, O, L}), ("small", 8, 1, {G, O}), ("small", 0, 0, {E, T, L}),
    ("star-511", 0, 1, {G, T, L}), ("star-512", 0, 1, {G, MX, T, L}), ("star-512", 16, 1, {G, T, L}),
    ("flat-0.48GB", 0, 1, {G, T, L}), ("flat-0.67GB", 0, 1, {G, O, L}), ("long-rows", 0, 1, {G, MX, T, L}),
]


@pytest.mark.parametrize("name,faults,groups,want", EXACT)
def test_exact(name, faults, groups, want):
    import paper_2310_15668_amd as M
    h = GRAPHS[name]()
    print(f"[gpu] {name}: |E|={h.num_edges}", flush=True)
    with M.Context(0) as ctx:
        g = M.mochy_project(ctx, h.edge_ptr, h.edge_nodes, h.num_nodes)
        assert M.mochy_last_routes(ctx) == set()
        ctx.set_option(M.MOCHY_OPT_TEST_FAULTS, faults)
        ctx.set_option(M.MOCHY_OPT_GROUPS, groups)
        M.mochy_count_exact(ctx, g)
        assert M.mochy_last_routes(ctx) == want
        if name == "small":
            M.mochy_count_exact_range_noalloc(ctx, g, 0, h.num_edges)
            assert M.mochy_last_routes(ctx) == {E, O}
        g.close()


@pytest.mark.parametrize("centres,want", [(5000, {G, T, L}), (32767, {G, T, L}), (32768, {G, O, L}), (40000, {G, O, L})])
def test_ranges(centres, want):
    """Ranges of up to half the centres, in rows of up to 32,768 bytes, have the
    table although all centres have not."""
    import paper_2310_15668_amd as M
    h = _flat(70000, 9000, 2)
    assert 2 * 32768 <= h.num_edges < 80000
    with M.Context(0) as ctx:
        g = M.mochy_project(ctx, h.edge_ptr, h.edge_nodes, h.num_nodes)
        M.mochy_count_exact_range(ctx, g, 7, 7 + centres)
        assert M.mochy_last_routes(ctx) == want
        g.close()


@pytest.mark.parametrize("n,want", [(16, {G, T, L}), (17, {G, O, L})])
def test_batch(n, want):
    import paper_2310_15668_amd as M
    h = GRAPHS["small"]()
    with M.Context(0) as ctx:
        M.mochy_profile(ctx, [(h.edge_ptr, h.edge_nodes, h.num_nodes)] * n)
        assert M.mochy_last_routes(ctx) == want


@pytest.mark.parametrize("name,faults,want", [("star-64", 0, "edge_scan"), ("star-65", 0, "edge_groups"),
                                              ("star-65", 1, "edge_scan")])
def test_edges(name, faults, want):
    import paper_2310_15668_amd as M
    h = GRAPHS[name]()
    with M.Context(0) as ctx:
        g = M.mochy_project(ctx, h.edge_ptr, h.edge_nodes, h.num_nodes)
        ctx.set_option(M.MOCHY_OPT_TEST_FAULTS, faults)
        M.mochy_count_sampled_edges(ctx, g, 5, 1)
        assert M.mochy_last_routes(ctx) == {want}
        M.mochy_hyperedge_profiles(ctx, g, 0, 5)
        assert M.mochy_last_routes(ctx) == {want}
        g.close()
