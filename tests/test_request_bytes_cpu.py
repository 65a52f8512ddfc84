"""What a request of the server is admitted at covers the light-pair correction:
its lists, and its table of overlaps where one can be made."""
import numpy as np
import pytest

from oracle import native
from paper_2310_15668_amd.serving import SMALL_TABLE, request_bytes
from workloads import from_edge_lists, powerlaw_hypergraph


def csr(h):
    return h.edge_ptr, h.edge_nodes, h.num_nodes


def flat(E, V, size=3):
    rows = np.unique(np.sort(np.random.default_rng(E).integers(0, V, size=(E, size)), axis=1), axis=0)
    return from_edge_lists(rows[(np.diff(rows, axis=1) > 0).all(axis=1)].tolist(), V)


def base(h):
    deg = np.bincount(h.edge_nodes, minlength=h.num_nodes).astype(np.int64)
    return (16 * (h.num_edges + 1) + 8 * h.nnz + 9 * (h.num_nodes + 1) + 40 * h.num_edges
            + 100 * int((deg * (deg - 1) // 2).sum()))


@pytest.mark.parametrize("E", [500, 5000, 20000])
def test_small_tables_are_covered(E):
    h = flat(E, 2 * E)
    assert h.num_edges ** 2 <= SMALL_TABLE
    assert request_bytes([csr(h)]) >= base(h) + h.num_edges ** 2
    assert request_bytes([csr(h)] * 3) == 3 * request_bytes([csr(h)])


def scanned(h):
    """Row entries that the pairs of light nodes scan: of the two hyperedges the
    one with the shorter row."""
    deg = np.bincount(h.edge_nodes, minlength=h.num_nodes)
    light = np.argsort(-deg, kind="stable")[64:]
    rows = native.line_graph_degrees(h, 8)[0]
    owner = np.repeat(np.arange(h.num_edges), np.diff(h.edge_ptr))
    order = np.argsort(h.edge_nodes, kind="stable")
    ends = np.cumsum(deg)
    total = 0
    for v in light[deg[light] > 1]:
        d = np.sort(rows[owner[order[ends[v] - deg[v]:ends[v]]]])[::-1].astype(np.int64)
        total += int((np.arange(len(d)) * d).sum())
    return total


def test_large_tables():
    sparse = flat(60000, 120000)  # pairs scan far less than 3.6e9 entries: no table
    assert scanned(sparse) < 1 << 20
    assert base(sparse) < request_bytes([csr(sparse)]) < base(sparse) + 64 * sparse.num_edges * 20
    h = powerlaw_hypergraph(8000, 26000, 2, 12, 2.2, 0.9, seed=3)
    assert h.num_edges ** 2 > SMALL_TABLE and scanned(h) > h.num_edges ** 2
    assert request_bytes([csr(h)]) >= base(h) + h.num_edges ** 2
    # beside it the flat one's may be made, if both together scan as many entries
    both = request_bytes([csr(h), csr(sparse)])
    assert both >= base(h) + base(sparse) + min(h.num_edges ** 2 + sparse.num_edges ** 2, scanned(h))


def test_without_light_nodes():
    # 64 nodes are all heavy; of 65 the last in one hyperedge shares no pair
    edges = [[v, (v + 1) % 64] for v in range(64)]
    h = from_edge_lists([sorted(e) for e in edges], 64)
    assert request_bytes([csr(h)]) == base(h)
    h = from_edge_lists([sorted(e) for e in edges] + [[0, 64]], 65)
    assert request_bytes([csr(h)]) == base(h)
    assert request_bytes([]) == 0 and request_bytes([(np.zeros(1, np.int64), np.zeros(0, np.int32), 0)]) == 16 + 9


@pytest.mark.parametrize("ptr", [
    np.append(np.arange(0, 401, 2), 400),        # the last hyperedge is empty
    np.insert(np.arange(0, 401, 2), 5, 8),       # one in the middle
    np.append(np.arange(0, 401, 2), 500),        # past the end
    np.insert(np.arange(0, 401, 2), 3, -1)])     # not increasing
def test_what_the_library_refuses(ptr):
    # such a request is admitted, and its error is given to whoever waits for it
    nodes = np.arange(200).repeat(2)
    deg = np.bincount(nodes)
    assert request_bytes([(ptr, nodes, 200)]) >= 100 * int((deg * (deg - 1) // 2).sum())
