"""What a context keeps after a request stays within the bytes that the server
admits it at (and whole pages of its buffers)."""
import numpy as np
import pytest

from workloads import from_edge_lists, powerlaw_hypergraph

pytestmark = pytest.mark.gpu

PAGES = 96 << 20  # up to 48 buffers of 2 MiB pages


def _flat(E, V, size, seed):
    rows = np.unique(np.sort(np.random.default_rng(seed).integers(0, V, size=(E, size)), axis=1), axis=0)
    return from_edge_lists(rows[(np.diff(rows, axis=1) > 0).all(axis=1)].tolist(), V)


CASES = {
    "flat-20000": lambda: [_flat(20000, 40000, 3, s) for s in (1, 2)],
    "flat-50000": lambda: [_flat(50000, 100000, 3, 1), _flat(100000, 200000, 2, 2)],
    "skewed": lambda: [powerlaw_hypergraph(3000, 9000, 2, 12, 2.5, 0.8, seed=s) for s in (3, 4)],
    "long-lists": lambda: [_flat(12000, 700, 2, s) for s in (5, 6, 7)],
}


@pytest.mark.parametrize("name", list(CASES))
def test_request_stays_within(name):
    import torch
    import paper_2310_15668_amd as M
    from paper_2310_15668_amd.serving import request_bytes
    graphs = [(h.edge_ptr, h.edge_nodes, h.num_nodes) for h in CASES[name]()]
    bound = request_bytes(graphs)
    print(f"[gpu] {name}: admitted at {bound >> 20} MiB", flush=True)
    with M.Context(0) as ctx:
        M.mochy_profile(ctx, [(np.array([0, 2], np.int64), np.array([0, 1], np.int32), 2)] * 2)
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info(0)[0]
        M.mochy_profile(ctx, graphs)
        torch.cuda.synchronize()
        held = before - torch.cuda.mem_get_info(0)[0]
    print(f"[gpu] {name}: {held >> 20} MiB kept", flush=True)
    assert held <= bound + PAGES
