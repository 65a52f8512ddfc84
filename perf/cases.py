"""The work this framework is timed on: what a program that counts hypergraph
motifs calls, over the sizes it calls it at.

A case names one entry point (``kind``) and a seeded synthetic hypergraph:
``nodes`` and ``edges`` drawn, hyperedge sizes from a truncated power law
(exponent ``gamma`` on [smin, smax]), members by Zipf node weights (exponent
``alpha``), repeated hyperedges dropped; the recipe of the repository's
workload generator, drawn on the GPU here so that inputs are quick to make.

kinds
  exact      one hypergraph, projected and counted exactly
  range      one range of centres of a projected hypergraph (a resumable count
             works through such ranges)
  noalloc    the allocation-free exact count of a projected hypergraph
  aplus      hyperwedge sampling on a projected hypergraph
  free       projection without a stored line graph, then hyperwedge sampling
  edges      hyperedge sampling on a projected hypergraph
  profiles   per-hyperedge profiles of a range of a projected hypergraph
  cp         significance and characteristic profile of a hypergraph against
             stub-matched copies, in one call
"""
import functools
import itertools
import math

import numpy as np
import torch

import paper_2310_15668_amd as M

COUNTED = ("exact", "range", "noalloc", "cp")  # kinds whose counts a plain count gives


def _case(name, kind, nodes, edges, smax=25, smin=2, gamma=2.5, alpha=1.0, samples=0, copies=0, host=False):
    return {"name": name, "kind": kind, "nodes": nodes, "edges": edges, "smin": smin, "smax": smax,
            "gamma": gamma, "alpha": alpha, "samples": samples, "copies": copies, "host": host}


def listed():
    return [
        # the tiny workload: a call where launches, allocations and read-backs are the time
        _case("exact-tiny", "exact", 300, 500, smax=8),
        # a serving-sized hypergraph (the median request) given as host arrays
        _case("exact-small-host", "exact", 1803, 4507, host=True),
        # the largest hypergraph of the default serving stream
        _case("exact-20k", "exact", 8004, 20011),
        # the headline workload: 100,000 hyperedges drawn over 20,000 nodes
        _case("exact-medium", "exact", 20000, 100000),
        # one step of a resumable count over the headline workload: 4,096 centres
        _case("range-medium", "range", 20000, 100000, samples=4096),
        # the count for callers that may not allocate (graph capture, tight loops)
        _case("noalloc-small", "noalloc", 2411, 6029),
        # a million hyperwedge samples of the headline workload
        _case("aplus-medium", "aplus", 20000, 100000, samples=1_000_000),
        # a hypergraph too large for a stored line graph (a fifth of the large
        # workload), projected and sampled
        _case("free-large", "free", 200_003, 400_009, gamma=2.8, alpha=0.9, samples=1_000_000),
        # a hundred hyperedge samples of the headline workload
        _case("edges-medium", "edges", 20000, 100000, samples=100),
        # per-hyperedge profiles of 1,501 hyperedges of a mid-sized hypergraph
        _case("profiles-mid", "profiles", 5003, 12503, samples=1501),
        # one request of the profile server: a hypergraph and eight copies, host arrays
        _case("cp-request", "cp", 1203, 3001, copies=8, host=True),
        # the batched workload at a twentieth of its size: 64 copies, resident in HBM
        _case("cp-batch", "cp", 2500, 7500, smax=20, alpha=1.1, copies=64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("exact", "exact", "exact", "range", "noalloc", "aplus", "free", "edges", "profiles", "cp", "cp"))
    top = {"exact": 90_000, "range": 90_000, "noalloc": 9_000, "aplus": 90_000, "free": 400_000, "edges": 90_000,
           "profiles": 20_000, "cp": 4_000}[kind]
    edges = _log_int(rng, 3_000 if kind == "free" else 400, top)
    nodes = max(25, int(edges * rng.uniform(0.25, 0.6)))
    samples = {"exact": 0, "noalloc": 0, "cp": 0, "range": _log_int(rng, 64, 8_192), "aplus": _log_int(rng, 1_000, 1_000_000),
               "free": _log_int(rng, 1_000, 1_000_000), "edges": _log_int(rng, 5, 100),
               "profiles": _log_int(rng, 20, 1_500)}[kind]
    copies = _log_int(rng, 2, 24) if kind == "cp" else 0
    gamma, alpha = (2.8, 0.9) if kind == "free" else (rng.choice((2.5, 2.8)), rng.choice((0.9, 1.0)))
    c = _case("", kind, nodes, edges, smax=rng.choice((8, 20, 25)), gamma=gamma, alpha=alpha, samples=samples,
              copies=copies, host=rng.random() < 0.4)
    del c["name"]
    return c


# ---------------------------------------------------------------------------
# Inputs


def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _first_distinct(rows):
    """Sorted padded node lists less repeats: the rows' 64-bit hashes, one row of each."""
    mult = torch.tensor([(0x9E3779B97F4A7C15 * (2 * p + 1) ** 5) % (1 << 63) | 1 for p in range(rows.shape[1])],
                        dtype=torch.int64, device=rows.device)
    x = (rows + 1) * -7046029254386353131
    x = (x ^ (x >> 29)) * mult
    key = (x ^ (x >> 32)).sum(dim=1)
    order = torch.sort(key, stable=True).indices
    k = key[order]
    keep = torch.ones_like(k, dtype=torch.bool)
    keep[1:] = k[1:] != k[:-1]
    return rows[torch.sort(order[keep]).values]


def _csr(rows):
    """(edge_ptr, edge_nodes) of sorted lists padded with -1 at the front."""
    ptr = torch.zeros(rows.shape[0] + 1, dtype=torch.int64, device=rows.device)
    ptr[1:] = torch.cumsum((rows >= 0).sum(dim=1), 0)
    return ptr, rows[rows >= 0].to(torch.int32)


def _pmf(c):
    s = torch.arange(c["smin"], c["smax"] + 1, dtype=torch.float64)
    w = s ** -c["gamma"]
    return s, w / w.sum()


def _hypergraph(c, gen):
    dev = gen.device
    n, v = c["edges"], c["nodes"]
    cdf = torch.cumsum(_pmf(c)[1], 0).to(dev)
    u = torch.rand(n, generator=gen, device=dev, dtype=torch.float64)
    sizes = c["smin"] + torch.clamp(torch.searchsorted(cdf, u, right=True), max=c["smax"] - c["smin"])
    w = torch.cumsum(torch.arange(1, v + 1, dtype=torch.float64) ** -c["alpha"], 0)
    w = (w / w[-1]).to(dev)
    rows = torch.full((n, c["smax"]), -1, dtype=torch.int64, device=dev)
    for p in range(c["smax"]):  # the p-th member, drawn again while it repeats an earlier one
        pending = torch.nonzero(sizes > p).flatten()
        while pending.numel():
            x = torch.searchsorted(w, torch.rand(pending.numel(), generator=gen, device=dev, dtype=torch.float64), right=True)
            x = torch.clamp(x, max=v - 1)
            ok = ~(rows[pending, :p] == x[:, None]).any(dim=1)
            rows[pending[ok], p] = x[ok]
            pending = pending[~ok]
    return _first_distinct(torch.sort(rows, dim=1).values)


def _copy(rows, nodes, gen):
    """Configuration-model copy: node stubs dealt back into the hyperedges' places."""
    held = rows >= 0
    stubs = rows[held]
    out = torch.full_like(rows, -1)
    out[held] = stubs[torch.randperm(stubs.numel(), generator=gen, device=gen.device)]
    out = torch.sort(out, dim=1).values
    out[:, 1:][out[:, 1:] == out[:, :-1]] = -1  # a hyperedge is a set: repeated members collapse
    return _first_distinct(torch.sort(out, dim=1).values)


def _graphs(case, seed):
    """The case's hypergraphs as (edge_ptr, edge_nodes, nodes), on the GPU."""
    gen = torch.Generator(device=_device())
    gen.manual_seed(int(seed))
    rows = _hypergraph(case, gen)
    every = [rows] + [_copy(rows, case["nodes"], gen) for _ in range(case["copies"])]
    return [(*_csr(r), case["nodes"]) for r in every]


@functools.lru_cache(maxsize=1)
def _context():
    return M.Context(0)  # a program keeps one context


def prepare(case, seed):
    graphs = _graphs(case, seed)
    if case["host"]:
        graphs = [(p.cpu().numpy(), n.cpu().numpy(), v) for p, n, v in graphs]
    torch.cuda.synchronize()  # the library works on its own stream
    state = {"case": case, "ctx": _context(), "graphs": graphs, "seed": int(seed)}
    if case["kind"] in ("range", "noalloc", "aplus", "edges", "profiles"):
        state["projected"] = M.mochy_project(state["ctx"], *graphs[0])
    return state


def run(state):
    case, ctx, kind = state["case"], state["ctx"], state["case"]["kind"]
    if kind == "exact":
        g = M.mochy_project(ctx, *state["graphs"][0])
        h, h3 = M.mochy_count_exact(ctx, g)
        wedges = g.num_hyperwedges
        g.close()
        return {"h": h, "h3": h3, "wedges": wedges}
    if kind == "cp":
        counts, sig26, cp26, sig431, cp431 = M.mochy_profile(ctx, state["graphs"])
        return {"counts": counts, "sig26": sig26, "cp26": cp26, "sig431": sig431, "cp431": cp431}
    if kind == "free":
        g = M.mochy_project(ctx, *state["graphs"][0], M.MOCHY_LG_FREE)
        out = M.mochy_count_sampled(ctx, g, case["samples"], state["seed"])
        wedges = g.num_hyperwedges
        g.close()
        return {"raw26": out[0], "est26": out[1], "raw431": out[2], "est431": out[3], "wedges": wedges}
    g = state["projected"]
    if kind in ("range", "noalloc"):
        a, b = _centres(case, g.num_edges)
        count = M.mochy_count_exact_range if kind == "range" else M.mochy_count_exact_range_noalloc
        h, h3 = count(ctx, g, a, b)
        return {"h": h, "h3": h3}
    if kind == "profiles":
        a, b = _centres(case, g.num_edges)
        return dict(zip(("hp26", "hp431"), M.mochy_hyperedge_profiles(ctx, g, a, b)))
    sample = M.mochy_count_sampled if kind == "aplus" else M.mochy_count_sampled_edges
    return dict(zip(("raw26", "est26", "raw431", "est431"), sample(ctx, g, case["samples"], state["seed"])))


def _centres(case, edges):
    """The range of hyperedges a case works on: `samples` of them from the middle, or all."""
    n = min(case["samples"], edges) if case["samples"] else edges
    return (edges - n) // 2, (edges - n) // 2 + n


def work(case):
    """Bytes: the CSRs read and the results written, once.  Operations: one
    per pair of hyperedges meeting at a node for whatever lists neighbours
    (expected degrees of the drawn hypergraph), the random numbers of a
    sample (about 80 integer operations) for sampling."""
    s, p = (x.numpy() for x in _pmf(case))
    w = np.arange(1, case["nodes"] + 1, dtype=np.float64) ** -case["alpha"]
    w /= w.sum()
    deg = case["edges"] * sum(q * -np.expm1(k * np.log1p(-w)) for k, q in zip(s, p))
    meets = float((deg * deg).sum() / 2)
    graphs = 1 + case["copies"]
    csr = (8 * (case["edges"] + 1) + 4 * float(deg.sum())) * graphs
    kind, n = case["kind"], case["samples"]
    out = 457 * 8 * (n if kind == "profiles" else graphs)
    share = min(1.0, n / case["edges"]) if kind in ("range", "profiles", "edges") else 1.0
    ops = meets * graphs * share
    if kind in ("aplus", "free"):
        ops = 80.0 * n + (meets if kind == "free" else 0.0)
    return {"bytes": csr + out, "flops": ops}


# ---------------------------------------------------------------------------
# Counts by definition


@functools.lru_cache(maxsize=1)
def _motif_table():
    """int64[2187, 2]: (h-motif id, 3h-motif id) of every ternary region
    pattern (R1 the most significant digit), zeros where no three distinct
    connected hyperedges have it.  A pattern's canonical form is its smallest
    relabelling; h-motifs go by (closed with R7, open, closed without R7),
    non-empty regions, form; 3h-motifs by (h-motif, form)."""
    regions = [{0}, {1}, {2}, {0, 1}, {1, 2}, {0, 2}, {0, 1, 2}]
    perms = [[regions.index({q[x] for x in r}) for r in regions] for q in itertools.permutations(range(3))]

    def canonical(t):
        return min(tuple(t[r] for r in q) for q in perms)

    def meets(t):
        return [any(t[r] for r in range(7) if {x, y} <= regions[r]) for x, y in ((0, 1), (1, 2), (0, 2))]

    def valid(t):
        distinct = all(any(t[r] for r in range(7) if (x in regions[r]) != (y in regions[r]))
                       for x, y in ((0, 1), (1, 2), (0, 2)))
        return distinct and sum(meets(t)) >= 2

    def binary(t):
        return tuple(int(v > 0) for v in t)

    def group(t):
        return 1 if not all(meets(t)) else (0 if t[6] else 2)

    h = {t: i + 1 for i, t in enumerate(sorted({canonical(t) for t in itertools.product((0, 1), repeat=7) if valid(t)},
                                               key=lambda t: (group(t), sum(t), t)))}
    every = [t for t in itertools.product((0, 1, 2), repeat=7) if valid(t)]
    h3 = {t: i + 1 for i, t in enumerate(sorted({canonical(t) for t in every}, key=lambda t: (h[canonical(binary(t))], t)))}
    table = np.zeros((3 ** 7, 2), dtype=np.int64)
    for t in every:
        table[functools.reduce(lambda a, v: 3 * a + v, t, 0)] = h[canonical(binary(t))], h3[canonical(t)]
    return table


def _count(ptr, nodes, num_nodes, centres=None):
    """(26 counts, 431 counts) by definition: every pair of neighbours of every
    centre e_i, classified by the seven region sizes; an open triple meets
    one such centre, a closed one three.  With a range of centres, what the
    range's centres own (an open triple its middle, a closed one its
    smallest hyperedge)."""
    dev = ptr.device
    E = ptr.numel() - 1
    size = ptr[1:] - ptr[:-1]
    inc = torch.zeros((E, num_nodes), dtype=torch.float32, device=dev)
    inc[torch.repeat_interleave(torch.arange(E, device=dev), size), nodes.long()] = 1.0
    w = (inc @ inc.T).round().to(torch.int32)
    tab = torch.from_numpy(_motif_table()).to(dev)
    codes = torch.zeros((2, 3 ** 7), dtype=torch.int64, device=dev)  # open, closed
    for i in range(*(centres or (0, E))):
        x = w[i].clone()
        x[i] = 0
        nb = torch.nonzero(x).flatten()
        b = inc[nb][:, nodes[ptr[i]:ptr[i + 1]].long()]
        for lo in range(0, nb.numel(), 1024):
            j, k = nb[lo:lo + 1024], nb
            t = (b[lo:lo + 1024] @ b.T).round().to(torch.int32)
            p, s, q = w[i, j][:, None], w[i, k][None, :], w[j][:, k]
            a, bj, ck = size[i].to(torch.int32), size[j].to(torch.int32)[:, None], size[k].to(torch.int32)[None, :]
            code = torch.zeros_like(t)
            for r in (a - p - s + t, bj - p - q + t, ck - s - q + t, p - t, q - t, s - t, t):
                code = code * 3 + torch.clamp(r, max=2)
            use = j[:, None] < k[None, :]
            if centres:
                use = use & ((q == 0) | (j[:, None] > i))
            index = (code + (q > 0) * 3 ** 7)[use].long()
            codes += torch.bincount(index, minlength=2 * 3 ** 7).reshape(2, -1)
    out = []
    for col, n in ((0, 26), (1, 431)):  # folded to motifs, then a third of the closed ones
        o = torch.zeros((2, n + 1), dtype=torch.int64, device=dev)
        o[0].index_add_(0, tab[:, col], codes[0])
        o[1].index_add_(0, tab[:, col], codes[1])
        out.append((o[0] + (o[1] if centres else o[1] // 3))[1:].cpu().numpy())
    return out


def exact(case, seed):
    """Counts, significance and profile by definition, for hypergraphs small
    enough.  Sampled results have no such value within seconds: a sample's
    hits need its whole neighbourhood, over up to a million samples."""
    kind = case["kind"]
    if kind not in COUNTED or case["edges"] * (1 + case["copies"]) > 30_000 or case["edges"] > 8_000:
        return None
    graphs = _graphs(case, seed)
    if kind == "cp":
        counts = np.array([np.concatenate(_count(*g)) for g in graphs], dtype=np.int64)
        m, mr = counts[0].astype(np.float64), counts[1:].sum(axis=0).astype(np.float64) / case["copies"]
        delta = (m - mr) / (m + mr + 1.0)
        d26, d431 = delta[:26], delta[26:]
        norm = [np.sqrt((d * d).sum()) for d in (d26, d431)]
        cp = [d / n if n else d * 0 for d, n in zip((d26, d431), norm)]
        return {"counts": counts, "sig26": d26, "cp26": cp[0], "sig431": d431, "cp431": cp[1]}
    ptr, nodes, v = graphs[0]
    if kind == "exact":
        h, h3 = _count(ptr, nodes, v)
        return {"h": h, "h3": h3, "wedges": None}
    h, h3 = _count(ptr, nodes, v, _centres(case, ptr.numel() - 1))
    return {"h": h, "h3": h3}
