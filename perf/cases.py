"""The workloads this library's speed is measured on.

Each case is one way a program uses the library, through its public entry
points: ``match_query`` one query at a time, ``match_batch`` (tables, counts
or projections), a :class:`Server` fed with a burst, and matching through a
compressed graph. The graph is resident before the call, as it is in a
program that answers queries. A case names its set of queries; a seed numbers
their vertices, orders their edges and (where only counts come back) the queries
themselves anew, so every seed has other inputs and other tables of the same
size.

Graphs are those of :mod:`kggen`: the tiny, medium and large power-law
knowledge graphs, the 1M-vertex graphs of the size / degree sweeps, the
scaling graphs, and graphs with similar vertices. Graphs of the sizes in
between are drawn by the same recipe. Queries on graphs of up to a few hundred
thousand vertices are drawn on the graph; those on larger graphs are sampled
from the stored workloads (drawing them takes minutes).
"""
import collections
import math

import numpy as np
import torch

import kggen
import paper_1807_08804_amd as P

MOST_TABLES = 60  # result tables one pass returns one by one


# --------------------------------------------------------------------------
# cases
# --------------------------------------------------------------------------

def listed():
    # sets of the stored pools are ones whose numbers of matches are near the
    # whole pool's: a few matches for most queries, a large table for one or two
    return [
        # one small question to a small knowledge graph: pure call latency
        {"name": "tiny-one", "call": "one", "graph": "power", "V": 2000, "E": 8000, "pool": "batch", "count": 1, "set": 0},
        # an interactive program: questions of 6 to 10 vertices, one after the other
        {"name": "medium-one", "call": "one", "graph": "medium", "pool": "walk", "count": 8, "set": 0},
        # answers are a few columns of each match: a batch of projected queries
        {"name": "medium-proj-batch", "call": "proj", "graph": "medium", "pool": "walk", "count": 60, "set": 0},
        # a graph held without its incoming edges (half the memory): whole-GPU kernels per query
        {"name": "medium-out-only", "call": "one", "graph": "medium", "pool": "walk", "count": 4, "set": 0, "option": "out_only"},
        # the large graph, mixed queries of 3 to 16 vertices one at a time
        {"name": "large-one", "call": "one", "graph": "large", "pool": "batch", "count": 12, "set": 6},
        # the same queries as one batch, every table to the host
        {"name": "large-batch", "call": "batch", "graph": "large", "pool": "batch", "count": 60, "set": 5},
        # the full mixed batch, counts only (analytics over many questions)
        {"name": "large-batch-counts", "call": "counts", "graph": "large", "pool": "batch", "count": 1024, "set": 0},
        # a server that gets a burst of user questions at once
        {"name": "large-served", "call": "served", "graph": "large", "pool": "serve", "count": 60, "set": 0},
        # unpinned cyclic queries with large intermediate tables, exact counts one at a time
        {"name": "large-cyclic", "call": "onecount", "graph": "large", "pool": "cyclic", "count": 6, "set": 3},
        # a dense graph (average degree 16): batch of 10-vertex queries with one concept node
        {"name": "dense-batch", "call": "batch", "graph": "sweep", "degree": 16, "pool": "size/10", "count": 59, "set": 0},
        # edges kept in host memory, read in place by the kernels
        {"name": "host-graph-batch", "call": "batch", "graph": "scale", "V": 1000000, "pool": "scale/1000000",
         "count": 60, "set": 0, "option": "host_graph"},
        # matching through a multi-level compression, expanded on the device
        {"name": "compressed-one", "call": "compressed", "graph": "twin", "V": 20000, "E": 80000, "pool": "twin", "count": 6, "set": 0},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["power", "power", "power", "twin", "medium", "large", "sweep", "scale"])
    if kind == "twin":
        V = _log(rng, 5000, 60000)
        return {"call": "compressed", "graph": "twin", "V": V, "E": int(V * rng.uniform(3.0, 5.0)),
                "pool": "twin", "count": rng.randint(1, 16), "set": rng.randrange(10000)}
    c = {"graph": kind, "set": rng.randrange(10000)}
    if kind == "power":
        c["V"] = _log(rng, 2000, 120000)
        c["E"] = int(c["V"] * rng.uniform(3.0, 8.0))
        c["pool"] = rng.choice(["walk", "batch", "any"])
    elif kind == "medium":
        c["pool"] = "walk"
    elif kind == "large":
        c["pool"] = rng.choice(["batch", "serve", "batch", "cyclic"])
    elif kind == "sweep":
        c["degree"] = rng.choice(kggen.SWEEP_DEGREES)
        c["pool"] = "degree/%d" % c["degree"]
        if c["degree"] == kggen.SWEEP_SIZE_DEGREE:
            c["pool"] = "size/%d" % rng.choice(kggen.SWEEP_SIZES)
    else:
        c["V"] = rng.choice(kggen.SCALE_VERTICES[:3])
        c["pool"] = "scale/%d" % c["V"]
    if c["pool"] == "cyclic":
        c["call"], c["count"] = "onecount", rng.randint(1, 6)
        return c
    drawn_live = c["pool"] in ("batch", "any") and kind == "power"
    c["call"] = rng.choice(["one", "batch", "counts", "proj", "served"])
    if c["call"] == "one":
        c["count"] = rng.randint(1, 16)
        if kind in ("power", "medium") and rng.random() < 0.3:
            c["option"] = "out_only"
            c["count"] = rng.randint(1, 4)
    elif c["call"] == "counts" and c["pool"] == "walk":
        c["count"] = _log(rng, 16, 200)
    elif c["call"] == "counts" and kind == "large":
        c["count"] = _log(rng, 16, 1000) if c["pool"] == "batch" else _log(rng, 16, 500)
    else:
        c["count"] = rng.randint(2, 32 if drawn_live else MOST_TABLES)
    if "option" not in c and c["call"] != "served" and kind in ("power", "scale") and rng.random() < 0.3:
        c["option"] = "host_graph"
    return c


# --------------------------------------------------------------------------
# graphs (resident on the device, kept between the states that share one)
# --------------------------------------------------------------------------

def _power_graph(V, E, seed, dmax=0):
    """kggen.make_graph(V, E, seed, dmax=dmax), the same arrays, with its
    sorts on the GPU for the large graphs (they take most of its time)."""
    if E < 4_000_000:
        return kggen.make_graph(V, E, seed, dmax=dmax)
    rng = np.random.Generator(np.random.PCG64(seed))
    deg = kggen._powerlaw_outdegrees(rng, V, E, kggen.DEG_EXPONENT, dmax)
    dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    tdeg = torch.from_numpy(deg).to(dev)
    src = torch.repeat_interleave(torch.arange(V, device=dev), tdeg)
    dst = torch.from_numpy(rng.integers(0, V - 1, size=E, dtype=np.int64)).to(dev)
    dst += (dst >= src).long()
    row = torch.zeros(V + 1, dtype=torch.int64, device=dev)
    torch.cumsum(tdeg, 0, out=row[1:])
    idx = torch.arange(E, device=dev)
    while True:
        # repeated destinations of one source are drawn again
        sk, order = torch.sort(src[idx] * V + dst[idx], stable=True)
        dup = torch.zeros(len(idx), dtype=torch.bool, device=dev)
        dup[order[1:]] = sk[1:] == sk[:-1]
        bad = idx[dup]
        if len(bad) == 0:
            break
        new = torch.from_numpy(rng.integers(0, V - 1, size=len(bad), dtype=np.int64)).to(dev)
        new += (new >= src[bad]).long()
        dst[bad] = new
        rows = torch.unique(src[bad])
        lens = row[rows + 1] - row[rows]
        first = row[rows] - torch.cumsum(lens, 0) + lens
        idx = torch.repeat_interleave(first, lens) + torch.arange(int(lens.sum()), device=dev)
    dst = (torch.sort(src * V + dst)[0] % V).to(torch.int32).cpu().numpy()
    zcdf = np.cumsum(np.arange(1, kggen.N_RELS + 1, dtype=np.float64) ** -kggen.ZIPF_S)
    zcdf /= zcdf[-1]
    rel = torch.searchsorted(torch.from_numpy(zcdf).to(dev), torch.from_numpy(rng.random(E)).to(dev), right=True)
    rel = rel.clamp_(max=kggen.N_RELS - 1).to(torch.int32).cpu().numpy()
    vtype = rng.integers(0, kggen.N_TYPES, size=V, dtype=np.int32)
    return kggen.KG(V=V, E=E, row_ptr=row.to(torch.int32).cpu().numpy(), col=dst, rel=rel, vtype=vtype)


class _Resident:
    """A graph in the library's hands, with what its program keeps beside
    it: the host arrays, a server, or a compression."""

    def __init__(self, case):
        kind, opt = case["graph"], case.get("option")
        if kind in kggen.GRAPHS:
            V, E, off = kggen.GRAPHS[kind]
            self.kg = _power_graph(V, E, kggen.BASE_SEED + off)
        elif kind == "power":
            self.kg = kggen.make_graph(case["V"], case["E"], kggen.BASE_SEED + case["V"] + case["E"])
        elif kind == "sweep":
            V, d = kggen.SWEEP_V, case["degree"]
            self.kg = _power_graph(V, d * V, kggen.BASE_SEED + 10 + d, V // kggen.SWEEP_DMAX_DIV)
        elif kind == "scale":
            V = case["V"]
            self.kg = _power_graph(V, kggen.SCALE_DEGREE * V, kggen.BASE_SEED + 40 + V % 997,
                                   V // kggen.SWEEP_DMAX_DIV)
        else:
            self.kg = kggen.twin_graph(case["V"], case["E"], kggen.BASE_SEED + case["V"])
        self.graph = P.Graph.from_kg(self.kg, **({opt: 1} if opt else {}))
        self.server = self.through = None
        self.sets = {}
        if case["call"] == "served":
            self.server = P.Server(self.graph)
        if case["call"] == "compressed":
            comp = P.Compressed.from_kg(self.kg)
            self.through = P.CompressedGraph(self.graph, comp)
            comp.close()

    def close(self):
        for x in (self.server, self.through, self.graph):
            if x is not None:
                x.close()


_resident = collections.OrderedDict()
_KEPT = 2  # graphs resident at once


def _graph(case):
    key = tuple((k, case.get(k)) for k in ("graph", "V", "E", "degree", "option"))
    key += (case["call"] if case["call"] in ("served", "compressed") else "",)
    if key not in _resident:
        while len(_resident) >= _KEPT:
            _resident.popitem(last=False)[1].close()
        _resident[key] = _Resident(case)
    _resident.move_to_end(key)
    return _resident[key]


# --------------------------------------------------------------------------
# queries
# --------------------------------------------------------------------------

_stored = {}


def _pool(name):
    """A stored workload of the large graphs (None for the others)."""
    if not _stored:
        _stored.update(kggen.load_sweep())
        _stored["batch"] = kggen.load_large_batch()[0]
        _stored["serve"] = kggen.load_large_serve()[0]
        _stored["cyclic"] = kggen.load_large_cyclic()
    return _stored[name]


def _query_set(case, kg):
    """The case's queries, each with the columns a projection keeps."""
    pool, count = case["pool"], case["count"]
    qseed = kggen.BASE_SEED + 5000 + case["set"]
    rng = np.random.default_rng(qseed)
    if case["graph"] in ("large", "sweep", "scale"):
        stored = _pool(pool)
        qs = [stored[int(i)] for i in rng.choice(len(stored), size=count, replace=False)]
    elif pool == "walk":
        qs = kggen.medium_queries(kg, count, seed=qseed)[0]
    elif pool == "batch":
        qs = kggen.batch_queries(kg, count, seed=qseed, hmax=1e5)[0]
    elif pool == "any":
        qs = kggen.sweep_queries(kg, int(rng.integers(3, 9)), count, seed=qseed, hmax=1e5)[0]
    else:
        qs = kggen.twin_queries(kg, count, seed=qseed, hmax=5e4)
    # a question asks for about a third of its query vertices
    return [(q, rng.choice(q.n, size=max(1, q.n // 3), replace=False)) for q in qs]


def _renumber(q, kept, rng):
    """The same query with its vertices and edges numbered another way."""
    new = rng.permutation(q.n).astype(np.int32)  # new index of vertex u
    old = np.argsort(new)
    e = rng.permutation(q.m)
    r = kggen.Query(n=q.n, vlabel=q.vlabel[old], vpin=q.vpin[old], esrc=new[q.esrc][e], edst=new[q.edst][e],
                    elabel=q.elabel[e], shape=q.shape)
    return r, sorted(new[kept].tolist())


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------

def prepare(case, seed):
    res = _graph(case)
    key = (case["pool"], case["count"], case["set"])
    if key not in res.sets:
        res.sets[key] = _query_set(case, res.kg)
    rng = np.random.default_rng(int(seed))
    qs = [_renumber(q, kept, rng) for q, kept in res.sets[key]]
    if case["call"] in ("counts", "onecount"):
        qs = [qs[i] for i in rng.permutation(len(qs))]
    state = {"call": case["call"], "resident": res, "queries": [q for q, _ in qs]}
    if case["call"] == "proj":
        state["projects"] = [kept for _, kept in qs]
    if case["call"] == "served":
        state["arrivals"] = np.zeros(len(qs))
    return state


def run(state):
    res, qs, call = state["resident"], state["queries"], state["call"]
    if call == "one":
        return [res.graph.match_query(q) for q in qs]
    if call == "onecount":
        return np.array([res.graph.match_query(q, count_only=True) for q in qs], np.int64)
    if call == "batch":
        return res.graph.match_batch(qs)
    if call == "counts":
        return np.array(res.graph.match_batch(qs, count_only=True), np.int64)
    if call == "proj":
        return res.graph.match_batch(qs, projects=state["projects"])
    if call == "served":
        return res.server.replay(qs, state["arrivals"])[1]
    return [res.through.match_query(q) for q in qs]


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------

# Means over each workload, per query: matches, candidates left over all
# query vertices, query vertices, and the share of queries with an unpinned
# root (whose candidates come from one read of all vertices' types).
_MEANS = {
    "walk": (800, 45, 8, 0.3), "batch": (4000, 115, 9.5, 0.3), "any": (300, 500, 6, 0.0),
    "serve": (10000, 150, 7.5, 0.3), "cyclic": (0, 200000, 11, 1.0), "twin": (900, 60, 5, 0.3),
    "size": (30000, 1700, 10, 0.0), "degree": (22000, 1700, 10, 0.0), "scale": (300, 260, 6, 0.0),
}


def work(case):
    """Each query's surviving candidates with their rows in both directions,
    its matches written once, and one read of the vertex types per call that
    has an unpinned root."""
    V, E = case.get("V"), case.get("E")
    if case["graph"] in kggen.GRAPHS:
        V, E, _ = kggen.GRAPHS[case["graph"]]
    elif case["graph"] == "sweep":
        V, E = kggen.SWEEP_V, kggen.SWEEP_V * case["degree"]
    elif case["graph"] == "scale":
        E = V * kggen.SCALE_DEGREE
    rows, cand, n, swept = _MEANS[case["pool"].split("/")[0]]
    tables = case["call"] not in ("counts", "onecount")
    per = cand * (8.0 + 16.0 * E / V) + (rows * n * 4.0 if tables else 8.0) + 32.0 * n
    calls = case["count"] if case["call"] in ("one", "onecount", "compressed") else 1
    sweeps = calls * swept if calls > 1 else (1.0 if case["count"] * swept >= 1 else swept)
    return {"bytes": case["count"] * per + sweeps * 8.0 * V, "flops": 0}
