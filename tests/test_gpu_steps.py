"""Branches of the kernels' dispatch at the sizes where they change: results
against the oracle, intermediate counts against the multi-kernel path."""
import numpy as np
import pytest

import oracle
import paper_1807_08804_amd as P
from tests.micro import MicroGraph, MicroQuery, random_graph, random_query

pytestmark = pytest.mark.gpu


def micro(seed, V, E, n_types=3, n_rels=3, nq=8, n_max=7, **kw):
    rng = np.random.default_rng(seed)
    mg = random_graph(rng, V, E, n_types=n_types, n_rels=n_rels)
    qs = [random_query(rng, int(rng.integers(2, n_max)), n_types, n_rels, V, p_pin=0.25, extra=3)
          for _ in range(nq)]
    return mg, qs, oracle.Graph(V, mg.src, mg.dst, mg.rel, mg.vtype)


@pytest.mark.parametrize("rounds,rev", [(0, 1), (1, 1), (1, 0), (-1, 0)])
@pytest.mark.parametrize("seed,V,E", [(1, 12, 40), (2, 60, 200), (3, 400, 1600), (4, 3000, 9000)])
def test_filter_counts_equal_on_both_paths(seed, V, E, rounds, rev):
    """Tests left out because they are known to hold change no candidate
    set: counts of candidates and candidate edges equal the multi-kernel
    path's, which runs every test."""
    mg, qs, og = micro(900 + seed, V, E)
    rp, col, rel, typ = mg.csr()
    gs = [P.Graph(rp, col, rel, typ, path=p, refine_rounds=rounds, refine_reversed=rev)
          for p in (P.SGM_PATH_NARROW, P.SGM_PATH_WIDE)]
    for i, q in enumerate(qs):
        print("case: query", i, flush=True)
        (rn, sn), (rw, sw) = [g.match_query(q, with_stats=True) for g in gs]
        assert np.array_equal(rn, rw) and np.array_equal(rn, og.match_query(q))
        assert sn["cand"] == sw["cand"]
        if min(sn["cand"]) > 0:
            assert sn["ec"] == sw["ec"]
            if min(sn["ec"], default=1) > 0 and len(rn):
                assert sn["level_rows"] == sw["level_rows"]


@pytest.mark.parametrize("n_types,n_rels,tbase,rbase", [
    (3, 3, 0, 0),                 # types in the adjacency entries
    (3, 3, 32764, 65531),         # the largest types and relations they hold
    (3, 3, 32766, 0), (3, 3, 0, 65533),  # one past each: entries without types
    (3, 3, 70000, 1 << 20),
])
def test_types_in_adjacency_entries(n_types, n_rels, tbase, rbase):
    """Entries that carry their vertex's type and graphs whose types or
    relations do not fit them give the same matches."""
    mg, qs, _ = micro(77, 200, 900, n_types, n_rels, nq=12)
    rp, col, rel, typ = mg.csr()
    typ, rel = np.asarray(typ) + tbase, np.asarray(rel) + rbase
    og = oracle.Graph(200, mg.src, mg.dst, np.asarray(mg.rel) + rbase, np.asarray(mg.vtype) + tbase)
    for path in (P.SGM_PATH_AUTO, P.SGM_PATH_WIDE):
        g = P.Graph(rp, col, rel, typ, path=path)
        for i, q in enumerate(qs):
            print("case: query", i, "path", path, flush=True)
            q2 = type(q)(**{**q.__dict__})
            q2.vlabel = np.where(q.vlabel >= 0, q.vlabel + tbase, q.vlabel).astype(np.int32)
            q2.elabel = np.where(q.elabel >= 0, q.elabel + rbase, q.elabel).astype(np.int32)
            assert np.array_equal(g.match_query(q2), og.match_query(q2))
        g.close()


@pytest.mark.parametrize("V,deg,n_types,n_rels", [
    (70, 1, 2, 1), (70, 6, 2, 2), (600, 3, 2, 2), (600, 40, 40, 8), (2000, 97, 60, 6),
    (3000, 130, 80, 8), (1200, 600, 300, 16),
])
def test_flat_filter_rows(V, deg, n_types, n_rels):
    """Filter steps whose candidates' rows are dealt to the lanes end to end:
    rows shorter and longer than a wave's window, around the limits where a
    row goes to the next tier, one candidate to several per lane; with the
    steps shared over helpers and not."""
    rng = np.random.default_rng(V + deg)
    src = np.repeat(np.arange(V), rng.integers(max(0, deg - 2), deg + 3, V))
    # a few rows up to five times as long
    src = np.concatenate([src, np.repeat(rng.integers(0, V, 6), 4 * deg)])
    mg = MicroGraph(V, src, rng.integers(0, V, len(src)), rng.integers(0, n_rels, len(src)),
                    rng.integers(0, n_types, V))
    og = oracle.Graph(V, mg.src, mg.dst, mg.rel, mg.vtype)
    rp, col, rel, typ = mg.csr()
    g = P.Graph(rp, col, rel, typ)
    qs = [random_query(rng, int(rng.integers(2, 6)), n_types, n_rels, V, p_any_label=p,
                       p_any_rel=p, p_pin=0.2, extra=2) for p in (0.0, 0.1, 0.5) for _ in range(4)]
    for tune in (dict(), dict(help_items=64, helpers=96), dict(help_items=0)):
        g.set_tuning(**tune)
        for i, q in enumerate(qs):
            print("case: query", i, tune, flush=True)
            if g.match_query(q, count_only=True) > 200000:
                continue
            assert np.array_equal(g.match_query(q), og.match_query(q))


@pytest.mark.parametrize("n_types,p_any", [(1, 1.0), (2, 0.4), (6, 0.2)])
@pytest.mark.parametrize("V,E", [(8, 60), (40, 400), (150, 1500), (400, 2600)])
def test_counts_without_rows(V, E, n_types, p_any):
    """A count-only query's last join level counts without writing rows: the
    counts are those of the tables, for levels with and without check edges,
    one block of parent rows and several (shared or not), repeated values in
    the fan-out, and leading single-candidate vertices."""
    rng = np.random.default_rng(31 * V + n_types)
    mg = random_graph(rng, V, E, n_types=n_types, n_rels=2)
    rp, col, rel, typ = mg.csr()
    og = oracle.Graph(V, mg.src, mg.dst, mg.rel, mg.vtype)
    qs = [random_query(rng, int(rng.integers(1, 5)), n_types, 2, V, p_any_label=p_any,
                       p_any_rel=p_any, p_pin=p, extra=x) for p in (0.0, 0.4) for x in (0, 3)
          for _ in range(4)]
    g = P.Graph(rp, col, rel, typ)
    wants = [len(og.match_query(q)) for q in qs]
    for tune in (dict(), dict(help_items=0)):
        g.set_tuning(**tune)
        for i, (q, want) in enumerate(zip(qs, wants)):
            print("case: query", i, "rows", want, flush=True)
            assert g.match_query(q, count_only=True) == want
        assert g.match_batch(qs, count_only=True) == wants


def hub_graph(hubs, row, V=20000):
    """`hubs` vertices of type 1, each with edges to `row` of the V vertices
    of types 0 and 2 (relation 0, every 40th 1) and back from a twentieth;
    the vertices among themselves carry sparse relation-1 edges."""
    rng = np.random.default_rng(hubs + row)
    vt = np.concatenate([np.where(rng.random(V) < 0.02, 2, 0), np.full(hubs, 1)])
    e = []
    for h in range(V, V + hubs):
        to = rng.permutation(V)[:row]
        e.append((np.full(row, h), to, np.arange(row) % 40 == 0))
        e.append((to[::20], np.full(len(to[::20]), h), np.ones(len(to[::20]))))
    a = rng.integers(0, V, 3000)
    e.append((a, rng.integers(0, V, 3000), np.ones(3000)))
    src, dst, rel = (np.concatenate(x).astype(np.int32) for x in zip(*e))
    return MicroGraph(V + hubs, src, dst, rel, vt)


@pytest.mark.parametrize("hubs,row", [(1, 16384), (4, 16383), (5, 16384), (8, 300), (9, 300),
                                      (8, 16385), (9, 2048), (40, 1200)])
def test_hub_candidates_against_many(hubs, row):
    """Few candidates with long rows beside neighbours with thousands: tests
    checked from the few's side, rows at the limits of the typed hub index
    and of the wave and workgroup tiers, edge tables of up to eight keys built
    together and of nine alone, values looked up one by one or scanned."""
    mg = hub_graph(hubs, row)
    og = oracle.Graph(mg.V, mg.src, mg.dst, mg.rel, mg.vtype)
    rp, col, rel, typ = mg.csr()
    hub = mg.V - 1
    qs = [MicroQuery(3, [1, 0, 2], [-1, -1, -1], [0, 1], [1, 2], [0, 1]),
          MicroQuery(3, [1, 0, 2], [-1, -1, -1], [1, 1, 0], [0, 2, 2], [1, 1, -1]),
          MicroQuery(3, [1, 0, 1], [hub, -1, -1], [0, 1, 2], [1, 2, 1], [0, 1, 0]),
          MicroQuery(4, [0, 1, -1, 2], [-1, hub, -1, -1], [1, 0, 2, 1], [0, 2, 3, 3], [1, 1, 1, -1])]
    gs = [P.Graph(rp, col, rel, typ, path=p) for p in (P.SGM_PATH_NARROW, P.SGM_PATH_WIDE)]
    for tune in (dict(), dict(help_items=64), dict(help_items=0)):
        gs[0].set_tuning(**tune)
        for i, q in enumerate(qs):
            print("case: query", i, tune, flush=True)
            (rn, sn), (rw, sw) = [g.match_query(q, with_stats=True) for g in gs]
            assert np.array_equal(rn, rw) and np.array_equal(rn, og.match_query(q))
            assert sn["cand"] == sw["cand"]
            if min(sn["cand"]) > 0:
                assert sn["ec"] == sw["ec"]


@pytest.mark.parametrize("row", [256, 257, 1024, 1025, 8192, 8193, 9216, 9217, 16384])
def test_long_rows_multi_kernel_path(row):
    """Rows a workgroup takes whole in the multi-kernel path: at the limit of
    the tier and at the ends of its rounds; both adjacency directions and the
    outgoing graph only."""
    mg = hub_graph(3, row)
    og = oracle.Graph(mg.V, mg.src, mg.dst, mg.rel, mg.vtype)
    rp, col, rel, typ = mg.csr()
    qs = [MicroQuery(3, [1, 0, 2], [-1, -1, -1], [0, 1], [1, 2], [0, 1]),
          MicroQuery(3, [1, 0, 1], [mg.V - 1, -1, -1], [0, 1, 2], [1, 2, 1], [0, 1, -1]),
          MicroQuery(2, [2, 1], [-1, -1], [1, 0], [0, 1], [-1, 1])]
    for opt in (dict(path=P.SGM_PATH_WIDE), dict(out_only=1)):
        g = P.Graph(rp, col, rel, typ, **opt)
        for i, q in enumerate(qs):
            print("case: query", i, opt, flush=True)
            assert np.array_equal(g.match_query(q), og.match_query(q))
        g.close()


@pytest.mark.parametrize("n", [1, 8191, 8193, 32767, 32768, 32769, 40000])
def test_scans_of_one_and_several_workgroups(n):
    """A join level's pair offsets over n parent rows: one round, several,
    and the sizes from which the scan runs in several workgroups."""
    i = np.arange(n)
    dst = n + np.concatenate([i, (i[::7] * 3 + 1) % n])
    mg = MicroGraph(2 * n, np.concatenate([i, i[::7]]), dst, np.zeros(len(dst)), i.repeat(2) * 0)
    rp, col, rel, typ = mg.csr()
    g = P.Graph(rp, col, rel, typ, path=P.SGM_PATH_WIDE)
    q = MicroQuery(2, [-1, -1], [-1, -1], [0], [1], [0])
    want = np.unique(np.stack([mg.src, mg.dst], 1), axis=0)
    assert np.array_equal(g.match_query(q), want)


@pytest.mark.parametrize("members,links", [(1, 1), (5, 64), (5, 65), (24, 4095), (24, 4096), (260, 300)])
def test_expansion_by_waves_and_threads(members, links):
    """Expansions of weighted matches: one to 260 members per mapping list
    (partial assignments below and above a wave's 64, more matches than the
    first table holds) and weighted matches on both sides of the number from
    which a thread takes each."""
    # `links` pairs of single vertices and one pair of groups of `members`
    # alike vertices, complete between the groups; types keep pairs apart
    n = 2 * links
    a, b = n + np.arange(members), n + members + np.arange(members)
    src = np.concatenate([np.arange(links), np.repeat(a, members)])
    dst = np.concatenate([links + np.arange(links), np.tile(b, members)])
    vt = np.concatenate([np.zeros(links), np.ones(links), np.full(members, 2), np.full(members, 3)])
    mg = MicroGraph(n + 2 * members, src, dst, np.zeros(len(src)), vt)
    rp, col, rel, typ = mg.csr()
    g = P.Graph(rp, col, rel, typ)
    cg = P.CompressedGraph(g, P.Compressed(rp, col, rel, typ, max_levels=8))
    og = oracle.Graph(mg.V, mg.src, mg.dst, mg.rel, mg.vtype)
    qs = [MicroQuery(2, [0, 1], [-1, -1], [0], [1], [0]), MicroQuery(2, [2, 3], [-1, -1], [0], [1], [0]),
          MicroQuery(2, [-1, -1], [-1, -1], [0], [1], [-1])]
    if members <= 24:
        qs.append(MicroQuery(3, [2, 3, 2], [-1, -1, -1], [0, 2], [1, 1], [0, 0]))
    for i, q in enumerate(qs):
        print("case: query", i, flush=True)
        want = og.match_query(q)
        assert np.array_equal(cg.match_query(q), want)
        assert cg.match_query(q, count_only=True) == len(want)
    cg.close()
    g.close()


@pytest.mark.parametrize("k", [1, 15, 16, 17, 18, 300, 4000])
@pytest.mark.parametrize("back", [0, 1])
def test_marks_kept_word_by_word_and_one_by_one(k, back):
    """A parent's candidates cut to the k that a step marked, below and above
    a quarter of the bitmap's 64 words, where the marks are taken from the
    scratch bitmap instead of one by one; all of them kept, and some."""
    V = 4096
    rng = np.random.default_rng(k)
    par = rng.permutation(V - 40)[:k]  # parents with a child of type 1
    src = np.concatenate([np.arange(V - 40), par])
    dst = np.concatenate([np.full(V - 40, V - 40), V - 39 + rng.integers(0, 39, k)])
    if back:
        src, dst = dst, src
    vt = np.concatenate([np.zeros(V - 40), [2], np.full(39, 1)])
    mg = MicroGraph(V, src, dst, np.zeros(len(src)), vt)
    og = oracle.Graph(V, mg.src, mg.dst, mg.rel, mg.vtype)
    rp, col, rel, typ = mg.csr()
    qs = [MicroQuery(3, [1, 0, 2], [-1, -1, V - 40], [1, 1], [0, 2], [0, 0]),
          MicroQuery(3, [2, 0, 1], [V - 40, -1, -1], [1, 1], [0, 2], [0, 0])]
    if back:
        qs = [MicroQuery(3, q.vlabel, q.vpin, q.edst, q.esrc, q.elabel) for q in qs]
    gs = [P.Graph(rp, col, rel, typ, path=p) for p in (P.SGM_PATH_NARROW, P.SGM_PATH_WIDE)]
    for tune in (dict(help_items=64), dict(help_items=0)):
        gs[0].set_tuning(**tune)
        for i, q in enumerate(qs):
            print("case: query", i, tune, flush=True)
            (rn, sn), (rw, sw) = [g.match_query(q, with_stats=True) for g in gs]
            assert len(rn) == k and np.array_equal(rn, rw) and np.array_equal(rn, og.match_query(q))
            assert sn["cand"] == sw["cand"] and sn["ec"] == sw["ec"]


@pytest.mark.parametrize("helpers,help_items", [(64, 64), (512, 1024), (0, 0)])
@pytest.mark.parametrize("V,every", [(1024, 8), (1024, 7), (4096, 64), (4097, 9), (9000, 300),
                                     (70000, 8), (70000, 33), (300001, 999)])
def test_roots_that_few_vertices_reach(V, every, helpers, help_items):
    """Roots whose degree bounds admit few of their range (one vertex in eight
    and fewer; just more than that; none), looked up by degrees alone: ranges
    of one round and many, one type and any, served and not."""
    hub = np.arange(0, V, every)
    k = 1 + np.arange(len(hub)) % 3  # spokes beyond the four they need
    src = np.concatenate([np.repeat(hub, 3 + k), np.arange(1, V)])
    dst = np.concatenate([np.arange(int((3 + k).sum())) * 7 % V, np.zeros(V - 1)])
    rel = np.concatenate([np.arange(int((3 + k).sum())) % 5, np.full(V - 1, 5)])
    vt = (np.arange(V) % 50 == 49).astype(np.int32)
    mg = MicroGraph(V, src, dst, rel, vt)
    og = oracle.Graph(V, mg.src, mg.dst, mg.rel, mg.vtype)
    rp, col, rl, typ = mg.csr()
    g = P.Graph(rp, col, rl, typ)
    g.set_tuning(help_items=help_items, helpers=helpers)
    star = lambda l, w: MicroQuery(w + 1, [l] + [-1] * w, [-1] * (w + 1), [0] * w,
                                   range(1, w + 1), [0, 1, 2, 3, 4, 0, 1, 2][:w])
    qs = [star(0, 4), star(-1, 4), star(1, 4), star(0, 5), star(-1, 8)]
    srv = P.Server(g)
    for i, q in enumerate(qs):
        print("case: query", i, flush=True)
        want = og.match_query(q)
        assert np.array_equal(g.match_query(q), want)
        assert np.array_equal(srv.wait(srv.submit(q), q.n)[1], want)
    srv.close()
    g.close()


@pytest.mark.parametrize("row", [95, 96, 97, 255, 256, 257, 511, 512, 513])
@pytest.mark.parametrize("cands", [6, 40, 700])
def test_rows_at_the_flat_window(cands, row):
    """Candidates whose rows are just as long as a wave's flat scan takes, one
    less and one more, alone in their wave and with others; shared or not."""
    T = 3000
    rng = np.random.default_rng(row + cands)
    dst = cands + np.concatenate([rng.permutation(T)[:row] for _ in range(cands)])
    src = np.repeat(np.arange(cands), row)
    mg = MicroGraph(cands + T, src, dst, rng.integers(0, 40, len(src)),
                    np.concatenate([np.zeros(cands), 1 + rng.integers(0, 30, T)]))
    og = oracle.Graph(mg.V, mg.src, mg.dst, mg.rel, mg.vtype)
    rp, col, rel, typ = mg.csr()
    qs = [MicroQuery(3, [0, 1, 2], [-1, -1, -1], [0, 0], [1, 2], [3, -1]),
          MicroQuery(3, [1, 0, 0], [-1, -1, -1], [1, 2], [0, 0], [5, 7])]
    g = P.Graph(rp, col, rel, typ)
    for tune in (dict(help_items=64), dict(help_items=0)):
        g.set_tuning(**tune)
        for i, q in enumerate(qs):
            print("case: query", i, tune, flush=True)
            assert np.array_equal(g.match_query(q), og.match_query(q))
    g.close()


def test_sparse_roots_of_a_compressed_graph():
    """Roots that few vertices reach, by a compressed graph's degree bounds
    instead of its row lengths."""
    V = 6000
    rng = np.random.default_rng(17)
    hub = rng.permutation(V)[:60]
    src = np.concatenate([rng.integers(0, V, V), np.repeat(hub, 7)])
    dst = np.concatenate([rng.integers(0, V, V), rng.integers(0, V, 60 * 7)])
    mg = MicroGraph(V, src, dst, rng.integers(0, 4, len(src)), rng.integers(0, 2, V))
    og = oracle.Graph(V, mg.src, mg.dst, mg.rel, mg.vtype)
    rp, col, rel, typ = mg.csr()
    g = P.Graph(rp, col, rel, typ)
    cg = P.CompressedGraph(g, P.Compressed(rp, col, rel, typ))
    rows = 0
    for w in (4, 5):
        for label in (-1, 0, 1):
            q = MicroQuery(w + 1, [label] + [-1] * w, [-1] * (w + 1), [0] * w, range(1, w + 1),
                           [0, 1, 2, 3, -1][:w])
            print("case: star of", w, "label", label, flush=True)
            want = og.match_query(q)
            rows += len(want)
            assert np.array_equal(g.match_query(q), want)
            assert np.array_equal(cg.match_query(q), want)
    assert rows > 0
    cg.close()
    g.close()
