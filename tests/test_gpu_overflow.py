"""Filter steps that outgrow their slot's candidate lists: the query leaves
the slot and is answered in a larger one, and nothing else is touched."""
import numpy as np
import pytest

import oracle
import paper_1807_08804_amd as P
from tests.micro import MicroGraph, MicroQuery

pytestmark = pytest.mark.gpu

LCAP = 65536  # entries of a regular slot's candidate list


def wide_root_graph(V, keep, longs=40):
    """Type 0: `keep` vertices with one relation-0 edge to a type-1 vertex and
    `longs` with rows of 97 to 9,000 entries of relation 1 only; all other
    vertices are of type 1."""
    rng = np.random.default_rng(keep)
    n0 = keep + longs
    lens = np.concatenate([[97, 513, 2049, 8193, 9000], rng.integers(97, 700, longs)])[:longs]
    src = np.concatenate([np.arange(keep), np.repeat(keep + np.arange(longs), lens)])
    dst = np.concatenate([n0 + np.arange(keep), n0 + rng.integers(0, V - n0, int(lens.sum()))])
    rel = np.concatenate([np.zeros(keep), np.ones(int(lens.sum()))])
    return MicroGraph(V, src, dst, rel, (np.arange(V) >= n0).astype(np.int32))


@pytest.fixture(scope="module", params=[LCAP - 40, LCAP - 39, 70000, 78085])
def overflow(request):
    """Roots at a regular list's capacity, one past it, and between it and the
    words of the bitmap (which a graph of more than 64 * 65,536 vertices has
    more of than a list has entries)."""
    mg = wide_root_graph(5_000_000, request.param)
    return request.param, mg, oracle.Graph(mg.V, mg.src, mg.dst, mg.rel, mg.vtype)


@pytest.mark.parametrize("help_items", [1024, 0])
def test_root_survivors_past_the_list(overflow, help_items):
    """A root step whose survivors outgrow the list while longer rows still
    fail their test: the counts run past the list, which then is not
    compacted by them. The root as the first and the last query vertex; the
    slots beside it and the next queries in its slot keep their answers."""
    keep, mg, og = overflow
    print("case: survivors", keep, "help_items", help_items, flush=True)
    rp, col, rel, typ = mg.csr()
    g = P.Graph(rp, col, rel, typ)
    g.set_tuning(help_items=help_items)
    big = [MicroQuery(2, [0, 1], [-1, -1], [0], [1], [0]),
           MicroQuery(3, [1, 1, 0], [-1, -1, -1], [2, 2], [0, 1], [0, -1])]
    small = [MicroQuery(2, [0, 1], [keep + k, -1], [0], [1], [1]) for k in range(8)]
    want = [og.match_query(q) for q in big + small]
    assert len(want[0]) == keep and len(want[1]) == 0
    for q, w in zip(big + small, want):
        assert np.array_equal(g.match_query(q), w)
    for r, w in zip(g.match_batch(big + small), want):
        assert np.array_equal(r, w)
    # the fixed area's one slot: refused past its list, whole again after
    # (how many of the long rows are listed until a later tier drops them
    # depends on the tiers, so a root of just a list's length may do either)
    if keep > LCAP:
        with pytest.raises(P.SGMError):
            g.match_query_noalloc(big[0], 1 << 17)
    for q, w in zip(small, want[2:]):
        assert np.array_equal(g.match_query_noalloc(q, 1 << 14), w)
    g.close()


def tier_graph(cands, hubs, row):
    """`cands` vertices of type 0 with short rows, `hubs` with `row` entries
    and six with 6,000, to the 20,000 vertices of types 1 and 2; each of those
    points back to a few of type 0."""
    rng = np.random.default_rng(cands + hubs)
    n0, T = cands + hubs, 20000
    deg = np.concatenate([rng.integers(1, 6, cands), np.full(hubs - 6, row), np.full(6, 6000)])
    src = np.repeat(np.arange(n0), deg)
    dst = n0 + rng.integers(0, T, len(src))
    back = rng.integers(0, n0, 2 * T)
    src, dst = (np.concatenate([src, n0 + np.arange(2 * T) % T]), np.concatenate([dst, back]))
    vt = np.concatenate([np.zeros(n0), 1 + (np.arange(T) % 8 == 0)])
    return MicroGraph(n0 + T, src, dst, rng.integers(0, 2, len(src)), vt)


@pytest.mark.parametrize("wg_rows", [64, 1024])
def test_no_tier_is_posted_after_a_give_up(wg_rows):
    """Steps whose candidates, long rows, longest rows and row segments are
    all shared, given up after one poll (forced from the host): the step ends
    there, and every table is the oracle's."""
    mg = tier_graph(3000, 80, 1200)
    og = oracle.Graph(mg.V, mg.src, mg.dst, mg.rel, mg.vtype)
    rp, col, rel, typ = mg.csr()
    g = P.Graph(rp, col, rel, typ)
    qs = [MicroQuery(3, [2, 0, 2], [-1, -1, -1], [0, 1], [1, 2], [0, r]) for r in (0, 1, -1)]
    qs += [MicroQuery(3, [0, 2, 0], [k, -1, -1], [0, 1, 2], [1, 2, 1], [-1, 0, -1]) for k in (0, 3010)]
    want = [og.match_query(q) for q in qs]
    g.set_tuning(slots=2, wg_rows=wg_rows, help_items=64, helpers=512, help_wait=1)
    gave_up = 0
    for rep in range(4):
        got, stats = g.match_batch(qs, with_stats=True)
        for i, (r, w) in enumerate(zip(got, want)):
            print("case: launch", rep, "query", i, flush=True)
            assert np.array_equal(r, w)
        gave_up += sum(st["fallback"] == 32 for st in stats)
    g.set_tuning(help_wait=0)
    for r, w in zip(g.match_batch(qs), want):
        assert np.array_equal(r, w)
    print("given up:", gave_up, flush=True)
    g.close()


@pytest.mark.parametrize("help_items", [1024, 0])
@pytest.mark.parametrize("kids", [LCAP - 1, LCAP, LCAP + 1, 90000])
def test_child_list_past_its_capacity(kids, help_items):
    """A step over a few candidates, one with a long row and nine or more
    beside it, that pushes up to and past a list's capacity of children."""
    n0, V = 60, 60 + 100000
    src = np.concatenate([np.repeat(np.arange(n0 - 1), 90), np.full(kids, n0 - 1)])[:kids]
    dst = n0 + np.arange(kids)
    mg = MicroGraph(V, src, dst, np.zeros(kids), (np.arange(V) >= n0).astype(np.int32))
    og = oracle.Graph(V, mg.src, mg.dst, mg.rel, mg.vtype)
    rp, col, rel, typ = mg.csr()
    g = P.Graph(rp, col, rel, typ)
    g.set_tuning(help_items=help_items)
    for q in (MicroQuery(2, [0, 1], [-1, -1], [0], [1], [0]),
              MicroQuery(2, [0, 1], [n0 - 1, -1], [0], [1], [0])):
        print("case: children", kids, "pin", q.vpin[0], flush=True)
        assert np.array_equal(g.match_query(q), og.match_query(q))
    g.close()


@pytest.mark.parametrize("help_items", [1024, 0])
def test_an_overflowing_root_step_stops(help_items):
    """A root whose survivors outgrow the regular list early: the attempt ends
    there, with a small part of the bytes that the whole step moves in the
    larger slot which answers the query."""
    V = 1_500_000
    a = np.arange(V, dtype=np.int32)
    g = P.Graph(np.arange(V + 1, dtype=np.int32), (a + 1) % V, a * 0, a * 0, profile=1)
    g.set_tuning(help_items=help_items)
    print("case: root of", V, "vertices, help_items", help_items, flush=True)
    q = MicroQuery(2, [-1, -1], [-1, -1], [0], [1], [0])
    g.reset_kernel_stats()
    n, st = g.match_query(q, count_only=True, with_stats=True)
    assert n == V and st["fallback"] == 1 and st["path"] == P.SGM_PATH_NARROW
    total = g.kernel_stats()["persist"]["bytes"]
    assert total - st["device_bytes"] < 0.5 * st["phase_bytes"][0]
    g.close()


@pytest.mark.parametrize("extra", [0, 1])
def test_roots_past_the_list_without_helpers(extra):
    """Served queries and launches without helpers give a root with more
    candidates than a regular list on to the larger slot at once (few of them
    would survive here); one with just as many, by its degree bounds, stays."""
    n0, V = LCAP + extra, 200000
    a = np.arange(n0)
    # n0 vertices of type 0 with an out-edge, 1,000 more without
    src, dst = a, V - 1 - a % 5000
    vt = np.where(np.arange(V) < n0 + 1000, 0, 1)
    mg = MicroGraph(V, src, dst, (a % 1000 != 0), vt)
    og = oracle.Graph(V, mg.src, mg.dst, mg.rel, mg.vtype)
    rp, col, rel, typ = mg.csr()
    q = MicroQuery(2, [0, 1], [-1, -1], [0], [1], [0])
    want = og.match_query(q)
    assert len(want) == 66
    g = P.Graph(rp, col, rel, typ)
    print("case: root candidates", n0, flush=True)
    srv = P.Server(g)
    status, rows, st = srv.wait(srv.submit(q), q.n)
    srv.close()
    assert status == P.SGM_OK and np.array_equal(rows, want) and st["fallback"] == extra
    g.set_tuning(help_items=0)
    rows, st = g.match_query(q, with_stats=True)
    assert np.array_equal(rows, want) and st["fallback"] == extra
    g.set_tuning(help_items=1024)
    rows, st = g.match_query(q, with_stats=True)
    assert np.array_equal(rows, want) and st["fallback"] == 0
    g.close()
