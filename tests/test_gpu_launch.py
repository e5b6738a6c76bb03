"""A batch as one kernel launch: counters that the launch itself resets, and
small tables that the kernel writes to host memory."""
import numpy as np
import pytest

import oracle
import paper_1807_08804_amd as P
from tests.micro import MicroGraph, MicroQuery

pytestmark = pytest.mark.gpu

PREFIX = 16384  # ints of the output arena that are host memory


def pinned_hubs(sizes):
    """A graph with one hub per size, of that many out-neighbours, and the
    queries that list them: `size` rows of two columns each."""
    T = max(sizes) + 1
    src = np.repeat(np.arange(len(sizes)), sizes)
    dst = len(sizes) + np.concatenate([np.arange(k) for k in sizes])
    mg = MicroGraph(len(sizes) + T, src, dst, np.zeros(len(src)), np.zeros(len(sizes) + T))
    qs = [MicroQuery(2, [-1, -1], [h, -1], [0], [1], [0]) for h in range(len(sizes))]
    return mg, qs


@pytest.fixture(scope="module")
def hubs():
    sizes = [1, 2, 3, 100, 4095, PREFIX // 2 - 1, PREFIX // 2, PREFIX // 2 + 1, 20000, 60000]
    mg, qs = pinned_hubs(sizes)
    og = oracle.Graph(mg.V, mg.src, mg.dst, mg.rel, mg.vtype)
    want = [og.match_query(q) for q in qs]
    assert [len(w) for w in want] == sizes
    return mg, qs, want


@pytest.mark.parametrize("slots", [1, 512])
@pytest.mark.parametrize("pick", [(6,), (7,), (5, 0), (0, 5, 0, 6), (6, 0), (3, 7, 3), (4, 4, 4, 4, 0),
                                  (8, 1, 0), (2, 9, 2), (5, 5, 3, 9, 6)])
def test_tables_around_the_host_part_of_the_arena(hubs, pick, slots):
    """Tables that end before, at and past the arena's host part, and small
    ones after those: one slot places them in the order of the queue."""
    mg, qs, want = hubs
    rp, col, rel, typ = mg.csr()
    g = P.Graph(rp, col, rel, typ)
    g.set_tuning(slots=slots)
    for rep in range(3):
        print("case: tables", pick, "launch", rep, flush=True)
        for r, i in zip(g.match_batch([qs[i] for i in pick]), pick):
            assert np.array_equal(r, want[i])
        for r, i in zip(g.match_batch([qs[i] for i in pick[::-1]], projects=[[1]] * len(pick)), pick[::-1]):
            assert np.array_equal(r, want[i][:, 1:])
    g.close()


def test_launches_of_changing_sizes(hubs):
    """One context's launches one after the other, of one query, of more than
    the slots and of a few, counts between tables, and one that fails in
    between: each finds its counters at zero."""
    mg, qs, want = hubs
    rp, col, rel, typ = mg.csr()
    g = P.Graph(rp, col, rel, typ)
    for rep, n in enumerate([1, 1200, 7, 513, 1, 64, 65, 512, 3]):
        print("case: launch", rep, "of", n, "queries", flush=True)
        ids = [(rep + k) % 5 for k in range(n)]
        for r, i in zip(g.match_batch([qs[i] for i in ids]), ids):
            assert np.array_equal(r, want[i])
        assert g.match_batch([qs[i] for i in ids], count_only=True) == [len(want[i]) for i in ids]
        if rep == 3:
            g.inject_fault(0)
            bad = g.match_batch([qs[0], qs[3]])
            assert isinstance(bad[0], P.SGMError) and np.array_equal(bad[1], want[3])
        assert np.array_equal(g.match_query(qs[9]), want[9])
    g.close()
