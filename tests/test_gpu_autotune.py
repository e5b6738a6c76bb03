"""What the autotuner times."""
import numpy as np
import pytest

import paper_1807_08804_amd as P
from tests.micro import MicroQuery, random_graph

pytestmark = pytest.mark.gpu


def test_autotune_times_whole_tables():
    """The sample batches are those of calls that return tables: their last
    join level, ordering and output are run, which a count leaves out."""
    mg = random_graph(np.random.default_rng(3), 20000, 60000, n_types=2, n_rels=3)
    rp, col, rel, typ = mg.csr()
    g = P.Graph(rp, col, rel, typ, profile=1)
    qs = [MicroQuery(2, [a, -1], [-1, -1], [0], [1], [-1]) for a in (0, 1)] * 4
    print("case: autotune on", len(qs), "queries", flush=True)
    tables, counts = [sum(s["device_bytes"] for s in g.match_batch(qs, count_only=c, with_stats=True)[1])
                      for c in (False, True)]
    assert tables > 1.5 * counts
    g.reset_kernel_stats()
    g.autotune(qs, reps=1)
    ks = g.kernel_stats()["persist"]
    assert ks["bytes"] / ks["launches"] > 0.95 * tables
    g.close()
