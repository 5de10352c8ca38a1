"""nvd_graph_stats' device memory of what the one-block solver keeps: the same
for a graph that became weighted after its first solve as for one that was
weighted from the start, and back to what it was when weights that a forest's
layout holds are replaced."""
import numpy as np
import pytest

from gpu_helpers import dev_graph, say
from nvdgen import watts_strogatz

pytestmark = pytest.mark.gpu


def test_bytes_after_new_weights(monkeypatch):
    monkeypatch.setenv("NVD_COLUMN", "1")
    rng = np.random.default_rng(8)
    g = watts_strogatz(3000, 6, 0.1, rng)
    gw = g.with_weights(rng.uniform(0.5, 2.0, g.num_edges))
    P, Q = rng.random((g.n, 4)), rng.random((g.n, 4))
    say("column bytes")
    a, b = dev_graph(g), dev_graph(gw)
    a.distances(P, Q)                 # unit weights first
    for dg in (a, b):
        for _ in range(2):
            dg.set_weights(gw.w)
            dg.distances(P, Q)
    assert a.stats()["device_bytes"] == b.stats()["device_bytes"]
    before = b.stats()["device_bytes"]
    # (two columns with a forest take the vectors of four without one)
    b.distances(P[:, :2], Q[:, :2], precond="tree")
    with_tree = b.stats()["device_bytes"]
    b.set_weights(gw.w)
    assert with_tree >= before + 12 * g.n
    assert b.stats()["device_bytes"] == before
