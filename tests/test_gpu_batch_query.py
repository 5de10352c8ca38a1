"""nvd_batch_query counts every call, whichever solver takes it: the batch of
small graphs that one block per pair solves counts as launched directly."""
import numpy as np
import pytest

from gpu_helpers import dev_graph, say
from nvdgen import ws_connected

pytestmark = pytest.mark.gpu


def test_calls_by_blocks_are_counted(monkeypatch):
    import paper_2310_11222_amd as nvd
    rng = np.random.default_rng(41)
    hosts = [ws_connected(1500, 6, 0.1, np.random.SeedSequence([41, i])) for i in range(8)]
    batch = nvd.Batch([dev_graph(g) for g in hosts])
    P, Q = [rng.random((g.n, 3)) for g in hosts], [rng.random((g.n, 3)) for g in hosts]
    say("batch query")
    assert batch.query() == {"captures": 0, "replays": 0, "eager": 0}
    for calls in (1, 2, 3):
        batch.distances(P, Q)
        assert batch.query() == {"captures": 0, "replays": 0, "eager": calls}
    monkeypatch.setenv("NVD_COLUMN", "0")
    batch.distances(P, Q)
    q = batch.query()
    assert q["eager"] == 3 and q["captures"] >= 1
