"""The choice between a block per column and tiles, where both were timed and
one is faster by half or more: dense weighted graphs, whose entries do not stay
in the L2 that a block reads them from, against sparse and small ones."""
import numpy as np
import pytest

from gpu_helpers import dev_graph, say
from nvdgen.graphs import barabasi_albert, watts_strogatz

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("model,n,d,weighted,precision,k,blocks", [
    ("ws", 17000, 48, True, "mixed", 7, False), ("ws", 20000, 48, True, "mixed", 27, False),
    ("ws", 13000, 48, True, "fp64", 5, False), ("ws", 28000, 48, True, "mixed", 27, False),
    ("ws", 500, 8, False, "fp64", 1, True), ("ws", 10007, 16, True, "fp64", 5, True),
    ("ba", 10000, 8, False, "mixed", 8, True), ("ws", 28000, 6, False, "mixed", 48, True),
    ("ba", 17000, 4, True, "mixed", 16, True), ("ws", 4000, 24, True, "mixed", 1, True)])
def test_faster_solver_is_taken(monkeypatch, model, n, d, weighted, precision, k, blocks):
    rng = np.random.default_rng(n + k)
    g = watts_strogatz(n, d, 0.1, rng) if model == "ws" else barabasi_albert(n, d, rng)
    if weighted:
        g = g.with_weights(rng.uniform(0.5, 2.0, g.num_edges))
    P, Q = rng.random((n, k)), rng.random((n, k))
    say("column rule", model, n, d, weighted, precision, k)
    dg = dev_graph(g)
    dg.distances(P, Q, precision=precision, rtol=1e-6)
    first = dg.stats()["device_bytes"]
    monkeypatch.setenv("NVD_COLUMN", "0")
    dg.distances(P, Q, precision=precision, rtol=1e-6)
    # (tiles need a workspace that a call by blocks does not make)
    assert (dg.stats()["device_bytes"] > first) == blocks


@pytest.mark.parametrize("n,precision,k,blocks", [
    (14183, "mixed", 4, False), (14183, "fp64", 4, False), (17000, "fp64", 8, False), (17000, "mixed", 3, False),
    (14183, "mixed", 1, True), (10000, "fp64", 4, True), (17000, "fp64", 16, True), (6000, "mixed", 8, True)])
def test_faster_solver_is_taken_with_a_forest(monkeypatch, n, precision, k, blocks):
    """Two edges a node: the forest is augmented, and costs a block two solves."""
    rng = np.random.default_rng(n + k)
    g = barabasi_albert(n, 2, rng)
    P, Q = rng.random((n, k)), rng.random((n, k))
    say("forest rule", n, precision, k)
    dg = dev_graph(g)
    dg.distances(P, Q, precision=precision, rtol=1e-6, precond="tree")
    first = dg.stats()["device_bytes"]
    monkeypatch.setenv("NVD_COLUMN", "0")
    dg.distances(P, Q, precision=precision, rtol=1e-6, precond="tree")
    assert (dg.stats()["device_bytes"] > first) == blocks


@pytest.mark.parametrize("n,d,k,G,blocks", [(16000, 120, 4, 2, False), (16000, 120, 64, 4, True),
                                            (9000, 12, 1, 2, True), (6000, 200, 4, 2, True)])
def test_faster_solver_is_taken_for_a_batch(n, d, k, G, blocks):
    """Few pairs on few graphs whose entries leave the L2 are swept (a call by
    blocks counts as launched directly)."""
    import paper_2310_11222_amd as nvd
    rng = np.random.default_rng(n + d)
    g = watts_strogatz(n, d, 0.1, rng)
    dg = dev_graph(g)
    batch = nvd.Batch([dg] * G)
    say("batch rule", n, d, k, G)
    P = [rng.random((n, k)) for _ in range(G)]
    batch.distances(P, [p[::-1].copy() for p in P])
    assert batch.query()["eager"] == (1 if blocks else 0)
