"""Which solver runs at the limits of the one-block solver.  It needs none of
the tiles' workspace, so a call that is then made with it off (NVD_COLUMN=0)
finds that workspace missing and the handle's device memory grows; a batch
counts its calls by blocks as direct launches."""
import numpy as np
import pytest

from gpu_helpers import dev_graph, say
from nvdgen import ws_connected
from nvdgen.graphs import star_graph, watts_strogatz

pytestmark = pytest.mark.gpu


def _solved_by_blocks(monkeypatch, dg, P, Q, **kw):
    monkeypatch.setenv("NVD_COLUMN", "1")
    dg.distances(P, Q, **kw)
    first = dg.stats()["device_bytes"]
    monkeypatch.setenv("NVD_COLUMN", "0")
    dg.distances(P, Q, **kw)
    return dg.stats()["device_bytes"] > first


@pytest.mark.parametrize("n,precision,precond,blocks", [
    (2, "fp64", "jacobi", True), (17408, "fp64", "jacobi", True), (17409, "fp64", "jacobi", False),
    (17409, "mixed", "jacobi", True), (32768, "mixed", "jacobi", True), (32769, "mixed", "jacobi", False),
    (17408, "fp64", "achol", True), (17409, "fp64", "achol", False), (24576, "mixed", "achol", True),
    (24577, "mixed", "achol", False), (9000, "mixed", "tree", True), (17409, "mixed", "tree", False)])
def test_limits_of_a_graph(monkeypatch, n, precision, precond, blocks):
    rng = np.random.default_rng(n)
    g = star_graph(n - 1) if n == 2 else watts_strogatz(n, 4, 0.1, rng)
    P, Q = rng.random((n, 2)), rng.random((n, 2))
    say("route", n, precision, precond)
    assert _solved_by_blocks(monkeypatch, dev_graph(g), P, Q, precision=precision, precond=precond,
                             rtol=1e-8) == blocks


def test_calls_that_keep_the_tiles(monkeypatch):
    """A tile asked for, a warm start, the switches of the other solvers."""
    rng = np.random.default_rng(1)
    g = watts_strogatz(1000, 4, 0.1, rng)
    P, Q = rng.random((1000, 2)), rng.random((1000, 2))
    say("route of tiles")
    assert _solved_by_blocks(monkeypatch, dev_graph(g), P, Q)
    assert not _solved_by_blocks(monkeypatch, dev_graph(g), P, Q, tile_k=2)
    assert not _solved_by_blocks(monkeypatch, dev_graph(g), P, Q, X0=np.zeros((1000, 2)))
    monkeypatch.setenv("NVD_SMALL", "0")
    assert not _solved_by_blocks(monkeypatch, dev_graph(g), P, Q)


@pytest.mark.parametrize("n,precision,blocks", [(17408, "fp64", True), (17409, "fp64", False),
                                                (17409, "mixed", True), (24576, "mixed", True),
                                                (24577, "mixed", False)])
def test_limits_of_a_batch(monkeypatch, n, precision, blocks):
    import paper_2310_11222_amd as nvd
    monkeypatch.setenv("NVD_COLUMN", "1")
    rng = np.random.default_rng(n)
    hosts = [ws_connected(m, 6, 0.1, np.random.SeedSequence([m, i])) for i, m in enumerate((500, n, 800))]
    batch = nvd.Batch([dev_graph(g) for g in hosts])
    say("route of a batch", n, precision)
    batch.distances([rng.random((g.n, 2)) for g in hosts], [rng.random((g.n, 2)) for g in hosts],
                    precision=precision)
    assert batch.query()["eager"] == (1 if blocks else 0)
