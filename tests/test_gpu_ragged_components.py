"""Ragged pair counts on a graph of a giant component and isolated nodes: the
time of its means grows with every column of the tile, used or not, so the rest
does not go into a wider one (the workspace stays that of the narrower tile)."""
import numpy as np
import pytest

from gpu_helpers import dev_graph, rel_err, say
from nvdgen.graphs import erdos_renyi, watts_strogatz

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("k,tile", [(5, 4), (9, 8)])
def test_tiles_of_a_giant_component(precision, k, tile):
    rng = np.random.default_rng(k)
    n = 60000
    g = erdos_renyi(n, 5 * n, rng)
    whole = watts_strogatz(n, 10, 0.1, rng)
    say("ragged components", precision, k)
    P, Q = rng.random((n, k)), rng.random((n, k))
    held = []
    for graph in (g, whole):
        dg = dev_graph(graph)
        assert (dg.stats()["n_comp"] > 1) == (graph is g)
        dg.distances(P[:, :tile], Q[:, :tile], precision=precision, tile_k=tile)
        narrow = dg.stats()["device_bytes"]
        d, _, info = dg.distances(P, Q, precision=precision)
        assert all(i["status"] == 0 for i in info)
        held.append(dg.stats()["device_bytes"] > narrow)
        one, _, _ = dg.distances(P[:, -1:], Q[:, -1:], precision=precision)
        assert rel_err(d.cpu().numpy()[-1:], one.cpu().numpy()).max() <= 1e-6
    assert held == [False, True]                 # one component: a tile of twice the width
