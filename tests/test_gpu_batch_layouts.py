"""The layouts by which blocks solve a batch of small graphs: on the device only
once a call is solved by blocks, with the weights that the batch was made with;
where they do not fit, the batch is swept."""
import numpy as np
import pytest

from gpu_helpers import dev_graph, rel_err, say
from nvdgen import ws_connected

pytestmark = pytest.mark.gpu


def _batch(n, G, seed, weighted=True):
    rng = np.random.default_rng(seed)
    hosts = [ws_connected(n, 6, 0.1, np.random.SeedSequence([seed, i])) for i in range(G)]
    if weighted:
        hosts = [g.with_weights(rng.uniform(0.5, 2.0, g.num_edges)) for g in hosts]
    P, Q = [rng.random((g.n, 2)) for g in hosts], [rng.random((g.n, 2)) for g in hosts]
    return hosts, P, Q


def test_other_solvers_hold_no_layouts(monkeypatch):
    """32 graphs of 16,000 nodes: 58 MB packed, as much again in layouts."""
    import torch
    import paper_2310_11222_amd as nvd
    hosts, P, Q = _batch(16000, 32, 51)
    dgs = [dev_graph(g) for g in hosts]
    torch.cuda.synchronize()
    say("layouts, memory")
    free = torch.cuda.mem_get_info()[0]
    batch = nvd.Batch(dgs)
    assert free - torch.cuda.mem_get_info()[0] <= 80 << 20
    swept = batch.distances(P, Q, persistent=True)[0].cpu().numpy()
    free = torch.cuda.mem_get_info()[0]
    d = batch.distances(P, Q)[0].cpu().numpy()
    assert free - torch.cuda.mem_get_info()[0] >= 40 << 20
    assert rel_err(d, swept).max() <= 1e-6


def test_weights_are_those_of_the_creation(monkeypatch):
    """New weights of a graph, and its end, before the first call by blocks."""
    import paper_2310_11222_amd as nvd
    hosts, P, Q = _batch(1200, 3, 52)
    dgs = [dev_graph(g) for g in hosts]
    want = np.concatenate([dg.distances(p, q)[0].cpu().numpy() for dg, p, q in zip(dgs, P, Q)])
    batch = nvd.Batch(dgs)
    say("layouts, weights")
    for dg, g in zip(dgs, hosts):
        dg.set_weights(3.0 * g.w)
    dgs[1].close()
    d, _, _ = batch.distances(P, Q, precision="fp64", rtol=1e-10)
    assert batch.query()["eager"] == 1
    assert rel_err(d.cpu().numpy(), want).max() <= 1e-8


def test_layouts_that_do_not_fit(monkeypatch):
    import paper_2310_11222_amd as nvd
    hosts, P, Q = _batch(2000, 6, 53, weighted=False)
    dgs = [dev_graph(g) for g in hosts]
    want = nvd.Batch(dgs).distances(P, Q, precision="fp64", rtol=1e-10)[0].cpu().numpy()
    batch = nvd.Batch(dgs)
    say("layouts, no memory")
    # the layouts take over 800 KB, two columns' vectors of the sweep 192 KB
    monkeypatch.setenv("NVD_ALLOC_LIMIT", "400000")
    for calls in (1, 2):
        d, _, info = batch.distances(P, Q, precision="fp64", rtol=1e-10)
        assert all(i["status"] == 0 for i in info)
        assert rel_err(d.cpu().numpy(), want).max() <= 1e-8
        assert batch.query()["eager"] == 0
