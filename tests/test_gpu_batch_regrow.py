"""Captured launches of a batch after another call has replaced the buffers
that they hold (the vectors grow with the tile, the results with the pairs):
both solvers, in turn, with the same arrays as when they were captured."""
import numpy as np
import pytest

from gpu_helpers import dev_graph, rel_err, say
from nvdgen import barabasi_albert, ws_connected

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("first", [False, True], ids=["sweep", "persistent"])
def test_capture_after_buffers_grew(monkeypatch, first):
    import torch
    import paper_2310_11222_amd as nvd
    monkeypatch.setenv("NVD_COLUMN", "0")
    rng = np.random.default_rng(31)
    hosts = [ws_connected(3000, 6, 0.1, np.random.SeedSequence([31, i])) for i in range(3)]
    hosts.append(barabasi_albert(1500, 4, rng))
    dgs = [dev_graph(g) for g in hosts]
    batch = nvd.Batch(dgs)
    P = [rng.random((g.n, 20)) for g in hosts]
    Q = [rng.random((g.n, 20)) for g in hosts]
    packs = {k: batch.pack([p[:, :k] for p in P], [q[:, :k] for q in Q]) for k in (3, 4, 20)}
    want = np.stack([dg.distances(p, q)[0].cpu().numpy() for dg, p, q in zip(dgs, P, Q)])
    outs = {k: torch.empty(4 * k, dtype=torch.float64, device="cuda") for k in packs}

    def call(k, persistent):
        say("regrow", k, "persistent" if persistent else "sweep")
        outs[k].fill_(-1.0)
        d, _, info = batch.distances(None, None, packed=packs[k], out=outs[k], persistent=persistent)
        assert all(i["status"] == 0 for i in info)
        assert rel_err(d.cpu().numpy().reshape(4, k), want[:, :k]).max() <= 1e-6

    # twice: the work plan, part of the key, follows the iterations of the call before
    for k, persistent in ((3, first), (3, first), (20, not first), (3, first), (4, not first), (3, first),
                          (20, first), (3, not first)):
        call(k, persistent)
