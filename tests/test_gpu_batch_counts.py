"""A batch called again with other pair counts: the sweep's per-call state is
laid out anew, and its arrival counters have to start at zero there."""
import numpy as np
import pytest

from gpu_helpers import dev_graph, rel_err, say
from nvdgen.graphs import barabasi_albert, watts_strogatz

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_sweep_called_with_other_pair_counts(monkeypatch, precision):
    import paper_2310_11222_amd as nvd
    monkeypatch.setenv("NVD_COLUMN", "0")
    rng = np.random.default_rng(11)
    graphs = [watts_strogatz(5000, 6, 0.1, rng), barabasi_albert(700, 3, rng), watts_strogatz(30000, 4, 0.1, rng)]
    P = [rng.random((g.n, 3)) for g in graphs]
    Q = [rng.random((g.n, 3)) for g in graphs]
    dgs = [dev_graph(g) for g in graphs]
    batch = nvd.Batch(dgs)
    for ks in ((2, 1, 3), (1, 1, 1), (1, 1, 1), (2, 2, 2), (3, 1, 1)):
        say("batch counts", precision, ks)
        d, _, info = batch.distances([p[:, :k] for p, k in zip(P, ks)], [q[:, :k] for q, k in zip(Q, ks)],
                                     precision=precision, rtol=1e-9)
        want = np.concatenate([dg.distances(p[:, :k], q[:, :k])[0].cpu().numpy()
                               for dg, p, q, k in zip(dgs, P, Q, ks)])
        assert rel_err(d.cpu().numpy(), want).max() <= 1e-8
        assert all(i["status"] == 0 for i in info)
