"""The sliced one-column apply at the edges of its row chunks: a row of 16,384
entries is the largest that a chunk holds, longer ones are summed in pieces,
and a chunk holds no more than 16,384 rows (isolated nodes).  Rows of 16 / 17
and 256 / 257 entries are the edges between a thread, 16 lanes and a wave per
row.  Bounds per entry as in test_gpu_slice: |Y - L X| <= tol (|L| |X|), tol
1e-13 in FP64 and 2e-6 in FP32; the sums take at most 1,024 terms in a row."""
import numpy as np
import pytest

import oracle
from nvdgen import Graph

from gpu_helpers import say, dev_graph, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("hub", [16383, 16384, 16385, 40000])
@pytest.mark.parametrize("nodes", [5000, 20352])
def test_chunk_edges(monkeypatch, hub, weighted, nodes):
    monkeypatch.setenv("NVD_SLICE", "1")
    monkeypatch.setenv("NVD_SLICE_NODES", str(nodes))
    monkeypatch.setenv("NVD_SMALL", "0")
    rng = np.random.default_rng(hub + weighted)
    m, alone = 45000, 20000
    eu, ev = [np.arange(m - 1)], [np.arange(1, m)]          # a path
    for node, deg in ((m // 2, hub), (7, 16), (8, 17), (9, 256), (10, 257), (m - 1, 300)):
        nb = rng.choice(np.setdiff1d(np.arange(20, m), [node - 1, node, node + 1]), deg - 2, replace=False)
        eu.append(np.minimum(nb, node))
        ev.append(np.maximum(nb, node))
    e = np.unique(np.stack([np.concatenate(eu), np.concatenate(ev)], 1), axis=0)
    g = Graph(m + alone, e[:, 0], e[:, 1])
    if weighted:
        g = g.with_weights(rng.lognormal(0, 1, g.num_edges))
    say("chunk edges", hub, weighted, nodes, g.n, g.nnz)
    dg = dev_graph(g)
    X = rng.standard_normal((g.n, 1))
    for dt, tol in (("float64", 1e-13), ("float32", 2e-6)):
        w = None if g.w is None else g.w.astype(dt).astype(np.float64)
        L = oracle.laplacian_sparse(g.n, g.row_ptr, g.col_idx, w)
        Xd = X.astype(dt).astype(np.float64)
        Y = dg.laplacian_apply(to_dev(Xd).to(getattr(__import__("torch"), dt))).cpu().numpy()
        assert not (np.abs(Y - L @ Xd) > tol * (abs(L) @ np.abs(Xd))).any(), dt
