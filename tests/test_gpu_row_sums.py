"""FP32 row sums of an odd number of columns on graphs that the sliced apply
serves (NVD_SLICE=1: at any size).  The slices sum a row in FP64 and round
once; a wider pass or tile that takes the odd column with others must not sum
it in FP32."""
import numpy as np
import pytest

import oracle
from nvdgen import Graph

from gpu_helpers import dev_graph, say

pytestmark = pytest.mark.gpu


def _graph(rng, n, weighted):
    """Average degree 100, a hub of 1,500 neighbours and isolated nodes."""
    m = n - 20
    e = rng.integers(0, m, (50 * m, 2))
    hub = rng.choice(np.arange(1, m), 1500, replace=False)
    e = np.concatenate([e, np.stack([np.zeros_like(hub), hub], 1)])
    e = e[e[:, 0] != e[:, 1]]
    e = np.unique(np.stack([e.min(1), e.max(1)], 1), axis=0)
    g = Graph(n, e[:, 0], e[:, 1])
    return g.with_weights(rng.lognormal(0, 1, g.num_edges)) if weighted else g


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("k", [1, 3, 5, 7, 13, 29])
def test_odd_column_of_an_fp32_apply(monkeypatch, k, weighted):
    """One rounding of an FP64 sum: half an ulp of the value, and the FP64
    error of a sum of up to 1,500 terms."""
    import torch
    monkeypatch.setenv("NVD_SLICE", "1")
    rng = np.random.default_rng(50 + k + weighted)
    g = _graph(rng, 4000, weighted)
    say("row sums", k, weighted)
    x = rng.standard_normal((g.n, k)).astype(np.float32)
    y = dev_graph(g).laplacian_apply(torch.from_numpy(x).cuda()).cpu().numpy()[:, -1].astype(np.float64)
    w = None if g.w is None else g.w.astype(np.float32).astype(np.float64)
    L = oracle.laplacian_sparse(g.n, g.row_ptr, g.col_idx, w)
    xl = x[:, -1].astype(np.float64)
    want = L @ xl
    bound = 2.0 ** -24 * np.abs(want) + 1500 * 2.0 ** -53 * (abs(L) @ np.abs(xl)) + 1e-37
    assert (np.abs(y - want) <= 1.01 * bound).all(), (np.abs(y - want) / bound).max()


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("k", [3, 7, 12, 15, 28])
def test_long_rows_of_a_ragged_fp32_apply(k, weighted):
    """Rows of more than 128 neighbours in one pass over a ragged number of
    columns, by default: FP64 sums rounded once, a segment of the row to FP64."""
    import torch
    rng = np.random.default_rng(70 + k + weighted)
    g = _graph(rng, 3000, weighted)
    deg = np.diff(g.row_ptr)
    say("long row sums", k, weighted)
    x = rng.standard_normal((g.n, k)).astype(np.float32)
    y = dev_graph(g).laplacian_apply(torch.from_numpy(x).cuda()).cpu().numpy().astype(np.float64)
    w = None if g.w is None else g.w.astype(np.float32).astype(np.float64)
    L = oracle.laplacian_sparse(g.n, g.row_ptr, g.col_idx, w)
    want = L @ x.astype(np.float64)
    bound = 2.0 ** -24 * np.abs(want) + 1500 * 2.0 ** -53 * (abs(L) @ np.abs(x.astype(np.float64))) + 1e-37
    assert (deg > 128).any()
    assert (np.abs(y - want) <= 1.01 * bound)[deg > 128].all()


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("k", [3, 5, 7, 11])
def test_odd_pair_of_a_mixed_tile(monkeypatch, k, weighted):
    """The residual that one FP32 solve reaches, of the last pair among k and
    of that pair alone (by slices): the same arithmetic, in another order of
    the FP64 sums.  With FP32 row sums it was 1.5 to 2 times as large here."""
    for name, value in (("NVD_SLICE", "1"), ("NVD_SMALL", "0"), ("NVD_COLUMN", "0")):
        monkeypatch.setenv(name, value)
    rng = np.random.default_rng(60 + k + weighted)
    g = _graph(rng, 4000, weighted)
    P, Q = rng.random((g.n, k)), rng.random((g.n, k))
    say("row sums of a tile", k, weighted)
    dg = dev_graph(g)
    kw = dict(precision="mixed", rtol=1e-12, inner_rtol=1e-7, max_refine=1)
    with_others = dg.distances(P, Q, **kw)[2][-1]
    alone = dg.distances(P[:, -1:], Q[:, -1:], **kw)[2][-1]
    assert with_others["iters"] == alone["iters"]
    assert with_others["rel_res"] <= 1.1 * alone["rel_res"], (with_others, alone)
