"""Work by CSR entry: the weight adjoint on every width of lane group, with
and without the entry map, on graphs with hubs, isolated nodes and rows in any
order; new weights checked entry by entry; degrees of long rows."""
import numpy as np
import pytest

from gpu_helpers import dev_graph, rel_err, say
from nvdgen.graphs import Graph as HostGraph, barabasi_albert, erdos_renyi, star_graph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("model,n", [("star", 3001), ("ba", 4000), ("er", 1000), ("none", 7)])
@pytest.mark.parametrize("k", [1, 2, 3, 8, 13, 32, 33, 64, 70])
def test_grad_weights_by_entry(model, n, k):
    import torch
    import paper_2310_11222_amd as nvd
    rng = np.random.default_rng(n + k)
    g = {"star": lambda: star_graph(n - 1), "ba": lambda: barabasi_albert(n, 3, rng),
         "er": lambda: erdos_renyi(n, n // 2, rng),
         "none": lambda: HostGraph(n, np.array([0]), np.array([n - 1]))}[model]()
    say("grad by entry", model, n, k)
    rows = np.repeat(np.arange(n), np.diff(g.row_ptr))
    # the entries of every row in a random order
    order = np.lexsort((rng.random(g.nnz), rows))
    ci = g.col_idx[order]
    X = rng.standard_normal((n, k + 3))
    gs = rng.standard_normal(k)
    want = -0.5 * (((X[rows, :k] - X[ci, :k]) ** 2) * gs).sum(1)
    size = 0.5 * (((X[rows, :k] - X[ci, :k]) ** 2) * np.abs(gs)).sum(1)
    dg = nvd.Graph(g.row_ptr, ci)
    Xd = torch.from_numpy(X).cuda()[:, :k]
    first = dg.grad_weights(Xd, gs).cpu().numpy()      # rows found in the kernel
    w = rng.uniform(0.5, 2.0, g.num_edges)
    dg.set_weights(w[g.csr_edge][order])
    again = dg.grad_weights(Xd, gs).cpu().numpy()      # from the map
    # k terms of three roundings each, and their sum
    assert (np.abs(first - want) <= (k + 6) * 2.0 ** -52 * size).all()
    assert np.array_equal(first, again)
    deg = np.zeros(n)
    np.add.at(deg, rows, w[g.csr_edge])
    assert rel_err(dg.query()[1], deg).max() <= 1e-13
    bad = w[g.csr_edge][order].copy()
    bad[-1] *= 1.5
    with pytest.raises(nvd.NvdError):
        dg.set_weights(bad)
    bad[-1] = np.nan
    with pytest.raises(nvd.NvdError):
        dg.set_weights(bad)
    assert rel_err(dg.query()[1], deg).max() <= 1e-13
