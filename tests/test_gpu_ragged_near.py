"""The rule of the ragged apply on graphs whose neighbours lie near their rows,
and on others: how many launches a call makes."""
import numpy as np
import pytest

import oracle
from gpu_helpers import dev_graph, say
from nvdgen.graphs import Graph, erdos_renyi, watts_strogatz

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("model,k,one", [("ring", 5, False), ("ring", 12, False), ("ring", 13, False),
                                         ("ring", 28, False), ("ring", 3, True), ("ring", 7, True),
                                         ("ring", 15, True), ("er", 5, True), ("er", 12, True),
                                         ("shuffled", 5, True)])
def test_one_pass_or_several(model, k, one):
    import torch
    import paper_2310_11222_amd as nvd
    n = 120000
    rng = np.random.default_rng(k)
    g = erdos_renyi(n, 4 * n, rng) if model == "er" else watts_strogatz(n, 8, 0.1, rng)
    if model == "shuffled":                       # the same lattice in an order of its own
        at = rng.permutation(n)
        g = Graph(n, at[g.eu], at[g.ev])
    say("ragged near", model, k)
    dg = dev_graph(g)
    X = torch.from_numpy(rng.standard_normal((n, k)).astype(np.float32)).cuda()
    Y = dg.laplacian_apply(X)
    nvd.prof_enable(True)
    dg.laplacian_apply(X, out=Y)
    torch.cuda.synchronize()
    launches = nvd.prof_read()["spmm_f32"]["launches"]
    nvd.prof_enable(False)
    # a pass for every power of two in k, the last ones perhaps as one
    assert (launches == 1) == one and launches <= bin(k).count("1")
    L = oracle.laplacian_sparse(n, g.row_ptr, g.col_idx, None)
    Xh = X.cpu().numpy().astype(np.float64)
    assert not (np.abs(Y.cpu().numpy() - L @ Xh) > 2e-6 * (abs(L) @ np.abs(Xh))).any()
