"""Pair counts that are no power of two: the rest of the pairs is solved in a
tile wider than it, whose other columns are never read or written.  P, Q are
columns of arrays whose other entries are NaN; every distance against the
oracle, on the multi-kernel path and the cooperative launch, with and without
a starting guess, and in the all-pairs matrix."""
import numpy as np
import pytest

import oracle
from gpu_helpers import dev_graph, rel_err, say
from nvdgen.graphs import barabasi_albert, erdos_renyi

pytestmark = pytest.mark.gpu
TOL = {"fp64": 1e-8, "mixed": 1e-6}


def _case(n, k, model="ba", weighted=False):
    rng = np.random.default_rng(n + k)
    g = barabasi_albert(n, 3, rng) if model == "ba" else erdos_renyi(n, 3 * n, rng)
    if weighted:
        g = g.with_weights(rng.uniform(0.5, 2.0, g.num_edges))
    P = np.where(rng.random((n, k)) < 0.05, rng.random((n, k)), 0.0)
    Q = np.where(rng.random((n, k)) < 0.05, rng.random((n, k)), 0.0)
    return g, P, Q


def _wide(M, left, right):
    import torch
    W = torch.full((M.shape[0], M.shape[1] + left + right), float("nan"), dtype=torch.float64, device="cuda")
    W[:, left:left + M.shape[1]] = torch.from_numpy(M)
    return W[:, left:left + M.shape[1]]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("model,n,k,weighted,precond", [
    ("ba", 40000, 3, False, "jacobi"), ("ba", 60000, 5, True, "jacobi"), ("er", 20000, 7, False, "jacobi"),
    ("ba", 300000, 3, False, "jacobi"), ("ba", 50000, 13, False, "jacobi"), ("ba", 40000, 33, True, "jacobi"),
    ("ba", 40000, 64 + 3, False, "jacobi"), ("ba", 3000, 3, True, "achol")])
def test_ragged_pairs(monkeypatch, precision, model, n, k, weighted, precond):
    g, P, Q = _case(n, k, model, weighted)
    say("ragged", precision, model, n, k, weighted, precond)
    monkeypatch.setenv("NVD_COLUMN", "0")
    dg = dev_graph(g)
    ref = oracle.ge_pcg(g.n, g.row_ptr, g.col_idx, g.w, P, Q)
    rtol = 1e-10 if precision == "fp64" else 1e-8
    d, X, info = dg.distances(_wide(P, 1, 2), _wide(Q, 2, 1), precision=precision, rtol=rtol,
                              return_x=True, precond=precond)
    assert rel_err(d.cpu().numpy(), ref["d"]).max() <= TOL[precision]
    assert all(i["status"] == 0 for i in info) and len(info) == k
    atol = (1e-7 if precision == "fp64" else 1e-5) * np.abs(ref["x"]).max()
    np.testing.assert_allclose(X.cpu().numpy(), ref["x"], rtol=0, atol=atol)
    d2, X2, info2 = dg.distances(P, Q, precision=precision, rtol=rtol, X0=ref["x"], precond=precond)
    assert rel_err(d2.cpu().numpy(), ref["d"]).max() <= TOL[precision]
    assert all(i["iters"] <= 4 for i in info2)
    np.testing.assert_allclose(X2.cpu().numpy(), ref["x"], rtol=0, atol=atol)


@pytest.mark.parametrize("n,m,column", [(40000, 5, "0"), (2000, 5, "1"), (18000, 3, "1")])
def test_ragged_matrix(monkeypatch, n, m, column):
    """All pairs from a ragged solve, and from one block per column (whose
    right-hand sides and residuals come back in node order)."""
    g, P, _ = _case(n, m)
    say("ragged matrix", n, m, column)
    monkeypatch.setenv("NVD_COLUMN", column)
    dg = dev_graph(g)
    iu = np.triu_indices(m, 1)
    ref = oracle.ge_pcg(g.n, g.row_ptr, g.col_idx, g.w, P[:, iu[0]], P[:, iu[1]])["d"]
    for precision in ("fp64", "mixed"):
        D, _, info = dg.pairwise(_wide(P, 1, 3), precision=precision, rtol=1e-9)
        D = D.cpu().numpy()
        assert rel_err(D[iu], ref).max() <= TOL[precision]
        assert np.array_equal(D, D.T) and not np.diag(D).any() and all(i["status"] == 0 for i in info)
    monkeypatch.setenv("NVD_REFINE_STALL_RATIO2", "0")
    D, _, info = dg.pairwise(P, precision="mixed", rtol=1e-9, inner_rtol=1e-2)
    assert rel_err(D.cpu().numpy()[iu], ref).max() <= 1e-8
    assert all(i["flags"] & 1 and i["status"] == 0 for i in info)
