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


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("model,n,k,pad", [("ba", 500, 3, 0), ("ba", 500, 63, 2), ("star", 9000, 5, 1),
                                           ("ba", 60000, 7, 0), ("ba", 60000, 13, 3), ("ba", 60000, 28, 0),
                                           ("ba", 60000, 33, 1), ("er", 20000, 100, 0)])
def test_ragged_apply(model, n, k, pad, weighted):
    """Y = L X on k columns of wider arrays whose other entries are NaN (X)
    and have to stay as they are (Y): rows within a lane group, long rows in
    one and in several segments, isolated nodes."""
    import torch
    from nvdgen.graphs import star_graph
    rng = np.random.default_rng(n + k)
    g = {"ba": lambda: barabasi_albert(n, 3, rng), "er": lambda: erdos_renyi(n, n, rng),
         "star": lambda: star_graph(n - 1)}[model]()
    if weighted:
        g = g.with_weights(rng.uniform(0.5, 2.0, g.num_edges))
    say("ragged apply", model, n, k, pad, weighted)
    dg = dev_graph(g)
    X = rng.standard_normal((n, k))
    rows = np.repeat(np.arange(n), np.diff(g.row_ptr))
    w = np.ones(g.nnz) if g.w is None else g.w
    for dtype, eps in ((torch.float64, 2.0 ** -53), (torch.float32, 2.0 ** -24)):
        Xd = _wide(X, pad, pad).to(dtype)
        Y = torch.full((n, k + 2 * pad), 7.0, dtype=dtype, device="cuda")
        dg.laplacian_apply(Xd[:, :k] if pad == 0 else Xd, out=Y[:, pad:pad + k])
        Xr = Xd.double().cpu().numpy()
        diff = w[:, None] * (Xr[rows] - Xr[g.col_idx])
        ref, size = np.zeros((n, k)), np.zeros((n, k))
        np.add.at(ref, rows, diff)
        np.add.at(size, rows, np.abs(diff) + w[:, None] * np.abs(Xr[rows]))
        # every term is rounded a few times and a row's sum once per entry
        deg = np.diff(g.row_ptr)[:, None]
        err = np.abs(Y[:, pad:pad + k].double().cpu().numpy() - ref)
        assert (err <= (deg + 8) * eps * size + 1e-300).all()
        assert bool((Y[:, :pad] == 7.0).all()) and bool((Y[:, pad + k:] == 7.0).all())
