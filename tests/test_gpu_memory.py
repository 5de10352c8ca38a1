"""Calls on a device whose memory does not hold the faster form (forced from
the host: NVD_ALLOC_LIMIT fails larger allocations): they go on with the form
that needs less, and their results are right."""
import numpy as np
import pytest

import oracle
from nvdgen import Graph

from gpu_helpers import dev_graph, rel_err, say

pytestmark = pytest.mark.gpu
TOL = {"fp64": 1e-8, "mixed": 1e-6}


def _ring(n, rng, extra=3):
    """A ring and extra random links per node: few iterations at any size."""
    i = np.arange(n)
    e = np.concatenate([np.stack([i, (i + 1) % n], 1), rng.integers(0, n, (extra * n, 2))])
    e = e[e[:, 0] != e[:, 1]]
    e = np.unique(e.min(1).astype(np.int64) * n + e.max(1))
    return Graph(n, e // n, e % n)


def _tile_bytes(n, T):
    return 8 * n * T


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_ragged_tile_wider_than_memory(monkeypatch, precision):
    """Three pairs take a tile of four; where four columns do not fit, tiles
    of two and one."""
    n = 1_500_000
    rng = np.random.default_rng(1)
    g = _ring(n, rng)
    P = np.where(rng.random((n, 3)) < 0.01, rng.random((n, 3)), 0.0)
    Q = np.where(rng.random((n, 3)) < 0.01, rng.random((n, 3)), 0.0)
    say("ragged tile, memory", precision)
    free = dev_graph(g)
    want, Xw, _ = free.distances(P, Q, precision=precision, rtol=1e-10, return_x=True)
    Dw = free.pairwise(P, precision=precision, rtol=1e-10)[0]
    free.close()
    dg = dev_graph(g)
    # between a vector of two columns and one of four
    limit = _tile_bytes(n, 3)
    monkeypatch.setenv("NVD_ALLOC_LIMIT", str(limit))
    for _ in range(2):
        d, X, info = dg.distances(P, Q, precision=precision, rtol=1e-10, return_x=True)
        assert all(i["status"] == 0 for i in info)
        assert rel_err(d.cpu().numpy(), want.cpu().numpy()).max() <= TOL[precision]
        assert float((X - Xw).abs().max()) <= 1e-6 * float(Xw.abs().max())
    say("ragged matrix, memory", precision)
    dg.close()
    monkeypatch.delenv("NVD_ALLOC_LIMIT")
    dg = dev_graph(g)
    monkeypatch.setenv("NVD_ALLOC_LIMIT", str(limit))
    D = dg.pairwise(P, precision=precision, rtol=1e-10)[0]
    assert rel_err(D.cpu().numpy(), Dw.cpu().numpy()).max() <= TOL[precision]
    # no room for one column: refused, as ever
    import paper_2310_11222_amd as nvd
    dg.close()
    monkeypatch.delenv("NVD_ALLOC_LIMIT")
    dg = dev_graph(g)
    monkeypatch.setenv("NVD_ALLOC_LIMIT", str(_tile_bytes(n, 1) // 2))
    with pytest.raises(nvd.NvdError) as ei:
        dg.distances(P, Q, precision=precision)
    assert ei.value.status == 7          # NVD_E_NOMEM
    monkeypatch.delenv("NVD_ALLOC_LIMIT")
    d, _, _ = dg.distances(P, Q, precision=precision, rtol=1e-10)
    assert rel_err(d.cpu().numpy(), want.cpu().numpy()).max() <= TOL[precision]


def test_tree_tile_wider_than_memory(monkeypatch):
    """The forest's scans need twice as much for each column of a tile."""
    n = 1_500_000
    rng = np.random.default_rng(2)
    i = np.arange(1, n)
    g = Graph(n, i, (rng.random(n - 1) * i).astype(np.int64))      # a tree of depth about log n
    P = np.where(rng.random((n, 3)) < 0.01, rng.random((n, 3)), 0.0)
    Q = np.zeros((n, 3))
    say("tree tile, memory")
    free = dev_graph(g)
    want, _, info = free.distances(P, Q, precond="tree")
    want = want.cpu().numpy()
    assert all(i["status"] == 0 for i in info)
    free.close()
    dg = dev_graph(g)
    monkeypatch.setenv("NVD_ALLOC_LIMIT", str(_tile_bytes(2 * n, 3)))
    for _ in range(2):
        d, _, info = dg.distances(P, Q, precond="tree")
        assert all(i["status"] == 0 for i in info)
        assert rel_err(d.cpu().numpy(), want).max() <= TOL["fp64"]


@pytest.mark.parametrize("what", ["layout", "scratch", "preconditioner"])
def test_one_block_solver_without_memory(monkeypatch, what):
    """A small graph whose layout, or the vectors of its columns, do not fit
    is solved by tiles, that call and the later ones; other graphs are not
    concerned."""
    n, k = 6000, 40
    rng = np.random.default_rng(4)
    g = _ring(n, rng)
    P, Q = rng.random((n, k)), rng.random((n, k))
    precond = "achol" if what == "preconditioner" else "jacobi"
    say("one block, memory", what)
    ref = oracle.ge_pcg(n, g.row_ptr, g.col_idx, None, P, Q)
    dg = dev_graph(g)
    monkeypatch.setenv("NVD_COLUMN", "0")              # the tiles' workspace (and the factor) first
    tiled, _, _ = dg.distances(P, Q, precision="mixed", precond=precond)
    before = dg.stats()["device_bytes"]
    monkeypatch.setenv("NVD_COLUMN", "1")
    # the layout takes some 400 KB, the factor's as much, the vectors 8 MB
    monkeypatch.setenv("NVD_ALLOC_LIMIT", str(4000 if what == "layout" else 4 << 20))
    for _ in range(2):
        d, X, info = dg.distances(P, Q, precision="mixed", rtol=1e-10, return_x=True, precond=precond)
        assert all(i["status"] == 0 for i in info)
        assert rel_err(d.cpu().numpy(), ref["d"]).max() <= TOL["mixed"]
        np.testing.assert_allclose(X.cpu().numpy(), ref["x"], rtol=0, atol=1e-5 * np.abs(ref["x"]).max())
    D = dg.pairwise(P[:, :5], precision="fp64")[0].cpu().numpy()
    monkeypatch.delenv("NVD_ALLOC_LIMIT")
    if what != "preconditioner":
        assert dg.stats()["device_bytes"] == before    # nothing of it is left
    again, _, _ = dg.distances(P, Q, precision="mixed", precond=precond)
    assert rel_err(again.cpu().numpy(), tiled.cpu().numpy()).max() <= 1e-12
    other = dev_graph(g)
    assert rel_err(other.pairwise(P[:, :5])[0].cpu().numpy(), D).max() <= TOL["fp64"]
    assert other.stats()["device_bytes"] > 0


def test_new_weights_without_memory_for_the_entry_map(monkeypatch):
    """Weights are checked and taken, and their gradient formed, without the
    map of rows and mirror entries."""
    import torch
    import paper_2310_11222_amd as nvd
    n = 3000
    rng = np.random.default_rng(5)
    g = _ring(n, rng)
    gw = g.with_weights(rng.uniform(0.5, 2.0, g.num_edges))
    say("entry map, memory")
    dg = dev_graph(g.with_weights(np.ones(g.num_edges)))
    monkeypatch.setenv("NVD_ALLOC_LIMIT", "1000")
    for _ in range(2):
        dg.set_weights(gw.w)
        deg = np.zeros(n)
        np.add.at(deg, np.repeat(np.arange(n), np.diff(g.row_ptr)), gw.w)
        assert rel_err(dg.query()[1], deg).max() <= 1e-13
        for at, value in ((0, np.nan), (-1, gw.w[-1] * 1.5), (g.nnz // 2, -1.0)):
            bad = gw.w.copy()
            bad[at] = value
            with pytest.raises(nvd.NvdError) as ei:
                dg.set_weights(bad)
            assert ei.value.status == 2          # NVD_E_GRAPH
    X = torch.from_numpy(rng.standard_normal((n, 3))).cuda()
    without = dg.grad_weights(X, np.ones(3))
    monkeypatch.delenv("NVD_ALLOC_LIMIT")
    dg.set_weights(gw.w)
    assert torch.equal(dg.grad_weights(X, np.ones(3)), without)
