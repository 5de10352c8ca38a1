"""The one-block-per-column solver (column.hip) at the edges of what it takes:
slices of 64 and slots of 1024 positions, graphs whose FP64 vector just fits
the LDS or does not, rows cut into parts, components of every size, ragged and
many columns, and the hand-over from FP32 to FP64 on both sides of that limit.
Every case against the oracle and the multi-kernel path (NVD_COLUMN=0,
NVD_SMALL=0)."""
import numpy as np
import pytest

import oracle
from gpu_helpers import dev_graph, rel_err, say
from nvdgen.graphs import Graph as HostGraph, barabasi_albert, erdos_renyi, star_graph, watts_strogatz

pytestmark = pytest.mark.gpu
TOL = {"fp64": 1e-8, "mixed": 1e-6}


def _pairs(n, k, rng):
    P = np.where(rng.random((n, k)) < 0.1, rng.random((n, k)), 0.0)
    Q = np.where(rng.random((n, k)) < 0.1, rng.random((n, k)), 0.0)
    P[rng.integers(0, n, k), np.arange(k)] += 1.0      # no pair is empty
    return P, Q


def _graph(model, n, rng, weighted):
    if model == "star":
        g = star_graph(n - 1)
    elif model == "ba":
        g = barabasi_albert(n, 3, rng)
    elif model == "ws":
        g = watts_strogatz(n, 6, 0.1, rng)
    elif model == "er":                                 # one giant component, isolated nodes
        g = erdos_renyi(n, 5 * n // 2, rng)
    else:                                               # three big components and 20 of 20 nodes
        parts = [watts_strogatz(m, 4, 0.1, rng) for m in [n // 4, n // 5, n // 6] + [20] * 20]
        eu, ev, at = [], [], 0
        for p in parts:
            eu.append(p.eu + at)
            ev.append(p.ev + at)
            at += p.n
        g = HostGraph(n, np.concatenate(eu), np.concatenate(ev))
    return g.with_weights(rng.uniform(0.5, 2.0, g.num_edges)) if weighted else g


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("model,n,k,weighted", [
    ("star", 2, 1, False), ("ws", 64, 2, True), ("ws", 65, 3, False), ("star", 1500, 2, True),
    ("ba", 1024, 5, False), ("ba", 1025, 1, True), ("er", 3000, 7, True), ("many", 4000, 3, False),
    ("ba", 8193, 2, False), ("ws", 17408, 3, True), ("ba", 17409, 2, False), ("er", 30000, 2, False),
    ("ba", 32768, 2, True), ("ws", 300, 261, False)])
def test_column_solver_matches(monkeypatch, precision, model, n, k, weighted):
    rng = np.random.default_rng(n + k)
    g = _graph(model, n, rng, weighted)
    P, Q = _pairs(g.n, k, rng)
    say("column", precision, model, n, k, weighted)
    dg = dev_graph(g)
    rtol = 1e-10 if precision == "fp64" else 1e-8
    runs = []
    for column in ("1", "0"):
        monkeypatch.setenv("NVD_COLUMN", column)
        if column == "0":
            monkeypatch.setenv("NVD_SMALL", "0")
        runs.append(dg.distances(P, Q, precision=precision, rtol=rtol, return_x=True))
    monkeypatch.delenv("NVD_SMALL")
    (d1, X1, i1), (d2, X2, i2) = runs
    d1, d2, X1, X2 = (v.cpu().numpy() for v in (d1, d2, X1, X2))
    ref = oracle.ge_pcg(g.n, g.row_ptr, g.col_idx, g.w, P, Q)
    assert rel_err(d1, ref["d"]).max() <= TOL[precision]
    assert rel_err(d1, d2).max() <= TOL[precision]
    assert all(i["status"] == 0 and i["rel_res"] <= rtol * 1.01 for i in i1), i1
    # rounding moves the iteration a residual crosses its threshold in by one
    # per solve (in mixed precision there are several)
    steps = 1 if precision == "fp64" else 3
    assert all(abs(a["iters"] - b["iters"]) <= steps for a, b in zip(i1, i2)), (i1, i2)
    scale = np.abs(ref["x"]).max()
    np.testing.assert_allclose(X1, ref["x"], rtol=0, atol=(1e-7 if precision == "fp64" else 1e-5) * scale)
    monkeypatch.setenv("NVD_COLUMN", "1")
    d3, X3, _ = dg.distances(P, Q, precision=precision, rtol=rtol, return_x=True)
    assert np.array_equal(d3.cpu().numpy(), d1) and np.array_equal(X3.cpu().numpy(), X1)


@pytest.mark.parametrize("n", [1200, 20000])
def test_column_hand_over_new_weights_and_strides(monkeypatch, n):
    """FP32 stalls by order: FP64 finishes in one block (n = 1200) or on the
    multi-kernel path (n = 20000); the weights are replaced in between; P and
    Q are columns of wider arrays."""
    import torch
    rng = np.random.default_rng(n)
    g = watts_strogatz(n, 6, 0.1, rng)
    say("column hand-over", n)
    dg = dev_graph(g)
    monkeypatch.setenv("NVD_COLUMN", "1")
    P, Q = _pairs(n, 4, rng)
    d, _, _ = dg.distances(P, Q, precision="mixed", rtol=1e-8)
    assert rel_err(d.cpu().numpy(), oracle.ge_pcg(n, g.row_ptr, g.col_idx, None, P, Q)["d"]).max() <= TOL["mixed"]
    g = g.with_weights(rng.uniform(0.5, 2.0, g.num_edges))
    dg.set_weights(g.w)
    ref = oracle.ge_pcg(n, g.row_ptr, g.col_idx, g.w, P, Q)
    Pw = torch.zeros(n, 9, dtype=torch.float64, device="cuda")
    Qw = torch.full((n, 9), 7.0, dtype=torch.float64, device="cuda")
    Pw[:, 2:6] = torch.from_numpy(P)
    Qw[:, 4:8] = torch.from_numpy(Q)
    monkeypatch.setenv("NVD_REFINE_STALL_RATIO2", "0")
    d, X, info = dg.distances(Pw[:, 2:6], Qw[:, 4:8], precision="mixed", rtol=1e-10, inner_rtol=1e-2,
                              return_x=True)
    monkeypatch.delenv("NVD_REFINE_STALL_RATIO2")
    assert rel_err(d.cpu().numpy(), ref["d"]).max() <= 1e-8
    assert all(i["flags"] & 1 and i["status"] == 0 for i in info)
    np.testing.assert_allclose(X.cpu().numpy(), ref["x"], rtol=0, atol=1e-7 * np.abs(ref["x"]).max())
    d2, _, _ = dg.distances(Pw[:, 2:6], Qw[:, 4:8], precision="fp64", out="dsq")
    assert rel_err(np.sqrt(d2.cpu().numpy()), ref["d"]).max() <= TOL["fp64"]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("precond,model,n,k,weighted", [
    ("achol", "star", 2, 1, True), ("achol", "many", 4000, 3, True), ("achol", "er", 1025, 2, False),
    ("achol", "ba", 6000, 3, True), ("achol", "ws", 17408, 2, False), ("achol", "ba", 24576, 1, False),
    ("tree", "star", 64, 2, True), ("tree", "ring", 1024, 3, True), ("tree", "many", 4000, 2, True),
    ("tree", "ba1", 9000, 3, False), ("tree", "ring", 17408, 2, True), ("tree", "er", 700, 2, True)])
def test_column_preconditioners(monkeypatch, precision, precond, model, n, k, weighted):
    """The factor's rounds and the augmented forest in one block (a forest
    alone, one or a few hundred edges off it; one component, many)."""
    rng = np.random.default_rng(n + k)
    if model == "ring":                                # a cycle with ten chords
        u = np.arange(n)
        a = rng.choice(n // 2 - 2, 10, replace=False)
        g = HostGraph(n, np.concatenate([u[:-1], [0], a]), np.concatenate([u[1:], [n - 1], a + n // 2]))
        g = g.with_weights(rng.lognormal(0, 1, g.num_edges)) if weighted else g
    elif model == "ba1":
        g = barabasi_albert(n, 1, rng)
    else:
        g = _graph(model, n, rng, weighted)
    P, Q = _pairs(g.n, k, rng)
    say("column", precond, precision, model, n, k, weighted)
    dg = dev_graph(g)
    rtol = 1e-10 if precision == "fp64" else 1e-8
    runs = []
    for column in ("1", "0"):
        monkeypatch.setenv("NVD_COLUMN", column)
        runs.append(dg.distances(P, Q, precision=precision, rtol=rtol, return_x=True, precond=precond))
    (d1, X1, i1), (d2, X2, i2) = runs
    d1, d2, X1, X2 = (v.cpu().numpy() for v in (d1, d2, X1, X2))
    assert all(i["status"] == 0 and i["rel_res"] <= rtol * 1.01 for i in i1), i1
    assert rel_err(d1, d2).max() <= TOL[precision]
    # another order of the sums: the counts stay close (a tenth covers FP32
    # recurrences of many iterations)
    assert all(abs(a["iters"] - b["iters"]) <= 2 + b["iters"] // 10 for a, b in zip(i1, i2)), (i1, i2)
    if model in ("star", "er", "ba", "many", "ws"):    # the rest is too long for plain CG on the CPU
        ref = oracle.ge_pcg(g.n, g.row_ptr, g.col_idx, g.w, P, Q)["d"]
        assert rel_err(d1, ref).max() <= TOL[precision]
    monkeypatch.setenv("NVD_COLUMN", "1")
    d3, X3, _ = dg.distances(P, Q, precision=precision, rtol=rtol, return_x=True, precond=precond)
    assert np.array_equal(d3.cpu().numpy(), d1) and np.array_equal(X3.cpu().numpy(), X1)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("sizes,ks", [((2, 64, 1025, 5000, 16384), (1, 3, 64, 2, 5)),
                                      ((17408, 700, 24576), (2, 1, 3)), ((300,) * 40, (7,) * 40)])
def test_column_batch(monkeypatch, precision, sizes, ks):
    """Batches of small graphs, unit and weighted together: a block per
    (graph, pair), against the sweep and against every graph on its own; a
    second call with other pair counts, the first again."""
    import torch
    import paper_2310_11222_amd as nvd
    rng = np.random.default_rng(len(sizes))
    graphs = [star_graph(1) if n == 2 else _graph("ba" if i % 2 else "ws", n, rng, i % 3 != 1)
              for i, n in enumerate(sizes)]
    Ps, Qs = zip(*[_pairs(g.n, k, rng) for g, k in zip(graphs, ks)])
    say("column batch", precision, sizes, ks)
    dgs = [dev_graph(g) for g in graphs]
    batch = nvd.Batch(dgs)
    rtol = 1e-10 if precision == "fp64" else 1e-8
    d1, X1, i1 = batch.distances(Ps, Qs, precision=precision, rtol=rtol, return_x=True)
    assert all(i["status"] == 0 and i["rel_res"] <= rtol * 1.01 for i in i1), i1
    d3, _, _ = batch.distances([p[:, :1] for p in Ps], [q[:, :1] for q in Qs], precision=precision, rtol=rtol)
    d4, X4, _ = batch.distances(Ps, Qs, precision=precision, rtol=rtol, return_x=True)
    assert torch.equal(d1, d4) and torch.equal(X1, X4)
    first = np.cumsum([0] + list(ks))[:-1]
    assert rel_err(d3.cpu().numpy(), d1.cpu().numpy()[first]).max() <= 1e-14
    monkeypatch.setenv("NVD_COLUMN", "0")
    d2, X2, _ = batch.distances(Ps, Qs, precision=precision, rtol=rtol, return_x=True)
    assert rel_err(d1.cpu().numpy(), d2.cpu().numpy()).max() <= TOL[precision]
    tol = (1e-7 if precision == "fp64" else 1e-5) * float(X2.abs().max())
    np.testing.assert_allclose(X1.cpu().numpy(), X2.cpu().numpy(), rtol=0, atol=tol)
    at = 0
    for g, dg, P, Q, k in zip(graphs, dgs, Ps, Qs, ks):
        one, _, _ = dg.distances(P, Q, precision="fp64")
        assert rel_err(d1.cpu().numpy()[at:at + k], one.cpu().numpy()).max() <= TOL[precision]
        at += k
