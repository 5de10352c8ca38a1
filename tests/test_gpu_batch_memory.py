"""Batches of small graphs, a block per (graph, pair), at the limits of their
scratch: more pairs than one launch's vectors hold, and a device (NVD_ALLOC_LIMIT)
without room for the layouts or the vectors, where the batch is swept."""
import numpy as np
import pytest

from gpu_helpers import dev_graph, rel_err, say
from nvdgen import barabasi_albert, cycle_graph, ws_connected

pytestmark = pytest.mark.gpu


def test_many_pairs_on_tiny_graphs(monkeypatch):
    """2,000 graphs of 2 to 30 nodes, 20 pairs each, some weighted: two
    launches (32,768 pairs of up to 1,024 nodes fill one's vectors); then few
    pairs, then the first call again."""
    import torch
    import paper_2310_11222_amd as nvd
    rng = np.random.default_rng(21)
    kinds = [cycle_graph(n) if n > 2 else barabasi_albert(2, 1, rng) for n in range(2, 31)]
    hosts, dgs = [], []
    for i in range(2000):
        g = kinds[i % len(kinds)]
        if i % 7 == 0:
            g = g.with_weights(rng.uniform(0.5, 2.0, g.num_edges))
        hosts.append(g)
        dgs.append(dev_graph(g))
    P = [rng.standard_normal((g.n, 20)) for g in hosts]
    Q = [rng.standard_normal((g.n, 20)) for g in hosts]
    say("batch of tiny graphs")
    batch = nvd.Batch(dgs)
    packed = batch.pack(P, Q)
    d1, X1, info = batch.distances(None, None, packed=packed, precision="fp64", rtol=1e-10, return_x=True)
    assert all(i["status"] == 0 for i in info)
    few = batch.distances([p[:, :1] for p in P], [q[:, :1] for q in Q], precision="fp64", rtol=1e-10)[0]
    d2, X2, _ = batch.distances(None, None, packed=packed, precision="fp64", rtol=1e-10, return_x=True)
    assert torch.equal(d1, d2) and torch.equal(X1, X2)
    d1 = d1.cpu().numpy().reshape(2000, 20)
    assert rel_err(few.cpu().numpy(), d1[:, 0]).max() <= 1e-14
    for i in range(2000):
        g = hosts[i]
        L = np.diag(np.bincount(np.repeat(np.arange(g.n), np.diff(g.row_ptr)),
                                None if g.w is None else g.w, g.n).astype(float))
        L[np.repeat(np.arange(g.n), np.diff(g.row_ptr)), g.col_idx] -= 1.0 if g.w is None else g.w
        b = P[i] - Q[i]
        b = b - b.mean(0)
        want = np.sqrt(np.einsum("ij,ij->j", b, np.linalg.pinv(L) @ b))
        assert rel_err(d1[i], want).max() <= 1e-8, (i, g.n)


@pytest.mark.parametrize("when", ["layout", "scratch"])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_batch_without_memory_is_swept(monkeypatch, when, precision):
    import paper_2310_11222_amd as nvd
    rng = np.random.default_rng(22)
    hosts = [ws_connected(2000, 6, 0.1, np.random.SeedSequence([22, i])) for i in range(6)]
    dgs = [dev_graph(g) for g in hosts]
    P = [rng.random((g.n, 12)) for g in hosts]
    Q = [rng.random((g.n, 12)) for g in hosts]
    say("batch without memory", when, precision)
    rtol = 1e-10 if precision == "fp64" else 1e-8
    tol = 1e-8 if precision == "fp64" else 1e-6
    want = nvd.Batch(dgs).distances(P, Q, precision=precision, rtol=rtol)[0].cpu().numpy()
    # the packed arrays take less than 300 KB each, the layouts over 800, the
    # 72 pairs' vectors 4.7 MB, the sweep's with 16 columns 1.5 MB each
    if when == "layout":
        monkeypatch.setenv("NVD_ALLOC_LIMIT", "400000")
    batch = nvd.Batch(dgs)
    monkeypatch.setenv("NVD_ALLOC_LIMIT", "3000000")
    for _ in range(2):
        d, _, info = batch.distances(P, Q, precision=precision, rtol=rtol)
        assert all(i["status"] == 0 for i in info)
        assert rel_err(d.cpu().numpy(), want).max() <= tol
    assert batch.query()["captures"] >= 1          # (only the sweep and the persistent launch capture)
    # and no room for the sweep either: refused, and well again with room
    monkeypatch.setenv("NVD_ALLOC_LIMIT", "400000")
    batch.close()
    monkeypatch.delenv("NVD_ALLOC_LIMIT")
    batch = nvd.Batch(dgs)
    monkeypatch.setenv("NVD_ALLOC_LIMIT", "400000")
    for persistent in (False, True):
        with pytest.raises(nvd.NvdError) as ei:
            batch.distances(P, Q, precision=precision, rtol=rtol, persistent=persistent)
        assert ei.value.status == 7                # NVD_E_NOMEM
    monkeypatch.delenv("NVD_ALLOC_LIMIT")
    for persistent in (False, True):
        for k in (3, 12):
            d = batch.distances([p[:, :k] for p in P], [q[:, :k] for q in Q], precision=precision, rtol=rtol,
                                persistent=persistent)[0].cpu().numpy()
            assert rel_err(d, want.reshape(6, 12)[:, :k].reshape(-1)).max() <= tol
