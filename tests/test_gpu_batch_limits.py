"""Iteration limits of a batch: a run of max_iter iterations that does not
converge counts, and the next refinement step (FP64: restart, two or three runs)
goes on from it, by blocks as in the sweep."""
import numpy as np
import pytest

import oracle
from gpu_helpers import dev_graph, rel_err, say
from nvdgen import ws_connected

pytestmark = pytest.mark.gpu
OK, NOCONV = 0, 4


@pytest.mark.parametrize("precision,max_iter,max_refine,status", [
    ("mixed", 12, 30, OK), ("mixed", 12, 2, NOCONV), ("mixed", 1000, 1, NOCONV), ("fp64", 40, 30, OK),
    ("fp64", 60, 1, OK), ("fp64", 8, 30, NOCONV), ("fp64", 1000, 1, OK)])
def test_limits_by_blocks_and_swept(monkeypatch, precision, max_iter, max_refine, status):
    import paper_2310_11222_amd as nvd
    rng = np.random.default_rng(61)
    hosts = [ws_connected(n, 6, 0.2, np.random.SeedSequence([61, n])) for n in (700, 1100, 2300)]
    P, Q = [rng.random((g.n, 3)) for g in hosts], [rng.random((g.n, 3)) for g in hosts]
    dgs = [dev_graph(g) for g in hosts]
    batch = nvd.Batch(dgs)
    ref = np.concatenate([oracle.ge_dense(g.n, g.row_ptr, g.col_idx, None, p, q)["d"]
                          for g, p, q in zip(hosts, P, Q)])
    kw = dict(precision=precision, rtol=1e-9, max_iter=max_iter, max_refine=max_refine)
    runs = []
    for column in ("1", "0"):
        monkeypatch.setenv("NVD_COLUMN", column)
        say("batch limits", precision, max_iter, max_refine, column)
        d, X, info = batch.distances(P, Q, return_x=True, **kw)
        runs.append((d.cpu().numpy(), info))
        assert [i["status"] for i in info] == [status] * 9, info
        if status == OK:
            assert rel_err(runs[-1][0], ref).max() <= 1e-7
    assert batch.query()["eager"] == 1                    # the first by blocks, the second swept
    if status == NOCONV:
        # what the iterations there were reached (their sums in another order)
        assert rel_err(runs[0][0], runs[1][0]).max() <= 1e-3
        assert max(i["rel_res"] for i in runs[0][1]) <= 2 * max(i["rel_res"] for i in runs[1][1])
