"""P and Q whose rows are a different distance apart (columns of wider arrays
beside contiguous blocks): the library takes one row stride for both."""
import numpy as np
import pytest

import oracle
from nvdgen import barabasi_albert

from gpu_helpers import dev_graph, rel_err, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("wide", [(9, 0), (0, 7), (8, 5)])
def test_rows_of_different_strides(wide, noalloc):
    import torch
    rng = np.random.default_rng(sum(wide))
    g = barabasi_albert(700, 3, rng)
    M = [rng.random((g.n, 4)) for _ in range(2)]
    dev = []
    for m, extra in zip(M, wide):
        W = torch.full((g.n, 4 + extra), 5.0, dtype=torch.float64, device="cuda")
        W[:, extra // 2:extra // 2 + 4] = torch.from_numpy(m)
        dev.append(W[:, extra // 2:extra // 2 + 4])
    say("strides", wide, noalloc)
    dg = dev_graph(g)
    ref = oracle.ge_dense(g.n, g.row_ptr, g.col_idx, None, *M)
    d, X, _ = dg.distances(*dev, return_x=True, noalloc=noalloc)
    assert rel_err(d.cpu().numpy(), ref["d"]).max() <= 1e-8
    np.testing.assert_allclose(X.cpu().numpy(), ref["x"], rtol=0, atol=1e-7 * np.abs(ref["x"]).max())
    D, norms = dg.project(*dev)
    delta = M[0] - M[1]
    delta = delta - delta.mean(0)
    # a difference, a mean of 700 terms and its removal
    np.testing.assert_allclose(D.cpu().numpy(), delta, rtol=0, atol=1e-13)
    assert rel_err(norms.cpu().numpy(), np.linalg.norm(delta, axis=0)).max() <= 1e-12


def test_gradients_of_rows_of_different_strides():
    """The forward pass through autograd, of the same views."""
    import torch
    from paper_2310_11222_amd.autograd import distance_sq
    rng = np.random.default_rng(3)
    g = barabasi_albert(500, 3, rng)
    W = torch.from_numpy(rng.random((g.n, 7))).cuda()
    P, Q = W[:, 2:5].requires_grad_(True), torch.from_numpy(rng.random((g.n, 3))).cuda().requires_grad_(True)
    say("strides, autograd")
    ref = oracle.ge_dense(g.n, g.row_ptr, g.col_idx, None, P.detach().cpu().numpy(), Q.detach().cpu().numpy())
    dsq = distance_sq(P, Q, dev_graph(g))
    gP, gQ = torch.autograd.grad(dsq.sum(), (P, Q))
    assert rel_err(np.sqrt(dsq.detach().cpu().numpy()), ref["d"]).max() <= 1e-8
    scale = np.abs(ref["x"]).max()
    np.testing.assert_allclose(gP.cpu().numpy(), 2 * ref["x"], rtol=0, atol=1e-7 * scale)
    np.testing.assert_allclose(gQ.cpu().numpy(), -2 * ref["x"], rtol=0, atol=1e-7 * scale)
