"""The weight adjoint of solutions that hold infinities (a diverged training
step): where a width of lane group has lanes past the last column, these must
not turn an infinite gradient into NaN."""
import numpy as np
import pytest

from gpu_helpers import dev_graph, say
from nvdgen import barabasi_albert

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 2, 3, 5, 8, 9, 33, 64, 65])
def test_infinite_columns(k):
    import torch
    rng = np.random.default_rng(k)
    g = barabasi_albert(300, 3, rng)
    say("grad inf", k)
    rows = np.repeat(np.arange(g.n), np.diff(g.row_ptr))
    X = rng.standard_normal((g.n, k))
    X[5, k - 1] = np.inf                  # the last column, which idle lanes repeat
    X[9, 0] = -np.inf
    gs = rng.uniform(0.5, 1.0, k)         # of one sign: no sum of opposite infinities
    with np.errstate(invalid="ignore"):
        want = (-0.5 * gs * (X[rows] - X[g.col_idx]) ** 2).sum(1)
    got = dev_graph(g).grad_weights(torch.from_numpy(X).cuda(), gs).cpu().numpy()
    assert np.isinf(want).any()
    # k terms of three roundings each, and their sum
    np.testing.assert_allclose(got, want, rtol=(k + 6) * 2.0 ** -52)
