"""The network's kernels at the edges of their row counts: a wave's row, a
partial's eight, the 32 rows dealt to four partials, and more partials and rows
than one launch has blocks (1024 x 8).  Inference, loss and gradient against the
FP64 oracle, to the bounds of the network's other tests (2e-5 of the scale)."""
import numpy as np
import pytest

from gpu_common import need_gpu
from oracle import mlp_oracle as M
from test_gpu_mlp import _data

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 4, 5, 7, 8, 9, 31, 32, 33, 129, 2049, 8197])
def test_row_counts_match_oracle(n):
    need_gpu()
    from paper_1004_5058_amd.mlp import MLP
    X, y = _data(8197, seed=5)
    mu, sd = X.mean(0), X.std(0)
    X, y = X[:n], y[:n]
    net = MLP(max_rows=8197)
    theta = M.init_params(2).astype(np.float32)
    net.set_params(theta)
    net.set_norm(mu, sd, 1e-4, 1e-4)
    net.set_data(X, y)
    Xs = (X.astype(np.float64) - mu) / sd
    ys = (y.astype(np.float64) - 1e-4) / 1e-4
    ref, _ = M.forward(theta.astype(np.float64), Xs)
    np.testing.assert_allclose((net.infer(X) - 1e-4) / 1e-4, ref, rtol=0, atol=2e-5)
    loss, g = net.loss_grad()
    lref, gref = M.loss_grad(theta.astype(np.float64), Xs, ys)
    assert loss == pytest.approx(lref, rel=2e-5, abs=1e-7)
    np.testing.assert_allclose(g, gref, rtol=0, atol=2e-5 * np.max(np.abs(gref)))
