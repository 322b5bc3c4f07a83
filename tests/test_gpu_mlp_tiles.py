"""The training gradient at the edges of its tiles (16 samples) and of its grid
(256 workgroups): against the float64 oracle, with the bounds of the other
gradient tests (FP32 sums: 2e-5 of the largest entry; loss 1e-5)."""
import numpy as np
import pytest
import torch

from oracle import mlp
from paper_2002_05024_amd import binding as neig

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [2, 15, 16, 17, 33, 4095, 4096, 4097, 8209])
def test_grad_tiles(B):
    g = np.random.default_rng(100 + B)
    theta = mlp.init(B).astype(np.float32)
    X = g.standard_normal((B, mlp.NIN)).astype(np.float32)
    a, c = g.integers(0, 8, B).astype(np.int32), g.integers(0, 8, B).astype(np.int32)
    w = g.exponential(1.0, B).astype(np.float32)
    L0, g0 = mlp.loss_and_grad(theta.astype(np.float64), X.astype(np.float64), a, c, w.astype(np.float64))
    dev = [torch.from_numpy(x).cuda() for x in (X, a, c, w, theta)]
    for _ in range(2):  # the second call reuses the workspace
        loss, grad = neig.mlp_grad(*dev)
        g1 = grad.cpu().numpy().astype(np.float64)
        assert abs(float(loss.item()) - L0) <= 1e-5 * max(1.0, abs(L0))
        assert np.all(np.abs(g1 - g0) <= 2e-5 * np.max(np.abs(g0)) + 1e-7)
        assert np.all(g1[: 2 * mlp.NIN] == 0.0)
