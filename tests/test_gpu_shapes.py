"""GPU tests at the sizes where a launch changes form: edges of tiles,
remainders, the smallest and the largest of a range."""
import numpy as np
import pytest

from oracle import mlp
from parity_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 15, 16, 17, 512, 16384, 16385, 20011])
def test_mlp_gradient_sample_counts(n):
    """One partial tile, whole tiles, and more tiles than blocks (1024 blocks
    of 16 samples).  Bound: FP32 forward and backward sums of at most 32 + 32
    + 10 terms, 1e-5 of the largest entry (the bound of the n = 3000 test)."""
    import torch
    from paper_2007_14933_amd import sensor as SN
    say("[gpu shapes] mlp gradient, n =", n)
    rng = np.random.default_rng(n)
    theta = mlp.bf16_round(mlp.init(3) + 0.05 * rng.normal(size=mlp.NPARAM))
    X = np.concatenate([rng.dirichlet(np.ones(4), n), rng.uniform(0, 0.5, (n, 6))], axis=1).astype(np.float32)
    y = (rng.uniform(size=n) < 0.6).astype(np.uint8)
    tr = SN.Trainer()
    tr.w.copy_(torch.from_numpy(mlp.bf16_bits(theta).view(np.int16)).cuda())
    g, L = tr.grad_loss(torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda())
    go = mlp.grad(theta, X.astype(np.float64), y)
    Lo = mlp.loss(theta, X.astype(np.float64), y)
    assert np.abs(g.cpu().numpy() - go).max() <= 1e-5 * np.abs(go).max()
    assert abs(float(L.item()) - Lo) <= 1e-6 * abs(Lo)
