"""Gradient of the surrogate at batch sizes around the training step's tiles (32
samples a workgroup, K ranges of at least 128 samples).

Ragged sizes against the FP64 oracle: BF16 roundings of relative 2^-9 through
nine products, sqrt(18) 2^-9 = 0.8 %, bound at five times that (few samples do
not average it).  Whole tiles against the gradients of 32 samples each: the
batch mean scales by a power of two, which BF16 keeps, so n g(n) equals the sum
of 32 g(32) up to the order of FP32 sums (1e-5)."""
import numpy as np
import pytest

from test_gpu_surrogate import _cos, _data, _rel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def net(orc):
    import torch
    assert torch.cuda.is_available()
    from paper_2307_01416_amd import vpmc as V
    c = V.vpmc_create(0)
    p = orc.mlp_init(5) * 0.5
    V.vpmc_surrogate_set_weights(c, p)
    yield V, c, p
    V.vpmc_destroy(c)


@pytest.mark.parametrize("n", [1, 2, 31, 33, 130, 257, 2049, 5000])
def test_ragged_batches(net, orc, n):
    V, c, p = net
    x, y, t = _data(n, seed=n)
    lg, gg = V.vpmc_surrogate_loss_grad(c, x, y, t)
    lo, go = orc.mlp_loss_grad(p, x, y, t)
    assert lg == pytest.approx(lo, rel=4e-2)
    assert _rel(gg, go) <= 4e-2 and _cos(gg, go) > 0.999


@pytest.mark.parametrize("n", [64, 512, 4096])
def test_batches_of_whole_tiles_add_up(net, n):
    V, c, _ = net
    x, y, t = _data(n, seed=3)
    l, g = V.vpmc_surrogate_loss_grad(c, x, y, t)
    parts = [V.vpmc_surrogate_loss_grad(c, x[k:k + 32], y[k:k + 32], t[k:k + 32]) for k in range(0, n, 32)]
    want = sum(np.asarray(q, np.float64) for _, q in parts) * (32.0 / n)
    assert l == pytest.approx(np.mean([q for q, _ in parts]), rel=1e-5)
    assert _rel(np.asarray(g, np.float64), want) <= 1e-5
