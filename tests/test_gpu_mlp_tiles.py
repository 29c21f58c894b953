"""GPU: the training and inference kernels over minibatches around its row tiles and block count.

One gradient block takes 16 rows at a time, at most 256 blocks share a minibatch: a
single row, a tile less and more than full, one round of all blocks and a ragged second
one.  Bars: those of the gradient test (binary32 sums against the binary64 oracle:
1e-5 of the loss, 1e-4 of the largest entry of each parameter block).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import mlp as om
from paper_1811_05579_amd.workloads import mlp_init

from test_gpu_mlp import NORM, _model, _oracle_inputs, _rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 15, 16, 17, 4096, 4096 + 21])
def test_gradient_over_row_tiles(n):
    rows = _rows(n, seed=n)
    m = _model()
    loss, g = m.grad(torch.from_numpy(rows).cuda())
    X, t = _oracle_inputs(rows, NORM)
    L, go = om.loss_and_grad(mlp_init().astype(np.float64), X, t)
    assert abs(loss - L) <= 1e-5 * abs(L)
    for a, b in [(0, 320), (320, 384), (384, 4480), (4480, 4544), (4544, 4608), (4608, 4609)]:
        assert np.max(np.abs(g[a:b] - go[a:b])) <= 1e-4 * np.max(np.abs(go[a:b])), (a, b)
    m.close()


@pytest.mark.parametrize("n", [1, 31, 32, 33, 127, 129, 1024 * 128 + 37])
def test_inference_over_row_tiles(n):
    """A wavefront takes 32 rows at a time, 1024 blocks of four wavefronts at most; bar of the inference test."""
    rows = _rows(n, seed=n)
    theta = mlp_init(seed=123, scale=2.0)
    theta[64 * 5:64 * 6] = np.linspace(-0.4, 0.6, 64)                 # b1
    theta[384 + 4096:384 + 4096 + 64] = np.linspace(-0.5, 0.5, 64)    # b2
    theta[4608] = 0.3
    m = _model(theta=theta)
    y = m.predict(torch.from_numpy(rows).cuda()).cpu().numpy()
    X, _ = _oracle_inputs(rows, NORM)
    yo, _ = om.forward(om.bf16_round(theta), X)
    assert np.max(np.abs(y - yo)) <= 1e-4 * max(1.0, np.max(np.abs(yo)))
    m.close()
