"""GPU: the network's outputs and loss where values are infinite or NaN on the way, against
the same network in numpy with gelu as 0.5 x (1 + erf(x / sqrt 2)): +inf stays +inf, -inf
and NaN give NaN, and no row takes another's.
"""
import numpy as np
import pytest
from scipy.special import erf

torch = pytest.importorskip("torch")

from oracle import mlp as om

from test_gpu_mlp import NORM, _model, _oracle_inputs, _rows

pytestmark = pytest.mark.gpu

N = 70                                                     # two full row tiles and a part
BAD = {0: np.inf, 31: -np.inf, 32: np.nan, 40: 3e38, 69: np.inf}


def _case(weight):
    """All parameters positive, so that a sum of infinities has one sign; W1[3, 0] as given."""
    rng = np.random.default_rng(5)
    theta = rng.uniform(0.25, 2.0, 4609).astype(np.float32)
    theta[3 * 5] = weight
    rows = _rows(N, seed=17)
    rows[:, :5] = NORM[:5] + np.abs(rows[:, :5] - NORM[:5]) + 0.5    # standardised inputs > 0
    for r, v in BAD.items():
        rows[r, 0] = v
    return theta, rows


def _forward(theta, rows):
    """In binary64 rounded to binary32 at each value, as far as the range goes."""
    X, t = _oracle_inputs(rows, NORM)
    W1, b1 = theta[:320].reshape(64, 5), theta[320:384]
    W2, b2 = theta[384:4480].reshape(64, 64), theta[4480:4544]
    gelu = lambda z: 0.5 * z * (1.0 + erf(z / np.sqrt(2.0)))
    narrow = lambda z: z.astype(np.float32).astype(np.float64)
    with np.errstate(all="ignore"):
        h = gelu(narrow(np.sum(W1[None] * narrow(X)[:, None, :], axis=2) + b1))
        h = gelu(narrow(np.sum(W2[None] * h[:, None, :], axis=2) + b2))
        return narrow(h @ theta[4544:4608] + theta[4608]), t


@pytest.mark.parametrize("weight", [1.0, 3.4e38])      # the second is infinite in bfloat16
def test_inference(weight):
    theta, rows = _case(weight)
    m = _model(theta=theta)
    y = m.predict(torch.from_numpy(rows).cuda()).cpu().numpy()
    m.close()
    ref, _ = _forward(om.bf16_round(theta).astype(np.float64), rows)
    assert np.array_equal(np.isnan(y), np.isnan(ref)) and np.array_equal(np.isposinf(y), np.isposinf(ref))
    if weight == 1.0:
        assert np.isposinf(ref[[0, 40, 69]]).all() and np.isnan(ref[[31, 32]]).all() and np.isfinite(ref).sum() == N - 5
    ok = np.isfinite(ref)
    # binary32 sums of 64 positive terms twice, gelu to 2.5e-7
    assert np.all(np.abs(y[ok] - ref[ok]) <= 2e-5 * np.abs(ref[ok]))


def test_loss():
    """One row of +inf makes the loss +inf."""
    theta, rows = _case(1.0)
    rows = rows[[0, 5, 6]]
    m = _model(theta=theta)
    loss, _ = m.grad(torch.from_numpy(rows).cuda())
    m.close()
    ref, t = _forward(theta.astype(np.float64), rows)
    assert np.isposinf(np.mean((ref - t) ** 2)) and np.isposinf(loss)
