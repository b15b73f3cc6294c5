"""Training batches with features or targets that are not finite: the loss says so
exactly where the network's output does, and a NaN feature reaches no gradient but
its own column's."""
import numpy as np
import pytest

from paper_1005_5384_amd import learned as L
from paper_1005_5384_amd import octgrav as og

pytestmark = pytest.mark.gpu

NAN_BITS = [0x7FC00000, 0xFFC00000, 0x7FFFFFFF, 0xFFFFFFFF, 0x7F800001, 0xFF800001]


def _batch(b):
    rng = np.random.default_rng(b)
    x = rng.uniform(0, 2, (b, 12)).astype(np.float32)
    return x, (-4 + rng.normal(0, 1, b)).astype(np.float32)


def _pinball(y, t, tau):
    r = t.astype(np.float64) - y.astype(np.float64)
    return np.where(r > 0, tau * r, (tau - 1) * r).mean()


def _step(x, t, params):
    import torch
    m = og.Mlp(params)
    xd = torch.from_numpy(x).cuda()
    y = m.forward(xd).cpu().numpy()
    loss, g = m.loss_grad(xd, torch.from_numpy(t).cuda(), tau=0.9)
    return y, loss, g


@pytest.mark.parametrize("bits", NAN_BITS)
@pytest.mark.parametrize("b,sample,k", [(1, 0, 0), (100, 17, 5), (5000, 4999, 11)])
def test_nan_features(bits, b, sample, k):
    x, t = _batch(b)
    x.view(np.uint32)[sample, k] = bits
    y, loss, g = _step(x, t, L.init_params(2))
    assert np.isfinite(np.delete(y, sample)).all()
    assert np.isnan(loss) == np.isnan(y[sample])
    if not np.isnan(loss):
        assert abs(loss - _pinball(y, t, 0.9)) <= 1e-5 * abs(loss)
    nan = np.isnan(g)
    w1 = nan[:768].reshape(64, 12)
    assert w1[:, k].all() and not np.delete(w1, k, 1).any() and not nan[768:].any()
    assert np.isfinite(g[~nan]).all()


@pytest.mark.parametrize("v", [np.inf, -np.inf, 3.4e38, -3.4e38, 1e-45])
def test_extreme_features(v):
    x, t = _batch(70)
    x[3, 2] = v
    y, loss, _ = _step(x, t, L.init_params(2))
    ref = _pinball(y, t, 0.9)
    assert (np.isnan(loss) and np.isnan(ref)) or loss == ref or abs(loss - ref) <= 1e-5 * abs(ref)


@pytest.mark.parametrize("v", [np.nan, np.inf, -np.inf])
def test_targets(v):
    x, t = _batch(130)
    ref = _step(x, t, L.init_params(2))
    t[65] = v
    y, loss, g = _step(x, t, L.init_params(2))
    assert np.array_equal(y, ref[0])
    assert np.isnan(loss) if np.isnan(v) else loss == np.inf
    assert np.isfinite(g).all()
