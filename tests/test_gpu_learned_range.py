"""Gradient of the proposal network where dLoss/da2 is of extreme size: row
weights near the end of FP32's normal numbers, infinite and NaN weights.

Small weights: the oracle's gradient of what follows from da2 (W2, b2, W1, b1)
within 1e-5 of the absolute-value sum of its products, as at ordinary sizes, plus 128 B times FP32's smallest step
(2^-149) for the roundings of products below the normal numbers, of which an
entry sums at most that many.  An infinite weight gives infinite entries where
FP32 products do, not NaN; a NaN of any payload gives NaN."""
import numpy as np
import pytest

from oracle import mlp
from paper_2511_07737_amd import tsat

from test_gpu_learned import rand_params, rand_rows

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as T

    if not T.cuda.is_available():
        pytest.skip("no GPU visible")
    return T


def gradient(torch, params, X, y, w):
    net = tsat.Mlp(mlp.flatten(params).astype(np.float32))
    Xd, yd = torch.from_numpy(X).cuda(), torch.from_numpy(y.astype(np.float32)).cuda()
    wd = torch.from_numpy(w).cuda()
    net.train_step_dev(Xd.data_ptr(), yd.data_ptr(), wd.data_ptr(), X.shape[0], 0.0,
                       torch.cuda.current_stream().cuda_stream)
    g, _ = net.get_grad()
    net.close()
    return g


@pytest.mark.parametrize("B", [64, 200])
@pytest.mark.parametrize("exponent", [-90, -108])
def test_small_row_weights(torch, B, exponent):
    params = rand_params(41)
    X = rand_rows(43 + B, B, params)
    y = (np.random.default_rng(B).random(B) < 0.5).astype(np.float64)
    w = np.full(B, 2.0 ** exponent, dtype=np.float32)
    w[:16] *= np.float32(2.0 ** 40)  # rows of both kinds
    w[:8] = 0.0
    for ww in (w, np.full(B, 2.0 ** exponent, dtype=np.float32)):
        g = gradient(torch, params, X, y, ww).astype(np.float64)
        _, ref, _ = mlp.loss_and_grad(params, X.astype(np.float64), y, ww.astype(np.float64))
        bound = mlp.flatten(mlp.abs_grad_bound(params, X.astype(np.float64), y, ww.astype(np.float64)))
        err = mlp.unflatten(np.abs(g - mlp.flatten(ref)))
        lim = mlp.unflatten(1e-5 * bound + 128 * B * 2.0 ** -149)
        for k in ("W2", "b2", "W1", "b1"):
            assert (err[k] <= lim[k]).all(), (k, (err[k] / lim[k]).max())


@pytest.mark.parametrize("bits", [0x7F800000, 0x7FC00000, 0x7FFFFFFF])
def test_non_finite_row_weight(torch, bits):
    B, row = 40, 21
    params = rand_params(41)
    X = rand_rows(44, B, params)
    y = (np.random.default_rng(5).random(B) < 0.5).astype(np.float64)
    w = np.ones(B, dtype=np.float32)
    w[row:row + 1].view(np.uint32)[:] = bits
    gW2 = mlp.unflatten(gradient(torch, params, X, y, w))["W2"]
    f = mlp.forward(params, X.astype(np.float64))
    on1, on2 = f["h1q"][row] > 0, f["a2"][row] > 0
    assert on1.any() and on2.any() and not on1.all() and not on2.all()
    assert np.isfinite(gW2[:, ~on2]).all()
    if bits == 0x7F800000:
        sign = np.sign(mlp.sigmoid(f["out"][row]) - y[row]) * np.sign(f["w3q"][on2])
        assert np.array_equal(gW2[np.ix_(on1, on2)], np.broadcast_to(sign * np.inf, (on1.sum(), on2.sum())))
        assert np.isnan(gW2[np.ix_(~on1, on2)]).all()  # 0 times infinity
    else:
        assert np.isnan(gW2[:, on2]).all()
