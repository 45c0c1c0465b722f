"""The dense backward's products (three-part bf16 operands on the matrix cores) against float64 at the
edges of their tiles, and with values outside the split's range."""
import numpy as np
import pytest
import torch

from paper_2105_08810_amd import snn

pytestmark = pytest.mark.gpu

INF = float("inf")


def _run(T, B, n_in, n_out, eps, trace, W, alpha):
    dev = lambda x: torch.from_numpy(x).cuda()
    dW, gi = snn.dense_backward_ref(dev(W), dev(trace), dev(np.zeros_like(eps)), dev(eps), alpha, INF,
                                    INF, 100.0)
    return dW.cpu().numpy().astype(np.float64), gi.cpu().numpy().astype(np.float64)


def _reference(eps, trace, W, alpha):
    T, B, n_out = eps.shape
    e, tr, w = eps.astype(np.float64), trace.astype(np.float64).reshape(T * B, -1), W.astype(np.float64)
    d = np.zeros_like(e)
    for t in range(T - 1, 0, -1):
        d[t - 1] = alpha * d[t] + e[t]
    return tr.T @ e.reshape(T * B, n_out), (d.reshape(T * B, n_out) @ w.T).reshape(T, B, -1)


@pytest.mark.parametrize("T,B,n_in,n_out", [
    (1, 1, 1, 1), (2, 3, 5, 7), (16, 2, 127, 33), (129, 1, 128, 128), (11, 31, 129, 130), (40, 7, 300, 31),
    (100, 41, 260, 100), (17, 241, 64, 257), (3, 1365, 36, 512)])
def test_dense_products(T, B, n_in, n_out):
    rng = np.random.default_rng(T * B + n_in)
    eps = rng.standard_normal((T, B, n_out)).astype(np.float32) * np.float32(1e-4)
    trace = (rng.random((T, B, n_in)) * 3).astype(np.float32)
    W = rng.standard_normal((n_in, n_out)).astype(np.float32)
    alpha = float(np.float32(0.9))
    dW, gi = _run(T, B, n_in, n_out, eps, trace, W, alpha)
    rW, rg = _reference(eps, trace, W, alpha)
    eW, eg = _reference(np.abs(eps), trace, np.abs(W), alpha)
    # left-out terms below 2^-24, one rounding of the running sum per 16 products (2^-24 of at most the
    # absolute sum each), and for the spike gradient the float32 recurrence (2^-23 a step, over 1 / (1 - alpha))
    u = 2.0 ** -24
    assert (np.abs(dW - rW) <= (T * B / 16 + 8) * 2 * u * eW).all()
    assert (np.abs(gi - rg) <= (n_out / 16 + 8 + 20) * 2 * u * eg).all()


@pytest.mark.parametrize("scale", [-105, -112, -120, -126, -140])
def test_dense_products_tiny_values(scale):
    """Spike gradients that have decayed to 2^scale keep float32's precision (of its subnormals: half a step each)."""
    T, B, n_in, n_out = 3, 120, 140, 136
    rng = np.random.default_rng(-scale)
    eps = np.ldexp(rng.standard_normal((T, B, n_out)), scale).astype(np.float32)
    trace = (rng.random((T, B, n_in)) * 3).astype(np.float32)
    W = rng.standard_normal((n_in, n_out)).astype(np.float32)
    alpha = 0.5
    dW, gi = _run(T, B, n_in, n_out, eps, trace, W, alpha)
    rW, rg = _reference(eps, trace, W, alpha)
    eW, eg = _reference(np.abs(eps), trace, np.abs(W), alpha)
    u, step = 2.0 ** -24, 2.0 ** -149
    # as above; a subnormal result is rounded to half a step, and delta = alpha delta + G to half a step per
    # operation (two of them, at most halved a step after) before its product with W
    assert (np.abs(dW - rW) <= (T * B / 16 + 8) * 2 * u * eW + 0.5 * step).all()
    lost = 2 * step * np.abs(W).sum(1, dtype=np.float64)
    assert (np.abs(gi - rg) <= (n_out / 16 + 8 + 4) * 2 * u * eg + lost + 0.5 * step).all()


@pytest.mark.parametrize("value", [2e38, 2.1e31, 2.026e31, 1.5e31, -INF, np.nan])
def test_dense_products_outside_the_split(value):
    """Values about 2^104 (the end of the split's range) and more, an infinity and a NaN give what float32 products give."""
    T, B, n_in, n_out = 3, 50, 140, 136
    rng = np.random.default_rng(5)
    eps = rng.standard_normal((T, B, n_out)).astype(np.float32)
    eps[2, 7, 130] = value
    trace = (rng.random((T, B, n_in)) < 0.5).astype(np.float32)
    W = rng.standard_normal((n_in, n_out)).astype(np.float32) * np.float32(0.01)
    dW, gi = _run(T, B, n_in, n_out, eps, trace, W, 0.5)
    with np.errstate(invalid="ignore"):
        rW, rg = _reference(eps, trace, W, 0.5)
    for x, r in ((dW, rW), (gi, rg)):
        assert np.array_equal(np.isnan(x), np.isnan(r)) and np.array_equal(np.isinf(x), np.isinf(r))
        ok = np.isfinite(r)
        assert np.array_equal(x[np.isinf(r)], r[np.isinf(r)])
        assert (np.abs(x[ok] - r[ok]) <= 1e-5 * np.maximum(np.abs(r[ok]), 1.0)).all()


def test_dense_products_past_the_range():
    """Products past float32's range are infinities of the product's sign, as float32 products give them, whatever
    the signs of the operands' parts."""
    T, B, n_in, n_out = 2, 130, 140, 136
    rng = np.random.default_rng(9)
    eps = np.zeros((T, B, n_out), np.float32)
    eps[1, np.arange(B), rng.integers(0, n_out, B)] = rng.uniform(0.5, 2, B) * 1e25 * rng.choice([-1, 1], B)
    trace = (rng.random((T, B, n_in)) < 0.5).astype(np.float32)
    W = (rng.uniform(0.5, 2, (n_in, n_out)) * 1e20 * rng.choice([-1, 1], (n_in, n_out))).astype(np.float32)
    dW, gi = _run(T, B, n_in, n_out, eps, trace, W, 0.5)
    rW, rg = _reference(eps, trace, W, 0.5)
    assert (np.abs(rg[0]) > 1e44).all() and np.array_equal(gi[0], np.sign(rg[0]) * INF)
    assert (np.abs(dW - rW) <= 1e-5 * np.abs(rW)).all()
