"""NaN and infinite features through the matrix-core kernels.  A hidden unit whose sum is
NaN gives 0 (ReLU as max(., 0), which drops NaN); a bad sample spoils only what depends
on it: its own probability in the forward pass, whose other samples share its tile, and
in the gradient the sums that its values enter.  Checked against float64 with the same
ReLU, to the tolerances of the finite checks."""
import numpy as np
import pytest

from oracle import priority as P
from gpu_helpers import new_context
from paper_2012_03119_amd import gss

pytestmark = pytest.mark.gpu


def _problem(n):
    rng = np.random.default_rng(n)
    params = rng.normal(0, 0.3, P.N_PARAMS).astype(np.float32)
    x = rng.normal(0, 1, (n, 12)).astype(np.float32)
    for i, (k, v) in enumerate([(0, np.nan), (3, np.inf), (7, -np.inf), (11, np.nan), (2, np.inf)]):
        x[(5 + 9 * i) % n, k] = v
    x[n - 1, [1, 4]] = np.inf, -np.inf
    return params, x, (rng.random(n) < 0.3).astype(np.float32)


def _forward(params, x):
    p = P.unpack(params.astype(np.float64))
    x = x.astype(np.float64)
    z1 = x @ p["W1"] + p["b1"]
    h1 = np.fmax(z1, 0.0)
    # products one input at a time: a matrix product may skip or reorder zeros and infinities
    z2 = p["b2"] + sum(h1[:, [i]] * p["W2"][i] for i in range(64))
    h2 = np.fmax(z2, 0.0)
    z3 = p["b3"][0] + sum(h2[:, i] * p["w3"][i] for i in range(64))
    return p, x, h1, h2, z3, 1.0 / (1.0 + np.exp(-z3))


@pytest.mark.parametrize("n", [33, 64, 1000])
def test_forward_with_bad_samples(n):
    print(f"nonfinite forward {n}", flush=True)
    params, x, _ = _problem(n)
    with new_context(100, 64) as ctx:
        got = gss.gss_mlp_forward(ctx.ctx, params, x)
    with np.errstate(all="ignore"):
        want = _forward(params, x)[-1]
    assert np.isfinite(want[np.isfinite(x).all(axis=1)]).all()
    np.testing.assert_allclose(got, want, atol=2e-6, rtol=1e-5)  # (NaN equals NaN)


@pytest.mark.parametrize("n", [17, 64, 5000])
def test_gradient_with_nan_features(n):
    """NaN features: the sample's hidden units are all 0, so that it gives the output
    biases' gradients as any sample, and NaN for its feature's weights alone."""
    print(f"nonfinite gradient {n}", flush=True)
    params, x, y = _problem(n)
    x[np.isinf(x)] = 0.5
    bad = np.isnan(x)
    with new_context(100, 64) as ctx:
        loss, g = gss.gss_mlp_loss_grad(ctx.ctx, params, x, y)
    with np.errstate(all="ignore"):
        p, x64, h1, h2, z3, prob = _forward(params, x)
        dz3 = (prob - y) / n
        dz2 = dz3[:, None] * p["w3"] * (h2 > 0)
        dz1 = (dz2 @ p["W2"].T) * (h1 > 0)
        w1 = sum(x64[[i]].T * dz1[i] for i in range(n))
        want = P.pack({"W1": w1, "b1": dz1.sum(0), "W2": h1.T @ dz2, "b2": dz2.sum(0), "w3": h2.T @ dz3,
                       "b3": np.array([dz3.sum()])})
        want_loss = np.mean(np.logaddexp(0.0, z3) - y * z3)
    spoilt = np.isnan(want)
    assert spoilt.sum() == 64 * bad.any(axis=0).sum() and spoilt.any()
    assert np.array_equal(np.isnan(g), spoilt)
    assert abs(loss - want_loss) <= 1e-5 * max(1.0, abs(want_loss))
    assert np.max(np.abs(g - want)[~spoilt]) <= 2e-5 * np.max(np.abs(want[~spoilt])) + 1e-8
