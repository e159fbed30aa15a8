"""The network's matrix-core kernels at the edges of their tiles: forward around the 32
samples of a wavefront step and past the resident workgroups, the gradient around its
groups of 16 samples and past its 256 workgroups, rows taken through an order.
Tolerances are those of the existing fp32 checks against the float64 oracle."""
import numpy as np
import pytest

from oracle import priority as P
from gpu_helpers import new_context
from paper_2012_03119_amd import gss

pytestmark = pytest.mark.gpu


def _problem(seed, n):
    rng = np.random.default_rng(seed)
    params = rng.normal(0, 0.3, P.N_PARAMS).astype(np.float32)
    return params, rng.normal(0, 1, (n, 12)).astype(np.float32), (rng.random(n) < 0.3).astype(np.float32)


@pytest.mark.parametrize("n", [1, 31, 32, 33, 129, 65_537])
def test_forward_tiles(n):
    print(f"forward {n}", flush=True)
    params, x, _ = _problem(n, n)
    with new_context(100, 64) as ctx:
        got = gss.gss_mlp_forward(ctx.ctx, params, x)
    want = P.forward(params.astype(np.float64), x.astype(np.float64))["prob"]
    np.testing.assert_allclose(got, want, atol=2e-6, rtol=1e-5)


@pytest.mark.parametrize("n", [15, 16, 17, 4096, 4097, 9_001])
def test_gradient_tiles(n):
    print(f"gradient {n}", flush=True)
    params, x, y = _problem(100 + n, n)
    with new_context(100, 64) as ctx:
        loss, g = gss.gss_mlp_loss_grad(ctx.ctx, params, x, y)
    want_loss, want_g = P.loss_grad(params.astype(np.float64), x.astype(np.float64), y.astype(np.float64))
    assert abs(loss - want_loss) <= 1e-5 * max(1.0, abs(want_loss))
    assert np.max(np.abs(g - want_g)) <= 2e-5 * np.max(np.abs(want_g)) + 1e-8


def test_one_step_through_an_order():
    """One Adam step on a ragged batch of scattered rows moves every parameter with a
    gradient by lr (Adam's first step), to within the epsilon's share."""
    params, x, y = _problem(7, 300)
    order = np.random.default_rng(8).permutation(300)[:77].astype(np.uint32)
    with new_context(100, 64) as ctx:
        got, losses = gss.gss_mlp_train(ctx.ctx, params, x, y, order, batch=100, lr=1e-2)
    xb, yb = x[order].astype(np.float64), y[order].astype(np.float64)
    want_loss, g = P.loss_grad(params.astype(np.float64), xb, yb)
    assert abs(losses[0] - want_loss) <= 1e-5 * max(1.0, abs(want_loss))
    step = got.astype(np.float64) - params
    big = np.abs(g) > 1e-3 * np.max(np.abs(g))  # far above fp32 rounding of the batch's sums
    np.testing.assert_allclose(step[big], -1e-2 * np.sign(g[big]), rtol=1e-3, atol=1e-6)
