"""SiLU of the surrogate network over its whole range, through the network's
own entry points: unit 0 of every hidden layer carries one value, the first
layer's z = x_0, and the second layer's weight is a power of two that brings
silu(z) above 17, where FP32 SiLU is the identity (two layers pass it on).

Tolerance.  z log2 e is rounded once (2^-24 of it: |z| 2^-24 of e^-z), the
hardware exponential, the sum, the reciprocal and the products add some
2^-23 each: (|z| + 8) 2^-23.
"""
import numpy as np
import pytest

from synth import make_system

pytestmark = pytest.mark.gpu

H, NIN = 128, 10
W1, B1, W2 = 0, NIN * H, NIN * H + H
W3 = W2 + H * H + H
W4 = W3 + H * H + H


@pytest.fixture(scope="module")
def net():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2306_16493_amd import Context
    from paper_2306_16493_amd.eph import Mlp
    ctx = Context(make_system("toy_sc"))
    m = Mlp(ctx, members=1, n_out=1, seed=1)
    x = np.ones((64, NIN), np.float32)
    x[::2] = -1.0  # mean 0, deviation 1: the normalisation leaves x and y as they are
    m.train(torch.tensor(x, device="cuda"), torch.tensor(x[:, :1].copy(), device="cuda"), steps=1, batch=32)
    yield m, torch
    m.close()
    ctx.close()


def chain(m, scale):
    p = np.zeros((1, m.n_params), np.float32)
    p[0, W1] = p[0, W3] = p[0, W4] = 1.0
    p[0, W2] = scale
    m.set_params(p)


def inputs(torch, z):
    x = np.zeros((len(z), NIN), np.float32)
    x[:, 0] = z
    return torch.tensor(x, device="cuda")


@pytest.mark.parametrize("lo,hi,exponent", [(-85.0, -60.0, 125), (-60.0, -1.0, 90), (-1.0, -1e-6, 30), (1e-6, 1.0, 30),
                                            (1.0, 87.0, 7)])
def test_accuracy(net, lo, hi, exponent):
    m, torch = net
    sign = -1.0 if hi < 0 else 1.0
    chain(m, sign * 2.0 ** exponent)
    z = np.linspace(lo, hi, 20001).astype(np.float32)
    z64 = z.astype(np.float64)
    want = z64 / (1.0 + np.exp(-z64))
    got = m.predict(inputs(torch, z)).cpu().numpy().ravel().astype(np.float64) * 2.0 ** -exponent * sign
    err = np.abs(got / want - 1.0)
    print(f"[silu] {lo} .. {hi}: max rel err {err.max() * 2 ** 23:.1f} x 2^-23", flush=True)
    assert np.all(err < (np.abs(z64) + 8.0) * 2.0 ** -23)


@pytest.mark.parametrize("z", [-87.5, -88.5, -100.0, -1e4, -1e20, -1e30, -1e37, -3e38])
def test_far_negative_is_zero(net, z):
    """silu and its derivative are below 1e-35 (z = -87.5: 9e-37 and 1e-36 by
    value), zero once e^-z overflows."""
    m, torch = net
    chain(m, -2.0 ** 20)
    y = m.predict(inputs(torch, [z] * 3)).cpu().numpy()
    assert np.all(np.abs(y) < 1e-35 * 2.0 ** 20)
    _, g = m.gradient(inputs(torch, [z] * 32), torch.ones(32, 1, device="cuda"))
    # by the first layer's bias: silu'(z) through two layers at 0 (1/2 each), 2^20 and 2 (y - 1)
    assert np.all(np.abs(g[0, B1:B1 + H]) < 1e-35 * 2.0 ** 20)


def test_not_a_number_stays(net):
    m, torch = net
    chain(m, 1.0)
    y = m.predict(inputs(torch, [1.0, np.nan, 1.0])).cpu().numpy().ravel()
    assert np.isfinite(y[[0, 2]]).all() and np.isnan(y[1])
