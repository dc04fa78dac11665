"""The surrogate's activations over their whole range: sigmoids that are subnormal FP32 numbers
(pre-activations below -87.3), 0 (below -104) and 1.
"""
import numpy as np
import pytest

from oracle import mlp
from workloads.surrogate import init_params, row_order, toy_dataset

from _helpers import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

BLOCKS = [(0, 256), (256, 320), (320, 4416), (4416, 4480), (4480, 4608), (4608, 4610)]


def _extreme_net(seed):
    """Hidden-1 units 0-7 at z of -88.5 to -87.5, their activations of 1e-36 brought back to order one
    by W2; units 8-15 at 92 to 100; units 16-23 below -106, where the activation is zero."""
    import torch
    import paper_1307_3711_amd as lc
    X, Y = toy_dataset(300, seed)
    p = mlp.unpack(init_params(seed).astype(np.float64))
    p["W1"][:24] *= 0.02
    p["b1"][:8] = np.linspace(-88.4, -87.6, 8)
    p["b1"][8:16] = np.linspace(92.0, 100.0, 8)
    p["b1"][16:24] = np.linspace(-120.0, -106.0, 8)
    p["W2"][:, :8] *= 1e36
    p["W2"][:, 8:16] *= 0.01
    theta = mlp.pack(p).astype(np.float32)
    net = lc.Surrogate(theta)
    Xd, Yd = torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda()
    net.fit_scaler(Xd, Yd)
    sc = {k: np.asarray(v, np.float64) for k, v in net.params()[1].items()}
    return net, theta.astype(np.float64), X, Y, Xd, Yd, sc


def test_gradient_beyond_the_normal_sigmoids():
    """Tolerance: 1e-3 a block as in test_gpu_mlp.py, twice: an FP32 sum near -88 is off by up to 2e-5, which
    is the relative error of its activation and flips the BF16 rounding of 0.5 % of them by 2^-8, 2^-8
    sqrt(0.005) = 2.8e-4 of the activations' norm beside the other units' flips."""
    import torch
    net, theta, X, Y, Xd, Yd, sc = _extreme_net(17)
    rows = row_order(300, 96, 1, 18)
    g, loss = net.grad(Xd, Yd, torch.from_numpy(rows).cuda(), 96)
    g = g.cpu().numpy().astype(np.float64)
    Xs, Ts = mlp.standardize(X, Y, sc)
    lo, go = mlp.loss_and_grad(theta, Xs[rows], Ts[rows], bf16=True)
    plain = theta.copy()
    plain[320:4416].reshape(64, 64)[:, :8] = 0.0  # those units' part is well above the tolerance
    for a, b in BLOCKS[:1] + BLOCKS[4:5]:
        far = mlp.loss_and_grad(plain, Xs[rows], Ts[rows], bf16=True)[1][a:b]
        assert np.linalg.norm(far - go[a:b]) > 2e-2 * np.linalg.norm(go[a:b])
    assert float(loss.cpu()[0]) == pytest.approx(lo, rel=2e-3)
    for a, b in BLOCKS:
        assert np.linalg.norm(g[a:b] - go[a:b]) <= 2e-3 * np.linalg.norm(go[a:b]), (a, b)


def test_inference_beyond_the_normal_sigmoids():
    """As the gradient; standardized outputs within 2e-2 as in test_gpu_mlp.py."""
    import torch
    net, theta, X, _, _, _, sc = _extreme_net(17)
    want = mlp.infer(theta, X, sc, bf16=True)
    out = net.infer(torch.from_numpy(X).cuda()).cpu().numpy().astype(np.float64)
    plain = theta.copy()
    plain[320:4416].reshape(64, 64)[:, :8] = 0.0
    assert np.max(np.abs(mlp.infer(plain, X, sc, bf16=True) - want) / sc["y_sd"]) > 2 * 2e-2  # the oracle's own
    assert np.max(np.abs(out - want) / sc["y_sd"]) <= 2e-2


@pytest.mark.parametrize("centre,third,back", [(0.0, 2.0**-16, 2.0**-40), (-20.0, 0.0, 2.0**-10), (-55.0, 0.0, 1.0)])
def test_inference_activation_within_its_fp32_rounding(centre, third, back):
    """One hidden unit whose pre-activation is an exact FP32 sum, brought into the range where the next
    activation is half its argument: the output shows the BF16 activation itself.  Its FP32 value is
    within 2.2e-7 of the true one (an ulp each of the exponential and of the sum, half an ulp each of the
    reciprocal and of the product, at most 2^-24 of 3.7), so it may only be rounded the other way
    within that distance of the middle between two BF16 numbers."""
    import torch
    import paper_1307_3711_amd as lc
    p = mlp.unpack(np.zeros(mlp.N_PARAMS))
    p["W1"][0, :3] = 1.0, 2.0**-8, third
    p["b1"][0] = centre
    p["W2"][0, 0] = back
    p["W3"][0, 0] = 1.0
    net = lc.Surrogate(mlp.pack(p).astype(np.float32))
    rng = np.random.Generator(np.random.Philox(key=[5, 5]))
    X = (rng.integers(-127, 128, (400000, 4)) / 16.0).astype(np.float32)
    got = net.infer(torch.from_numpy(X).cuda()).cpu().numpy()[:, 0].astype(np.float64) * (2.0 / back)
    z = X.astype(np.float64) @ p["W1"][0] + centre
    assert np.array_equal(z, z.astype(np.float32))
    h = mlp.silu(z)
    lo, hi = mlp.to_bf16((h * (1.0 - 2.2e-7)).astype(np.float32)), mlp.to_bf16((h * (1.0 + 2.2e-7)).astype(np.float32))
    assert np.all((got == lo) | (got == hi))


def test_first_adam_step_bitwise_with_tiny_gradients():
    """Weights of zero whose gradients are 1e-39 to 1e-34: Adam's first step in FP32, operation by
    operation, bit for bit."""
    import torch
    import paper_1307_3711_amd as lc
    f = np.float32
    X, Y = toy_dataset(300, 4)
    p = mlp.unpack(init_params(4).astype(np.float64))
    p["W1"][:16] *= 0.02
    p["b1"][:16] = np.linspace(-85.0, -76.0, 16)
    p["W2"][:, :16] = 0.0
    theta = mlp.pack(p).astype(f)
    net = lc.Surrogate(theta)
    Xd, Yd = torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda()
    net.fit_scaler(Xd, Yd)
    rows = torch.from_numpy(row_order(300, 64, 1, 5)).cuda()
    g = net.grad(Xd, Yd, rows, 64)[0].cpu().numpy()
    net.train(Xd, Yd, rows, 64, 1, 1e-3)
    c1, c2 = f(1) - f(0.9), f(1) - f(0.999)
    m, v = c1 * g, c2 * g * g
    want = theta - f(1e-3) * (m / c1) / (np.sqrt(v / c2) + f(1e-8))
    tiny = np.zeros(mlp.N_PARAMS, bool)
    tiny[320:4416].reshape(64, 64)[:, :16] = True
    small = np.abs(g[tiny])
    assert np.sum((small > 0) & (small < 1e-37)) > 100
    assert np.array_equal(net.params()[0], want)
