"""The surrogate's kernels at the sizes where their work division changes.

Tolerances: gradients and inference as in test_gpu_mlp.py (FP32 against FP64 sums and the BF16
rounding flips they cause); steps split over calls, bit for bit.
"""
import numpy as np
import pytest

from oracle import mlp
from workloads.surrogate import init_params, row_order, toy_dataset

from _helpers import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

BLOCKS = [(0, 256), (256, 320), (320, 4416), (4416, 4480), (4480, 4608), (4608, 4610)]


def _net(n, seed, steps=0, batch=32):
    import torch
    import paper_1307_3711_amd as lc
    X, Y = toy_dataset(n, seed)
    theta = init_params(seed)
    net = lc.Surrogate(theta)
    Xd, Yd = torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda()
    net.fit_scaler(Xd, Yd)
    rows = torch.from_numpy(row_order(n, batch, max(steps, 1), seed + 1)).cuda()
    sc = {k: np.asarray(v, np.float64) for k, v in net.params()[1].items()}
    return net, theta.astype(np.float64), X, Y, Xd, Yd, rows, sc


@pytest.mark.parametrize("batch", [64, 160, 224])
def test_gradient_where_some_waves_hold_no_rows(batch):
    """Two to fourteen of the sixteen waves hold rows; every wave takes a tile of dW2."""
    net, theta, X, Y, Xd, Yd, rows, sc = _net(300, 21, 1, batch)
    g, loss = net.grad(Xd, Yd, rows, batch)
    g = g.cpu().numpy().astype(np.float64)
    Xs, Ts = mlp.standardize(X, Y, sc)
    r = rows.cpu().numpy()
    lo, go = mlp.loss_and_grad(theta, Xs[r], Ts[r], bf16=True)
    assert float(loss.cpu()[0]) == pytest.approx(lo, rel=1e-4)
    for a, b in BLOCKS:
        assert np.linalg.norm(g[a:b] - go[a:b]) <= 1e-3 * np.linalg.norm(go[a:b])


@pytest.mark.parametrize("batch,split", [(32, 64), (96, 65), (256, 1)])
def test_steps_split_over_calls_bitwise(batch, split):
    """Factors of Adam's step count come 64 steps at a time: a run of 130 steps against the same
    steps in two calls, cut at and beside that length."""
    out = []
    for cuts in ([130], [split, 130 - split]):
        net, _, _, _, Xd, Yd, rows, _ = _net(700, 5, 130, batch)
        at, loss = 0, []
        for k in cuts:
            loss.append(net.train(Xd, Yd, rows[at * batch:], batch, k, 1e-3).cpu().numpy())
            at += k
        out.append((net.params()[0], np.concatenate(loss)))
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
    assert np.all(np.isfinite(out[0][0])) and not np.array_equal(out[0][0], init_params(5))


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 65, 4096, 65536, 65537, 131111])
def test_inference_at_tile_edges(n):
    """16 rows a tile, 64 a block; from 65,536 rows on a wave takes more than one tile."""
    import torch
    net, theta, _, _, _, _, _, sc = _net(512, 31)
    X, _ = toy_dataset(n, 77)
    out = net.infer(torch.from_numpy(X).cuda())
    assert out.shape == (n, 2)
    d = np.abs(out.cpu().numpy().astype(np.float64) - mlp.infer(theta, X, sc, bf16=True)) / sc["y_sd"]
    assert d.max() <= 2e-2 and np.quantile(d, 0.99) <= 1e-4


def test_inference_keeps_nonfinite_rows_apart():
    """A row with an infinity or NaN gives no finite answer and leaves its tile's other rows alone."""
    import torch
    net, theta, _, _, _, _, _, sc = _net(512, 31)
    X, _ = toy_dataset(40, 78)
    ref = net.infer(torch.from_numpy(X).cuda()).cpu().numpy()
    for row, value in ((3, np.nan), (17, np.inf), (33, -np.inf)):
        bad = X.copy()
        bad[row, 1] = value
        out = net.infer(torch.from_numpy(bad).cuda()).cpu().numpy()
        keep = np.arange(40) != row
        assert np.array_equal(out[keep], ref[keep]) and not np.isfinite(out[row]).any()


@pytest.mark.parametrize("n", [1, 2, 255, 257, 1023, 2049, 4096, 16387])
def test_scaler_sizes_and_constant_column(n):
    """Fewer elements than threads, whole and ragged rounds of loads; a constant column has
    deviation 1.  FP64 sums of FP32 values: the FP32 result is within an ulp of numpy's."""
    import torch
    import paper_1307_3711_amd as lc
    X, Y = toy_dataset(n, 91)
    X[:, 2] = 3.25
    net = lc.Surrogate(init_params(1))
    net.fit_scaler(torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda())
    _, sc = net.params()
    for a, mu, sd in ((X, sc["x_mu"], sc["x_sd"]), (Y, sc["y_mu"], sc["y_sd"])):
        a = a.astype(np.float64)
        want = a.std(axis=0)
        assert np.allclose(mu, a.mean(axis=0), rtol=1.2e-7, atol=1e-30)
        assert np.allclose(sd, np.where(want > 0, want, 1.0), rtol=1.2e-7, atol=0)
