"""Inference called on several streams: each result is that of its own rows, also where its memory goes
back to the caller's stream at once and is taken again there.
"""
import numpy as np
import pytest

from workloads.surrogate import init_params, toy_dataset

from _helpers import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("n", [1, 4097, 200000])
def test_results_of_alternating_streams(n):
    import torch
    import paper_1307_3711_amd as lc
    X, Y = toy_dataset(512, 3)
    net = lc.Surrogate(init_params(3))
    net.fit_scaler(torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda())
    base = torch.from_numpy(toy_dataset(n, 4)[0]).cuda()
    rows = [base + 0.01 * k for k in range(4)]
    want = []
    for x in rows:
        want.append(net.infer(x).cpu())
    torch.cuda.synchronize()
    streams = [torch.cuda.current_stream()] + [torch.cuda.Stream() for _ in range(2)]
    got = []
    for i in range(24):
        with torch.cuda.stream(streams[i % 3]):
            y = net.infer(rows[i % 4])
            keep = y.clone()
            del y  # its block is free again on this stream
            torch.full((n, 2), np.nan, device="cuda")
            got.append(keep)
    torch.cuda.synchronize()
    for i, y in enumerate(got):
        assert torch.equal(y.cpu(), want[i % 4]), i
