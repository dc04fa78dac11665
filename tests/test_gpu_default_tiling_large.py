"""The FP64 tiling of large runs without one of their own: the splits and targets per lane chosen beside
and at 16,384 and 32,768 macroparticles a cluster, with splits limited by the handle, and the states
they give against an explicit one-sided tiling (tolerance as in test_gpu_default_tiling.py).
"""
import numpy as np
import pytest

from _helpers import gpu_available
from test_gpu_default_tiling import _run, _sim

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


# ions of each cluster (as many electrons), the handle's most splits; targets per lane and splits expected
@pytest.mark.parametrize("sizes,max_splits,R,S", [
    ([8191], 16, 1, 16), ([8192] * 3, 16, 1, 8), ([8191] * 3, 16, 1, 6), ([8192] * 3, 5, 1, 5),
    ([16383], 16, 1, 8), ([16384], 16, 4, 16), ([16384], 15, 1, 8), ([16384], 3, 1, 3)])
def test_fp64_tiling_of_large_clusters(sizes, max_splits, R, S):
    sim = _sim("fp64", sizes, ionize=False, max_splits=max_splits)
    sim.start()
    t = sim.tuning()
    assert (t["R"], t["WJ"], t["S"], t["newton3"]) == (R, 4, S, 0)
    sim.close()
    ref = _sim("fp64", sizes, ionize=False, max_splits=max_splits)
    ref.set_tuning(R=2, WJ=1)
    for a, b in zip(_run(ref, 4), _run(_sim("fp64", sizes, ionize=False, max_splits=max_splits), 4)):
        assert np.array_equal(a["Z"], b["Z"])
        for key in ("x", "u", "wl", "wc"):
            assert np.max(np.abs(a[key] - b[key])) <= 1e-11 * np.max(np.abs(a[key])), key
