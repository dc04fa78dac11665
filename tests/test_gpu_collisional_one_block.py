"""Collisional rates formed by the ionizing block (from its own sums, or from the partial sums of a
launch before it) against the rates of k_ci_final, which runs past 2048 blocks of ions: cluster 0 alone,
beside a larger cluster and beside 2050 small ones, bit for bit."""
import numpy as np
import pytest

from test_gpu_ionize_one_block import _run

from _helpers import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("precision,ofi", [("fp64", "local"), ("fp32_acc64", "laser_only")])
@pytest.mark.parametrize("n", [1, 65, 256, 700])
def test_rates_from_every_route(n, precision, ofi):
    runs = [_run(s, precision, ofi, True, 9, 6) for s in ([n], [n, 700], [n, 1100], [n, 1100] + [4] * 2050)]
    first, first_diag = runs[0].particles(0), runs[0].diagnostics(0)
    for r in runs[1:]:
        p = r.particles(0)
        for key in ("x", "u", "Z", "wl", "wc"):
            assert np.array_equal(first[key], p[key]), key
        assert np.array_equal(first_diag, r.diagnostics(0))
    for r in runs:
        r.close()
