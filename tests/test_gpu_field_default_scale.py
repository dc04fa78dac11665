"""A default field call that takes each pair once, at any length scale: lengths and softening scaled by
powers of ten leave the relative rounding of every pair term alone (tolerances as in
test_gpu_field_default.py, twice over for a difference of two results).
"""
import numpy as np
import pytest

from _helpers import gpu_available
from test_gpu_field import EPS2, _scales
from test_gpu_field_default import _particles

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def _field(x, q, f, phi):
    import torch
    import paper_1307_3711_amd as lc
    xyzq = torch.tensor(np.concatenate([f * x.T, q[None, :]], axis=0), dtype=torch.float64, device="cuda").contiguous()
    E, P = lc.field(xyzq, EPS2 * f * f, precision="fp64", want_phi=phi)
    return (E.cpu().numpy() * f) * f, P.cpu().numpy() * f if phi else None


@pytest.mark.parametrize("scale", [1e-60, 1e-20, 1e20, 1e90])
@pytest.mark.parametrize("n,phi", [(4097, False), (4099, True), (5000, True)])
def test_field_and_potential(n, phi, scale):
    x, q = _particles(n, 3)
    at = np.arange(0, n, 41)
    s1, s0 = _scales(x, q, EPS2, at)
    (E, P), (Es, Ps) = _field(x, q, 1.0, phi), _field(x, q, scale, phi)
    assert np.all(np.abs(Es - E).T[at] <= 2e-12 * s1[:, None])
    if phi:
        assert np.all(np.abs(Ps - P)[at] <= 2e-12 * s0)


@pytest.mark.parametrize("n", [4097, 4100, 4351, 4352])
def test_potential_where_the_field_underflows(n):
    """Lengths of 1e142: a last wave of 1, 4, 63 or 64 equal charges; the places past them add nothing."""
    x, q = _particles(n, 3)
    at = np.arange(0, n, 41)
    _, s0 = _scales(x, q, EPS2, at)
    (_, P), (_, Ps) = _field(x, q, 1.0, True), _field(x, q, 1e144, True)
    assert np.all(np.abs(Ps - P)[at] <= 2e-12 * s0)
