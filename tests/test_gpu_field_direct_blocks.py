"""A default field call's direct kernel: sizes where Kahan sums change their blocks, and charges that are
equal in whole chunks of 2048 sources (left out of the pair terms), the targets' own chunks among them.

Oracle and tolerances as in test_gpu_field_default.py.
"""
import numpy as np
import pytest

import oracle

from _helpers import gpu_available
from test_gpu_field import EPS2, U32, _scales
from test_gpu_field_default import _check_default, _particles

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("phi", [False, True])
@pytest.mark.parametrize("n", [4095, 4097, 6144, 8191, 8193])
def test_kahan_blocks(n, phi):
    """16 waves up to 4096 charges, then 8 waves with 8 or 16 targets."""
    _check_default(n, "fp32_kahan", phi, n + 3)


@pytest.mark.parametrize("precision", ["fp64", "fp32_acc64", "fp32_kahan"])
@pytest.mark.parametrize("n,mixed", [(63, 0), (2050, 0), (4000, 0), (4000, 2048), (4000, 4000)])
def test_equal_charges_in_whole_chunks(n, mixed, precision):
    """The first `mixed` charges differ, the others are all 3."""
    import torch
    import paper_1307_3711_amd as lc
    x, q = _particles(n, 5)
    q = q.copy()
    q[mixed:] = 3.0
    u, xr, qr, eps2 = (64.0 * U32, x.astype(np.float32).astype(np.float64), q.astype(np.float32).astype(np.float64),
                       float(np.float32(EPS2))) if precision != "fp64" else (1e-12, x, q, EPS2)
    Eo, Po = oracle.coulomb_field(xr, qr, eps2)
    xyzq = torch.tensor(np.concatenate([x.T, q[None, :]], axis=0), dtype=torch.float64, device="cuda").contiguous()
    E, P = lc.field(xyzq, EPS2, precision=precision, want_phi=True)
    s1, s0 = _scales(xr, qr, eps2, np.arange(n))
    assert np.all(np.abs(E.cpu().numpy().T - Eo) <= u * s1[:, None] + 1e-300)
    assert np.all(np.abs(P.cpu().numpy() - Po) <= u * s0 + 1e-300)
