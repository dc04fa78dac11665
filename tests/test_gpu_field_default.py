"""A default call of the standalone field (no tiling given): each of its kernels against the FP64
oracle at the sizes where the division of the work changes.

Tolerances as in test_gpu_field.py: |dE| <= u S1 and |dphi| <= u S0 per target, u = 1e-12 in FP64 and
64 2^-24 against the oracle on the FP32-rounded inputs for the FP32 pair terms.
"""
import numpy as np
import pytest

import oracle

from _helpers import gpu_available
from test_gpu_field import EPS2, U32, _scales, _state

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def _particles(n, seed, r0=2.5):
    x, q = _state(n + 1, seed, r0)   # whole ion-electron pairs
    assert x.shape[0] >= n
    return x[:n], q[:n]


def _check_default(n, precision, phi, seed):
    """A default call of n charges against the oracle at a hundred targets (the first and last
    hundred's ends among them), with the elementwise tolerances above, and lc_field_static with it."""
    import torch
    import paper_1307_3711_amd as lc
    x, q = _particles(n, seed, r0=2.5 * (n / 2000.0) ** (1.0 / 3.0))
    u, xr, qr, eps2 = (64.0 * U32, x.astype(np.float32).astype(np.float64), q.astype(np.float32).astype(np.float64),
                       float(np.float32(EPS2))) if precision != "fp64" else (1e-12, x, q, EPS2)
    Eo, Po = oracle.coulomb_field(xr, qr, eps2)
    xyzq = torch.tensor(np.concatenate([x.T, q[None, :]], axis=0), dtype=torch.float64, device="cuda").contiguous()
    E, P = lc.field(xyzq, EPS2, precision=precision, want_phi=phi)
    Es, Ps = lc.field_static(xyzq, EPS2, precision=precision, want_phi=phi)
    assert torch.equal(E, Es) and (not phi or torch.equal(P, Ps))
    idx = np.unique(np.concatenate([[0, n - 1], np.random.default_rng(seed).integers(0, n, 98)]))
    s1, s0 = _scales(xr, qr, eps2, idx)
    assert np.all(np.isfinite(E.cpu().numpy()))
    assert np.all(np.abs(E.cpu().numpy().T[idx] - Eo[idx]) <= u * s1[:, None] + 1e-300)
    if phi:
        assert np.all(np.abs(P.cpu().numpy()[idx] - Po[idx]) <= u * s0 + 1e-300)


@pytest.mark.parametrize("precision", ["fp64", "fp32_acc64", "fp32_kahan"])
@pytest.mark.parametrize("n,phi", [(15, True), (17, False), (2047, True), (2049, True), (3583, True), (3584, True),
                                   (3585, False), (4096, False), (4097, True)])
def test_default_field_where_its_kernels_change(n, phi, precision):
    """Blocks of 16 targets and chunks of 2048 sources below 3584 charges, blocks of 256 taken in
    pairs from there on: sizes at and beside their edges."""
    _check_default(n, precision, phi, n + 5)


@pytest.mark.parametrize("n,precision,phi", [(23041, "fp64", True), (26881, "fp64", False), (32769, "fp32_acc64", True)])
def test_default_field_in_strips(n, precision, phi):
    """Row sums of more block pairs than a strip holds: at least two strips each."""
    _check_default(n, precision, phi, 7)


@pytest.mark.parametrize("precision", [0, 1])
def test_default_field_in_the_one_sided_workspace(precision):
    """A workspace of one split's size (source records and four FP64 sums a charge) stays enough at
    any size: the one-sided kernel takes the call."""
    import ctypes
    import torch
    import paper_1307_3711_amd as lc
    n = 4097
    x, q = _particles(n, 12)
    xyzq = torch.tensor(np.concatenate([x.T, q[None, :]], axis=0), dtype=torch.float64, device="cuda").contiguous()
    t = lc.make_tuning(S=1)
    need = lc.lib().lc_field_workspace_bytes(precision, n, ctypes.byref(t))
    assert lc.lib().lc_field_workspace_bytes(precision, n, None) > need
    work = torch.empty(need, dtype=torch.uint8, device="cuda")
    E = torch.empty((3, n), dtype=torch.float64, device="cuda")

    def call(bytes_):
        return lc.lib().lc_field(precision, n, ctypes.c_void_p(xyzq.data_ptr()), EPS2, ctypes.c_void_p(E.data_ptr()),
                                 None, ctypes.c_void_p(work.data_ptr()), bytes_, None,
                                 ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))

    assert call(need - 256) == lc.LC_E_INVALID
    assert call(need) == lc.LC_OK
    E2, _ = lc.field(xyzq, EPS2, precision=precision, want_phi=False)
    idx = np.arange(0, n, 41)
    s1, _ = _scales(x, q, EPS2, idx)
    u = 1e-12 if precision == 0 else 64.0 * U32
    assert np.all(np.abs((E - E2).cpu().numpy().T[idx]) <= 2.0 * u * s1[:, None])


@pytest.mark.parametrize("scale", [1e-60, 1e-20, 1e20, 1e90])
@pytest.mark.parametrize("n,tuning", [(300, None), (3600, None), (300, dict(R=4, WJ=4, newton3=1)), (300, dict(R=2, S=2))])
def test_fp64_field_at_any_length_scale(n, tuning, scale):
    """E scales as q / length^2: lengths and softening scaled by powers of ten leave the relative
    rounding of every pair term alone."""
    import torch
    import paper_1307_3711_amd as lc
    x, q = _particles(n, 3)
    s1, _ = _scales(x, q, EPS2, np.arange(0, n, 29))
    out = []
    for f in (1.0, scale):
        xyzq = torch.tensor(np.concatenate([f * x.T, q[None, :]], axis=0), dtype=torch.float64, device="cuda").contiguous()
        t = lc.make_tuning(**tuning) if tuning else None
        E, _ = lc.field(xyzq, EPS2 * f * f, precision="fp64", want_phi=False, tuning=t)
        out.append((E.cpu().numpy() * f) * f)
    assert np.all(np.abs(out[1] - out[0]).T[::29] <= 2e-12 * s1[:, None])
