"""Default field calls that cannot take each pair once, for want of rows in a strip or of workspace: the
one-sided kernel takes those whose blocks fill their last round, with the bits of its explicit tiling,
the direct kernel the others, within the tolerances of test_gpu_field.py of it (twice over).
"""
import ctypes

import numpy as np
import pytest

from _helpers import gpu_available
from test_gpu_field import EPS2, U32, _scales
from test_gpu_field_default import _particles

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("n,precision,phi,small,same", [
    (524288, "fp32_acc64", True, True, True), (499501, "fp32_acc64", False, True, True),
    (499000, "fp32_acc64", False, True, False), (262144, "fp32_acc64", False, True, False),
    (476626, "fp64", False, True, True), (476000, "fp64", True, True, False),
    (393216, "fp64", False, True, False), (1048577, "fp64", False, False, True)])
def test_kernel_of_a_large_call(n, precision, phi, small, same):
    import torch
    import paper_1307_3711_amd as lc
    L, prec = lc.lib(), ["fp64", "fp32_acc64"].index(precision)
    x, q = _particles(n, 2, r0=2.5 * (n / 2000.0) ** (1.0 / 3.0))
    xyzq = torch.tensor(np.concatenate([x.T, q[None, :]], axis=0), dtype=torch.float64, device="cuda").contiguous()
    t = lc.make_tuning(S=1)
    E, P = lc.field(xyzq, EPS2, precision=precision, want_phi=phi, tuning=t)
    need = L.lc_field_workspace_bytes(prec, n, ctypes.byref(t) if small else None)
    work = torch.empty(need, dtype=torch.uint8, device="cuda")
    got = torch.empty((4, n), dtype=torch.float64, device="cuda")
    ptr = lambda a: ctypes.c_void_p(a.data_ptr())
    assert L.lc_field(prec, n, ptr(xyzq), EPS2, ptr(got), ptr(got[3]) if phi else None, ptr(work), need, None,
                      ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == lc.LC_OK
    equal = torch.equal(got[:3], E) and (not phi or torch.equal(got[3], P))
    assert equal == same
    at = np.linspace(0, n - 1, 20).astype(np.int64)
    s1, s0 = _scales(x, q, EPS2, at)
    u = 1e-12 if precision == "fp64" else 64.0 * U32
    assert np.all(np.abs((got[:3] - E).cpu().numpy().T[at]) <= 2.0 * u * s1[:, None])
    if phi:
        assert np.all(np.abs((got[3] - P).cpu().numpy()[at]) <= 2.0 * u * s0)
