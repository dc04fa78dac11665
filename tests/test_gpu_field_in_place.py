"""Field calls whose results lie over their charges: the charges are read before a result is written,
so a default call gives what the one-sided tiling of the same fields gives into buffers of its own, bit
for bit.
"""
import ctypes

import numpy as np
import pytest

from _helpers import gpu_available
from test_gpu_field import EPS2
from test_gpu_field_default import _particles

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


# first double of E and of the potential in the 4 n doubles of charges, in units of n (None: elsewhere)
@pytest.mark.parametrize("at_E,at_phi", [(0, 3), (1, None), (None, 0), (0.5, None)])
@pytest.mark.parametrize("precision,n", [("fp64", 1000), ("fp32_acc64", 4099), ("fp32_kahan", 5001), ("fp64", 26881)])
@pytest.mark.parametrize("api", ["field", "static"])
def test_results_over_the_charges(api, precision, n, at_E, at_phi):
    """Sizes of the direct kernel, of the pairs and of their strips."""
    import torch
    import paper_1307_3711_amd as lc
    x, q = _particles(n, 9)
    xyzq = torch.tensor(np.concatenate([x.T, q[None, :]], axis=0), dtype=torch.float64, device="cuda").contiguous()
    E, phi = lc.field(xyzq, EPS2, precision=precision, tuning=lc.make_tuning(R=2 if precision == "fp64" else 4, WJ=1))
    own = torch.zeros(4 * n, dtype=torch.float64, device="cuda")
    flat = xyzq.clone().reshape(-1)
    got_E = own[:3 * n] if at_E is None else flat[int(at_E * n):int(at_E * n) + 3 * n]
    got_phi = own[3 * n:] if at_phi is None else flat[at_phi * n:(at_phi + 1) * n]
    L, prec = lc.lib(), ["fp64", "fp32_acc64", "fp32_kahan"].index(precision)
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    if api == "field":
        need = L.lc_field_workspace_bytes(prec, n, None)
        work = torch.empty(need, dtype=torch.uint8, device="cuda")
        code = L.lc_field(prec, n, ptr(flat), EPS2, ptr(got_E), ptr(got_phi), ptr(work), need, None, st)
    else:
        code = L.lc_field_static(prec, n, ptr(flat), EPS2, ptr(got_E), ptr(got_phi), None, st)
    assert code == lc.LC_OK
    assert torch.equal(got_E.reshape(3, n), E) and torch.equal(got_phi, phi)
