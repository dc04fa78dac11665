"""Workspace of a default call of the standalone field (host side only)."""
import ctypes

import pytest

import paper_1307_3711_amd as lc


@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("n", [0, 1, 3583, 3584, 20000, 23041, 200000, 900000, 1 << 20, 1 << 24])
def test_stays_within_the_static_one(precision, n):
    """Wherever one split's workspace fits lc_field_static's array, so does a default call's."""
    L = lc.lib()
    one = lc.make_tuning(S=1)
    least = L.lc_field_workspace_bytes(precision, n, ctypes.byref(one))
    need = L.lc_field_workspace_bytes(precision, n, None)
    assert least <= need <= max(least, lc.LC_FIELD_STATIC_MAX_BYTES)
    assert precision != 2 or need == least   # Kahan sums keep no rows
