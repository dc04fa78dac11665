"""A default field call beside 4096 charges, up to which the direct kernel takes it and beyond which each
pair is taken once (oracle and tolerances as in test_gpu_field_default.py).
"""
import pytest

from _helpers import gpu_available
from test_gpu_field_default import _check_default

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("precision", ["fp64", "fp32_acc64", "fp32_kahan"])
@pytest.mark.parametrize("n,phi", [(4095, True), (4095, False), (4096, True), (4097, False), (4098, True), (4098, False)])
def test_border_of_the_pairs(n, phi, precision):
    _check_default(n, precision, phi, n + 5)
