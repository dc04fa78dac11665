"""Runs without a tiling of their own: the one chosen from the particle counts against the tiling
whose fields were the defaults alone.

FP32 pair terms: the same sums in the same order, so every particle and record bit for bit.  FP64:
other splits of the same sums, a difference of FP64 rounding (1e-15 of a sum's terms) that a few
steps do not grow past 1e-11 of the largest value.
"""
import os
import tempfile

import numpy as np
import pytest

from workloads import Cluster, Laser, initial_state
from workloads.species import SPECIES

from _helpers import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def _sim(precision, sizes, boundary="open", ionize=True, max_splits=16):
    import paper_1307_3711_amd as lc
    cl = [Cluster(species="Ar", r0_nm=2.0 + 0.2 * k, n_ion=n, capacity=3 * n + 1, z_init=1,
                  laser=Laser(intensity_wcm2=2e15, envelope="flat")) for k, n in enumerate(sizes)]
    cfg = lc.make_config(precision, ionize=ionize, dt=0.02, softening_nm=0.3, t0=1.0, diag_every=3, max_records=8,
                         seed=4, max_splits=max_splits, boundary=boundary, t_switch=1.07)
    sim = lc.Simulation(cfg, [lc.make_cluster(SPECIES["Ar"], c.r0_nm, c.n_ion, c.capacity, c.laser.intensity_wcm2,
                                              envelope="flat", z_max=2) for c in cl])
    for k, c in enumerate(cl):
        st = initial_state(c, 4, k)
        sim.init_from_host(k, st["x_nm"], st["u"], st["Z"])
    return sim


def _run(sim, steps=7):
    sim.start()
    sim.set_graph(3)
    sim.step(steps)
    out = [dict(sim.particles(k), rec=sim.diagnostics(k)) for k in range(sim.n_clusters)]
    sim.close()
    return out


@pytest.mark.parametrize("precision,boundary", [("fp32_acc64", "open"), ("fp32_kahan", "open"),
                                                ("fp32_acc64", "periodic"), ("fp32_acc64", "mixed")])
@pytest.mark.parametrize("sizes,ionize,max_splits", [([1], True, 16), ([31, 700], True, 16), ([1600], False, 64),
                                                     ([20, 33, 129, 515], True, 3)])
def test_fp32_same_bits_as_the_default_fields(precision, boundary, sizes, ionize, max_splits):
    ref = _sim(precision, sizes, boundary, ionize, max_splits)
    ref.set_tuning(R=4, WJ=1)
    got = _run(_sim(precision, sizes, boundary, ionize, max_splits))
    for a, b in zip(_run(ref), got):
        for key in ("x", "u", "Z", "wl", "wc", "rec"):
            assert np.array_equal(a[key], b[key]), key


@pytest.mark.parametrize("boundary", ["open", "periodic"])
@pytest.mark.parametrize("sizes,max_splits", [([1], 16), ([40, 500], 16), ([1700], 16), ([300], 2)])
def test_fp64_within_rounding_of_the_default_fields(sizes, max_splits, boundary):
    ref = _sim("fp64", sizes, boundary, max_splits=max_splits)
    ref.set_tuning(R=2, WJ=1)
    got = _run(_sim("fp64", sizes, boundary, max_splits=max_splits))
    for a, b in zip(_run(ref), got):
        assert np.array_equal(a["Z"], b["Z"])
        for key in ("x", "u", "wl", "wc"):
            assert np.max(np.abs(a[key] - b[key])) <= 1e-11 * np.max(np.abs(a[key]))


@pytest.mark.parametrize("precision", ["fp64", "fp32_acc64"])
def test_saved_run_goes_on_the_same(precision):
    """A checkpoint keeps the tiling that the run began with: charges change in between."""
    whole = _sim(precision, [60, 400])
    want = _run(whole, 12)
    half = _sim(precision, [60, 400])
    half.start()
    half.step(6)
    with tempfile.TemporaryDirectory() as d:
        path = os.path.join(d, "chk")
        half.save(path)
        half.close()
        rest = _sim(precision, [60, 400])
        rest.load(path)
    rest.step(6)
    for k, a in enumerate(want):
        p = rest.particles(k)
        for key in ("x", "u", "Z", "wl", "wc"):
            assert np.array_equal(a[key], p[key])
    rest.close()
