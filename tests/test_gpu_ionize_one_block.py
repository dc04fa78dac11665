"""Ionization check and spawns in one block per cluster (256 or 1024 threads) against the two launches
that larger clusters take: the same cluster alone and beside one of 1100 ions, bit for bit."""
import numpy as np
import pytest

from workloads import Cluster, Laser, initial_state
from workloads.species import SPECIES

from _helpers import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def _run(sizes, precision, ofi, collisional, room, n_steps):
    import paper_1307_3711_amd as lc
    cl = [Cluster(species="Ar", r0_nm=2.0, n_ion=n, capacity=room * n, z_init=1, z_max=8,
                  laser=Laser(intensity_wcm2=2e15, envelope="flat")) for n in sizes]
    cfg = lc.make_config(precision, ionize=True, ofi_field=ofi, collisional=collisional, dt=0.05, softening_nm=0.2,
                         t0=1.2, diag_every=2, max_records=8, seed=12)
    sim = lc.Simulation(cfg, [lc.make_cluster(SPECIES["Ar"], c.r0_nm, c.n_ion, c.capacity, c.laser.intensity_wcm2,
                                              envelope="flat", z_max=8, n_steps=n_steps) for c in cl])
    for k, c in enumerate(cl):
        st = initial_state(c, 12, k)
        sim.init_from_host(k, st["x_nm"], st["u"], st["Z"])
    sim.set_tuning(R=2, WJ=2, S=2)  # one tiling for both runs
    sim.start()
    sim.step(8)
    return sim


@pytest.mark.parametrize("precision,ofi,collisional", [("fp64", "laser_only", False), ("fp32_acc64", "laser_only", True),
                                                       ("fp64", "local", True)])
@pytest.mark.parametrize("n", [1, 63, 65, 256, 257, 1024])
def test_same_electrons_as_in_two_launches(n, precision, ofi, collisional):
    one = _run([n], precision, ofi, collisional, 9, 6)
    two = _run([n, 1100], precision, ofi, collisional, 9, 6)
    a, b = one.particles(0), two.particles(0)
    assert a["n"] == b["n"] and (n < 63 or a["n"] > 2 * n)
    for key in ("x", "u", "Z", "wl", "wc"):
        assert np.array_equal(a[key], b[key]), key
    assert np.array_equal(one.diagnostics(0), two.diagnostics(0))
    one.close()
    two.close()


def test_same_count_past_the_capacity():
    one, two = (_run(s, "fp64", "laser_only", False, 2, 0) for s in ([500], [500, 1100]))
    a, b = one.counters(0), two.counters(0)
    assert a == b and a["n"] == 1000
    one.close()
    two.close()
