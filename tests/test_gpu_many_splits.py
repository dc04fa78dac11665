"""Sums over the splits of a one-sided pass, whose loads go out 4, 8 or 16 at a time (push and
diagnostics): every number of splits around those against a single split.

Tolerance: splits regroup a target's FP64 sum, at most N rounding errors of 2^-53 relative to its
absolute terms (1e-13 for 600 sources), and 12 steps of 0.05 let a difference grow by well below 1e3:
1e-9 of R0 in position, of the largest momentum and of the energies' scale.
"""
import numpy as np
import pytest

from workloads import Cluster, Laser, initial_state
from workloads.species import SPECIES

from _helpers import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def _run(S):
    import paper_1307_3711_amd as lc
    c = Cluster(species="D", r0_nm=3.0, n_ion=301, capacity=602, z_init=1, z_max=1,
                laser=Laser(intensity_wcm2=5e15, envelope="flat"))
    cfg = lc.make_config("fp64", ionize=False, dt=0.05, softening_nm=0.2, t0=1.2, diag_every=4, max_records=8,
                         max_splits=20, seed=5)
    sim = lc.Simulation(cfg, [lc.make_cluster(SPECIES["D"], c.r0_nm, c.n_ion, c.capacity, c.laser.intensity_wcm2,
                                              envelope="flat", z_max=1)])
    st = initial_state(c, 5, 0)
    sim.init_from_host(0, st["x_nm"], st["u"], st["Z"])
    sim.set_tuning(R=1, WJ=4, S=S)
    sim.start()
    sim.step(12)
    p, d = sim.particles(0), np.array(sim.diagnostics(0))
    sim.close()
    return p, d


@pytest.mark.parametrize("S", [2, 4, 5, 7, 8, 9, 15, 16, 17, 20])
def test_against_one_split(S):
    (a, da), (b, db) = _run(1), _run(S)
    for key in ("x", "u", "wl", "wc"):
        assert np.max(np.abs(a[key] - b[key])) <= 1e-9 * np.max(np.abs(a[key])), key
    assert da.shape == db.shape and np.all(np.isfinite(db))
    assert np.max(np.abs(da - db)) <= 1e-9 * np.max(np.abs(da))
