"""Collisional ionization over electron temperatures from far below to far above the ionization
potentials: the rate's exponential integral on both of its branches and beside their border.  The
same Philox numbers and FP64 decisions on both sides, so the same charges as the oracle's."""
import numpy as np
import pytest

import oracle
from oracle import units
from workloads import Cluster, Laser, Run, initial_state

from _helpers import gpu_available, gpu_run

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("kinetic_ev", [1.0, 8.0, 23.6, 24.0, 41.0, 120.0, 1000.0, 30000.0])
def test_same_charges_as_the_oracle(kinetic_ev):
    """T = 2/3 of the mean kinetic energy: 23.6 and 24 eV put P / T of Ar+ (15.76 eV, then 27.6) at
    and beside 1."""
    c = Cluster(species="Ar", r0_nm=2.0, n_ion=700, capacity=6300, z_init=1, z_max=8,
                laser=Laser(intensity_wcm2=1e14, envelope="flat"))
    run = Run(dt=0.05, ionize=True, collisional=True, diag_every=2, seed=6)
    st = initial_state(c, run.seed)
    v = np.random.default_rng(3).normal(size=(c.n_ion, 3))
    g = 1.0 + kinetic_ev / units.MEC2_EV
    st["u"] = st["u"].copy()
    st["u"][c.n_ion:] = v * (np.sqrt(g * g - 1.0) / np.linalg.norm(v, axis=1))[:, None]
    sim, _ = gpu_run([c], run, "fp64", states=[st])
    ref = oracle.Sim.from_workload(c, run, st)
    ref.start()
    ref.run(6)
    sim.step(6)
    p = sim.particles(0)
    assert p["n"] == ref.N and np.array_equal(p["Z"], ref.charges())
    if kinetic_ev >= 24.0:
        assert ref.counters[1] > 0
    sim.close()
