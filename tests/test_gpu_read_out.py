"""Read-out of particles and records in pieces (4096 particles or 693 records a piece): sizes at and
beside the pieces' ends, fewer rows than there are, and missing arrays.  The values are those put
in (positions: the same product with the unit conversion), and records those read one by one."""
import ctypes

import numpy as np
import pytest

from workloads.species import SPECIES

from _helpers import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def _sim(sizes, **cfg):
    import paper_1307_3711_amd as lc
    c = lc.make_config("fp32_acc64", ionize=False, dt=0.02, softening_nm=0.3, seed=2, max_splits=2,
                       **{"diag_every": 0, "max_records": 1, **cfg})
    return lc.Simulation(c, [lc.make_cluster(SPECIES["Ar"], 3.0, n, n + 5, 1e14, envelope="flat", z_max=4)
                             for n in sizes])


@pytest.mark.parametrize("sizes", [[1, 4095], [4096, 3], [4097], [8193, 64, 8192]])
def test_particles_come_back_as_they_went_in(sizes):
    import paper_1307_3711_amd as lc
    sim = _sim(sizes)
    rng = np.random.default_rng(5)
    k = lc.units(0.8)["k_per_nm"]
    for c, n in enumerate(sizes):
        x, u = rng.normal(size=(n, 3)), rng.normal(size=(n, 3))
        Z = rng.integers(0, 5, n).astype(np.int8)
        sim.init_from_host(c, x, u, Z)
        p = sim.particles(c)
        assert p["n"] == n and np.array_equal(p["u"], u) and np.array_equal(p["Z"], Z)
        assert np.allclose(p["x"], x * k, rtol=4e-16, atol=0)
        assert not p["wl"].any() and not p["wc"].any()
        # two arrays of four fewer rows; rows past them stay as they are
        m = max(n - 4, 0)
        u2, z2, got = np.full((n, 3), 9.0), np.full(n, 9, np.int8), ctypes.c_int64()
        dp = ctypes.POINTER(ctypes.c_double)
        assert lc.lib().lc_read_particles(sim.h, c, None, u2.ctypes.data_as(dp),
                                          z2.ctypes.data_as(ctypes.POINTER(ctypes.c_int8)), None, None, m,
                                          ctypes.byref(got)) == lc.LC_OK
        assert got.value == n
        assert np.array_equal(u2[:m], u[:m]) and np.all(u2[m:] == 9.0)
        assert np.array_equal(z2[:m], Z[:m]) and np.all(z2[m:] == 9)
    sim.close()


def test_records_in_pieces_and_past_the_ring():
    steps, ring = 760, 700
    one, many = _sim([6, 9], diag_every=1, max_records=ring), _sim([6, 9], diag_every=1, max_records=ring)
    each = [[], []]
    for sim in (one, many):
        sim.init_generate(-1, 0)
        sim.start()
    for _ in range(steps):
        one.step(1)
        for c in range(2):
            r = one.diagnostics(c, 1)
            assert r.shape == (1, 48)
            each[c].append(r[0])
    many.step(steps)
    for c in range(2):
        want = np.array(each[c])
        assert np.array_equal(want[:, 1], np.arange(steps))
        for ask in (1, 693, 694, ring, ring + 50):
            assert np.array_equal(many.diagnostics(c, ask), want[-min(ask, ring):])
    one.close()
    many.close()
