"""A tile finds its cluster among the starts of all clusters, 64 at a time: ensembles of sizes at and
beside a wave's width and the square of it, with clusters that retire (and leave no tiles), against
each sampled cluster run by itself, bit for bit."""
import numpy as np
import pytest

from workloads.species import SPECIES

from _helpers import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def _cluster(c):
    rng = np.random.default_rng(c)
    n = 1 + c % 3
    x = rng.normal(size=(2 * n, 3))
    return n, x, rng.normal(size=(2 * n, 3)) * 1e-3, np.array([1] * n + [-1] * n, np.int8), 1 if c % 5 == 2 else 0


def _run(ids, tiling, steps=3):
    import paper_1307_3711_amd as lc
    cfg = lc.make_config("fp64", ionize=False, dt=0.02, softening_nm=0.2, t0=1.0, diag_every=0, max_records=1, seed=1,
                         max_splits=2, max_pair_blocks=1)
    descs = []
    for c in ids:
        n, _, _, _, retire = _cluster(c)
        descs.append(lc.make_cluster(SPECIES["Ar"], 1.0, n, 2 * n, 1e15, envelope="flat", z_max=2, n_steps=retire))
    sim = lc.Simulation(cfg, descs)
    for k, c in enumerate(ids):
        _, x, u, Z, _ = _cluster(c)
        sim.init_from_host(k, x, u, Z)
    sim.set_tuning(**tiling)
    sim.start()
    sim.step(steps)
    return sim


@pytest.mark.parametrize("tiling", [dict(R=1, WJ=4, S=2), dict(R=4, WJ=4, newton3=1)])
@pytest.mark.parametrize("count", [2, 63, 64, 65, 129, 4096, 4097, 4161])
def test_every_tile_finds_its_cluster(count, tiling):
    sim = _run(range(count), tiling)
    for c in sorted({0, 1, 2, count // 2, 62, 63, 64, 65, 127, 128, 4095, 4096, count - 2, count - 1}):
        if not 0 <= c < count:
            continue
        one, p = _run([c], tiling), sim.particles(c)
        q = one.particles(0)
        one.close()
        for key in ("x", "u", "wl", "wc"):
            assert np.array_equal(p[key], q[key]), (c, key)
    sim.close()
