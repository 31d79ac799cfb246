"""Materials whose critical stretch is one or more, up to an infinite fracture energy (no
bond ever breaks), with both readings of the break test and on every bond path."""
import dataclasses
import math

import numpy as np
import pytest

from paper_2506_05362_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("abs_stretch", [False, True])
@pytest.mark.parametrize("s0", [1.5, 3.0, math.inf])
def test_no_bond_breaks(oracle_lib, s0, abs_stretch):
    """Random displacements of 2% of a spacing: |s| stays far below s0.  The tolerance is that
    of the bond law's test: some 120 terms a node, each right to a few units in the last
    place, 1e-12 of the largest entry."""
    from paper_2506_05362_amd import pd
    wl = I.two_spheres(radius_cells=5, speed=1.0, gap=1.0)
    m = wl.materials[0]
    delta = wl.params.horizon_factor * wl.grain_h[0]
    energy = 9.0 * m.bulk_modulus * delta / 5.0 * s0 ** 2  # s0 = sqrt(5 G_c / (9 K delta))
    wl.materials = [dataclasses.replace(m, fracture_energy=energy)]
    wl.u0[:] = np.random.default_rng(3).normal(0.0, 0.02 * wl.grain_h[0], size=wl.u0.shape)
    ora = oracle_lib.Oracle(wl, flags=oracle_lib.CELL_LIST | (oracle_lib.ABS_STRETCH if abs_stretch else 0))
    want = ora.state()["a"]
    for launch in (dict(), dict(loop=pd.LOOP_PERSISTENT), dict(bond_path=pd.BONDS_TILES)):
        sim = pd.Sim(wl, flags=pd.FLAG_ABS_STRETCH if abs_stretch else 0)
        sim.set_launch(**launch)
        a = sim.get("accel")
        assert np.abs(a - want).max() <= 1e-12 * np.abs(want).max()
        sim.step(3)
        assert np.array_equal(sim.get("intact_count"), sim.get("initial_count"))
        assert np.isfinite(sim.get("displacement")).all()
        sim.close()
