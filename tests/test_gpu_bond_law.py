"""The bond law across its three forms (series of degree 6 and 8, exact) on every bond
path, with one material and with two, against the oracle."""
import dataclasses

import numpy as np
import pytest

from paper_2506_05362_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("amp", [1e-4, 1.5e-3, 6e-3, 3e-2])  # |x| of the stiffest bonds: about 3 amp to 10 amp
@pytest.mark.parametrize("two", [False, True])
def test_bond_law_forms(oracle_lib, amp, two):
    """Random displacements of amp spacings put bonds on both sides of |x| = 0.0055 and 0.02.
    A node sums some 120 terms, each right to a few units in the last place, against a
    field whose largest entry is of the size of a few terms: 1e-12 of it bounds the
    difference (120 x 10 ulp = 2.7e-13).  The paths agree bitwise."""
    from paper_2506_05362_amd import pd
    wl = I.two_spheres(radius_cells=5, speed=1.0, gap=1.0)
    # (new objects: the workload's own are shared defaults); nothing breaks
    wl.materials = [dataclasses.replace(m, fracture_energy=1e8 * m.fracture_energy) for m in wl.materials]
    if two:
        m = wl.materials[0]
        wl.materials.append(I.Material(0.4 * m.bulk_modulus, 1.3 * m.density, m.fracture_energy))
        wl.grain_material[1] = len(wl.materials) - 1
    wl.u0[:] = np.random.default_rng(5).normal(0.0, amp * wl.grain_h[0], size=wl.u0.shape)
    ora = oracle_lib.Oracle(wl, flags=oracle_lib.CELL_LIST)
    sims = [pd.Sim(wl) for _ in range(3)]
    sims[1].set_launch(loop=pd.LOOP_PERSISTENT)
    sims[2].set_launch(bond_path=pd.BONDS_TILES)
    a, o = sims[0].get("accel"), ora.state()["a"]
    assert np.abs(a - o).max() <= 1e-12 * np.abs(o).max()
    for sim in sims:
        sim.step(3)
    for f in ("displacement", "velocity", "accel"):
        want = sims[0].get(f)
        assert np.isfinite(want).all()
        for sim in sims[1:]:
            assert np.array_equal(sim.get(f), want), f
