"""Lined rows as the bond memory of the steps that read them: breaks, the bond law's forms and
self-contact's look-ups in slices of two materials, with both readings of the break test,
bitwise against the persistent loop, which steps over the compact rows."""
import dataclasses

import numpy as np
import pytest

from paper_2506_05362_amd import inputs as I
from test_gpu_device_memory import Recorder

pytestmark = pytest.mark.gpu
# (energies first: the first field that brings the column words up to date)
FIELDS = ("energy", "displacement", "velocity", "accel", "intact_count", "bond_broken", "force_density", "damage")


@pytest.fixture(scope="module")
def grains():
    """20 grains of alternating material: axis orders and tables meet within slices."""
    wl = I.grain_aggregate(n_grains=20, seed=2, grid=(5, 2, 2), n_min=1.4e4, n_max=2.6e4, platen_speed=5.0, rebuild_every=5)
    assert (wl.n_nodes + 63) // 64 >= 4096
    m = wl.materials[0]
    wl.materials = [m, I.Material(0.4 * m.bulk_modulus, 1.3 * m.density, m.fracture_energy)]
    wl.grain_material[:] = np.arange(wl.n_grains) % 2
    return wl


def _sim(wl, flags=0, **launch):
    from paper_2506_05362_amd import pd
    mem = Recorder()
    sim = pd.Sim(wl, flags=flags, plumbing=mem, candidate_capacity_per_node=96)
    if launch:
        sim.set_launch(**launch)
    return sim, mem


def _first_steps(sim, mem, n):
    """bytes a node that the first steps allocate: lined rows take more than a hundred"""
    before = mem.in_use
    sim.step(n)
    return (mem.in_use - before) / sim.n


def _equal(sims, what):
    want = {f: sims[0].get(f) for f in FIELDS}
    for sim in sims[1:]:
        for f in FIELDS:
            got = sim.get(f)
            assert np.array_equal(got, want[f]), (what, f)
    return want


@pytest.mark.parametrize("abs_stretch", [False, True])
@pytest.mark.parametrize("self_contact", [False, True])
def test_breaking_over_lined_rows(grains, abs_stretch, self_contact):
    """Bonds break at the build, over lined rows, and after a checkpoint and changes of the
    launch; fields, energies and checkpoints read the bond memory in between."""
    from paper_2506_05362_amd import pd
    h = float(grains.grain_h[0])
    wl = dataclasses.replace(grains, u0=grains.u0.copy(), v0=grains.v0.copy(), params=dataclasses.replace(
        grains.params, self_contact=self_contact, skin=0.5 * h, contact_damping=6.7e21, friction=0.2))
    wl.materials = [dataclasses.replace(m, fracture_energy=400.0 * m.fracture_energy) for m in grains.materials]
    rng = np.random.default_rng(1)
    wl.u0[:] = rng.normal(0.0, 0.02 * h, size=wl.u0.shape)
    wl.v0[:] += rng.normal(0.0, 10.0, size=wl.v0.shape)
    flags = pd.FLAG_ABS_STRETCH if abs_stretch else 0
    sims = []
    for launch in (dict(loop=pd.LOOP_PERSISTENT), {}, dict(loop=pd.LOOP_PER_GRAIN)):
        sim, mem = _sim(wl, flags, **launch)
        grown = _first_steps(sim, mem, 7)
        assert grown < 10 if launch.get("loop") == pd.LOOP_PERSISTENT else grown > 100, grown
        sims.append(sim)
    broken = _equal(sims, "first steps")["bond_broken"].mean()
    for sim in sims:
        sim.step(6)
    states = [sim.get_state() for sim in sims]
    assert states[1] == states[0] and states[2] == states[0]
    sims[1].set_state(states[0])
    sims[2].set_launch(loop=pd.LOOP_DIRECT)
    for sim in sims:
        sim.step(5)
    _equal(sims, "after a checkpoint")
    sims[1].set_launch(bond_path=pd.BONDS_TILES)   # lined rows -> column words -> masks
    sims[2].set_launch(loop=pd.LOOP_PERSISTENT)    # lined rows -> column words
    sims[0].set_launch()                           # column words -> lined rows
    for sim in sims:
        sim.step(5)
    want = _equal(sims, "after other launches")
    assert np.isfinite(want["displacement"]).all()
    assert 0.0 < broken < want["bond_broken"].mean() < 1.0
    for sim in sims:
        sim.close()


@pytest.mark.parametrize("amp", [1e-4, 1.5e-3, 6e-3, 3e-2])  # |x| of the stiffest bonds: about 3 amp to 10 amp
def test_bond_law_forms_over_lined_rows(grains, amp):
    from paper_2506_05362_amd import pd
    wl = dataclasses.replace(grains, u0=grains.u0.copy(), v0=grains.v0.copy(), walls=[])
    wl.materials = [dataclasses.replace(m, fracture_energy=1e8 * m.fracture_energy) for m in grains.materials]
    wl.u0[:] = np.random.default_rng(5).normal(0.0, amp * wl.grain_h[0], size=wl.u0.shape)
    sims = []
    for launch in (dict(loop=pd.LOOP_PERSISTENT), {}):
        sim, mem = _sim(wl, **launch)
        grown = _first_steps(sim, mem, 3)
        assert grown < 10 if launch else grown > 100, grown
        sims.append(sim)
    want = _equal(sims, amp)
    assert np.isfinite(want["displacement"]).all() and not want["bond_broken"].any()
    for sim in sims:
        sim.close()
