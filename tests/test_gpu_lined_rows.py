"""Steps over lined rows (meshes of 4096 slices and more) against the compact rows, which
the persistent loop reads, and against the tiles: bitwise the same node state, through
breaking bonds, changes of the launch and a checkpoint."""
import numpy as np
import pytest

from paper_2506_05362_amd import inputs as I

pytestmark = pytest.mark.gpu
FIELDS = ("displacement", "velocity", "intact_count", "bond_broken")


def workloads():
    return {
        # two grains, breaking where they meet
        "spheres": lambda: I.two_spheres(radius_cells=32, speed=60.0, gap=0.0, rebuild_every=5),
        # one grain with cuts, thin: rows of another axis order, slices that do not line up
        "plate": lambda: I.notched_plate(nx=260, ny=210, nz=5, h=5e-4, notch_x=(65 * 5e-4, 195 * 5e-4),
                                         notch_len=105 * 5e-4, steps=1),
        # a plain block, 3 nodes in the last slice
        "block": lambda: I.notched_plate(nx=67, ny=63, nz=63, h=5e-4, notch_x=(1e-2, 2e-2), notch_len=1e-2, steps=1),
        # grains of several axis orders, slices that hold two of them
        "grains": lambda: I.grain_aggregate(n_grains=20, seed=2, grid=(5, 2, 2), n_min=1.4e4, n_max=2.6e4,
                                            platen_speed=5.0, rebuild_every=10),
    }


@pytest.mark.parametrize("name", list(workloads()))
def test_lined_rows_bitwise_equal_to_compact(name):
    from paper_2506_05362_amd import pd
    wl = workloads()[name]()
    print(name, wl.n_nodes, flush=True)
    assert (wl.n_nodes + 63) // 64 >= 4096
    wl.v0[:] += np.random.default_rng(1).normal(0.0, 2.0, size=wl.v0.shape)
    a, b, c = pd.Sim(wl), pd.Sim(wl), pd.Sim(wl)
    b.set_launch(loop=pd.LOOP_PERSISTENT)
    a.step(20)
    b.step(20)
    blob = a.get_state()
    c.step(3)
    c.set_state(blob)                       # onto lined rows, with broken bonds
    a.set_launch(bond_path=pd.BONDS_TILES)  # lined -> masks
    a.step(5)
    a.set_launch(loop=pd.LOOP_DIRECT)       # masks -> lined
    for sim, steps in ((a, 10), (b, 15), (c, 15)):
        sim.step(steps)
    want = {f: b.get(f) for f in FIELDS}
    if name == "spheres":
        assert want["bond_broken"].any()
    for sim in (a, c):
        for f in FIELDS:
            assert np.array_equal(sim.get(f), want[f]), f
