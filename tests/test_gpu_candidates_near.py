"""Candidates where only the nodes near other grains are binned: long grains of which an end
touches, both ends (the box around the near ones then spans the grain), nothing at first;
dense and hashed cells; and nodes that come near between rebuilds."""
import numpy as np
import pytest

from paper_2506_05362_amd import inputs as I
from test_gpu_candidates import H, brute_force

pytestmark = pytest.mark.gpu
CASES = {
    "one_end": [((30, 5, 5), (0, 0, 0)), ((5, 5, 5), (30, 0, 0.3))],
    "both_ends": [((30, 5, 5), (0, 0, 0)), ((5, 5, 5), (30, 0, 0.3)), ((5, 5, 5), (-5, 0.2, 0))],
    "crossed": [((30, 5, 5), (0, 0, 0)), ((5, 30, 5), (12, -12, 5))],
    "hashed": [((30, 5, 5), (0, 0, 0)), ((5, 5, 5), (30, 0, 0.3)), ((4, 4, 4), (9e4, 7e4, 0)), ((4, 4, 4), (9e4, 7e4 + 4, 0))],
    "empty_between": [((30, 5, 5), (0, 0, 0)), ((30, 5, 5), (0, 12, 0)), ((5, 5, 5), (10, 5, 0))],
    "small": [((30, 3, 3), (0, 0, 0)), ((5, 5, 5), (30, 0, 0.3)), ((6, 10, 9), (12, 3, 0))],
}


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_rows_of_nodes_near_other_grains(name, axis):
    from paper_2506_05362_amd import pd
    bl = []
    for n, at in CASES[name]:
        ijk, o = I.grain_block(I.box_offsets(*np.roll(n, axis)), np.roll(np.asarray(at, dtype=np.float64), axis) * H, H)
        bl.append((ijk, o, H, 0))
    wl = I.assemble("blocks", bl, [I.SAND], I.default_params(H, 1e-8, rebuild_every=10), [], [], 1)
    rng = np.random.default_rng(axis)
    wl.u0[:] = rng.uniform(-0.02 * H, 0.02 * H, size=wl.u0.shape)
    # grains move by a tenth of a spacing between rebuilds
    wl.v0[:] = rng.uniform(-50.0, 50.0, size=(3, wl.n_grains))[:, wl.grain_of_node()]
    wl.params.skin = 0.5 * H
    print(name, axis, wl.n_nodes, flush=True)
    sim = pd.Sim(wl, candidate_capacity_per_node=60)
    for steps in (0, 10, 30):  # rebuilds at multiples of 10 steps, at the positions read
        sim.step(steps)
        wl.u0[:] = sim.get("displacement")
        ptr, col = sim.candidates()
        rows = brute_force(wl)
        assert sum(len(r) for r in rows) > 0
        assert np.array_equal(np.diff(ptr), [len(r) for r in rows]), steps
        assert np.array_equal(col, np.concatenate(rows)), steps
    sim.close()
