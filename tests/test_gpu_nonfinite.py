"""A position that is not finite when the contact candidates are rebuilt: the step reports
it, and the rebuild bins no node outside its cell grid."""
import dataclasses

import numpy as np
import pytest

from paper_2506_05362_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("self_contact", [True, False])
@pytest.mark.parametrize("grains", [1, 2])
@pytest.mark.parametrize("bad", [np.nan, -np.nan, np.inf, -np.inf])
def test_rebuild_with_a_nonfinite_position(grains, bad, self_contact):
    """A velocity component that is not finite makes the position of step 1 so on that axis
    alone (the force at step 0 is finite), and with a rebuild every step the rebuild is the
    first to see it.  The evaluation of step 1 then flags the force: the call stops there."""
    from paper_2506_05362_amd import pd
    if grains == 1:
        wl = I.notched_plate(nx=24, ny=20, nz=6, notch_x=(3e-3, 9e-3), notch_len=4e-3)
    else:
        wl = I.two_spheres(radius_cells=6, gap=0.0)
    wl.params = dataclasses.replace(wl.params, self_contact=self_contact, rebuild_every=1)
    for axis in range(3):
        wl.v0[:] = 0.0
        wl.v0[axis, 7] = bad
        print(grains, bad, self_contact, axis, flush=True)
        sim = pd.Sim(wl)
        assert sim.step_status(5) == pd.PD_ERR_UNSTABLE
        assert "non-finite" in pd.lib().pd_last_error(sim.h).decode()
        assert sim.info()["step"] == 1
        ptr, col = sim.candidates()
        assert (np.diff(ptr) >= 0).all() and ((col >= 0) & (col < wl.n_nodes)).all()
        sim.close()
