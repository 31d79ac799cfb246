"""A HIP error while the lined rows are made is reported, and the rows are made again."""
import ctypes as C

import numpy as np
import pytest

from paper_2506_05362_amd import inputs as I
from test_gpu_device_memory import Recorder

pytestmark = pytest.mark.gpu


def test_error_while_lined_rows_are_filled():
    """The allocator hands out the last array (z of the second copy of u) with the error of
    another call left behind, which the launch that follows reports."""
    from paper_2506_05362_amd import pd
    wl = I.two_spheres(radius_cells=32, speed=50.0, gap=0.0)
    wl.v0[:] += np.random.default_rng(1).normal(0.0, 1.0, size=wl.v0.shape)
    mem, left = Recorder(), [0]
    hip, whole = pd.lib(), mem.alloc  # (hipMalloc of the runtime that the library loads)

    def leave_error(nbytes, user):
        p = whole(nbytes, user)
        if left[0] and 8 * wl.n_nodes <= nbytes < 9 * wl.n_nodes:
            left[0] -= 1
            if left[0]:
                return p
            q = C.c_void_p()
            assert hip.hipMalloc(C.byref(q), C.c_size_t(1 << 60)) != 0
        return p

    mem.alloc = pd.ALLOC_FN(leave_error)
    sim, other = pd.Sim(wl, plumbing=mem), pd.Sim(wl)
    left[0] = 2
    assert sim.step_status(5) == pd.PD_ERR_HIP
    assert sim.info()["step"] == 0
    assert left[0] == 0
    before = mem.in_use
    for s in (sim, other):
        s.step(5)
    assert mem.in_use - before > 100 * wl.n_nodes  # made after all
    for f in ("displacement", "velocity"):
        assert np.array_equal(sim.get(f), other.get(f)), f
    sim.close()
