"""Inference into memory that overlaps the inputs."""
import numpy as np
import pytest

from oracle import mlp_ref as M

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("din,dout", [(16, 4), (6, 6), (6, 7)])
@pytest.mark.parametrize("shift", [0, 1000])  # floats from the inputs' start to the outputs'
def test_outputs_over_the_inputs(din, dout, shift):
    """Against the same network into memory of its own; the two may take different kernels,
    whose rounding of activations to BF16 differs as in the test of their tile edges: 2e-4."""
    import ctypes as C

    import torch
    from paper_2506_05362_amd import mlp
    dims, batch = [din, 256, 256, 256, dout], 16500
    net = mlp.Net(dims, max_batch=batch)
    net.set_params(M.init_params(dims, seed=2))
    x = torch.randn((batch, din), generator=torch.Generator("cuda").manual_seed(din), device="cuda")
    want = net.forward(x)
    buf = torch.zeros(shift + batch * max(din, dout), device="cuda")
    buf[:batch * din] = x.reshape(-1)
    torch.cuda.synchronize()
    at = lambda o: C.c_void_p(buf.data_ptr() + 4 * o)  # noqa: E731
    assert mlp.lib().pdm_forward(net.h, at(0), batch, at(shift)) == 0
    torch.cuda.synchronize()
    y = buf[shift:shift + batch * dout].view(batch, dout)
    assert torch.isfinite(want).all()
    assert float((y - want).norm()) <= 2e-4 * float(want.norm())
    assert np.isfinite(float(y.sum()))
