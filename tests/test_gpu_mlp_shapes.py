"""Gradients and inference of the surrogate network at the edges of its kernels:
batches around the 128-row chunks of the weight gradients and around the
switch between 32 x 32 and 64 x 64 tiles, layer widths that are no multiple of
4 (padded rows) or exceed a tile, one-column layers, and an input that is not
16-byte aligned, against the BF16 emulation of the FP64 oracle.

Tolerance: FP32 sums over at most 4200 rows in another order than the
emulation's are within 4200 * 2^-24 = 2.5e-4 of it; an activation on a BF16
rounding boundary (2^-8) flips with probability about 2^-24 / 2^-8, which adds
2^-8 * 2^-8 = 1.5e-5 per layer; 2e-3 covers both with room for the GELU's own
rounding."""
import numpy as np
import pytest

from oracle import mlp_ref as M
from test_gpu_mlp import forward_bf16, gradients_bf16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,batch", [([6, 256, 256, 256, 7], 1), ([6, 256, 256, 256, 7], 127),
                                        ([6, 256, 256, 256, 7], 129), ([6, 256, 256, 256, 7], 512),
                                        ([6, 256, 256, 256, 7], 4161), ([5, 33, 70, 3], 640), ([8, 1, 9, 1], 513),
                                        ([1, 130, 1], 65)])
@pytest.mark.parametrize("shift", [0, 1])
def test_gradients_at_tile_and_chunk_edges(dims, batch, shift):
    import torch
    from paper_2506_05362_amd import mlp
    print(dims, batch, shift, flush=True)
    rng = np.random.default_rng(batch + shift)
    p = (M.init_params(dims, seed=1) + rng.normal(0, 0.02, M.n_params(dims))).astype(np.float32).astype(np.float64)
    X = rng.normal(size=(batch, dims[0])).astype(np.float32)
    Y = rng.normal(size=(batch, dims[-1])).astype(np.float32)
    net = mlp.Net(dims, max_batch=batch + 3)
    net.set_params(p)
    x = torch.empty(X.size + shift, device="cuda")[shift:].view(X.shape)
    x.copy_(torch.from_numpy(X))
    loss, g = net.gradients(x, torch.from_numpy(Y))
    emu = gradients_bf16(p, dims, X, Y)
    assert loss == pytest.approx(M.loss(p, dims, X, Y), rel=2e-2)
    assert np.linalg.norm(g - emu) <= 2e-3 * np.linalg.norm(emu)


@pytest.mark.parametrize("din,dout", [(6, 7), (8, 16), (9, 1), (16, 4)])
def test_fused_inference_at_tile_edges(din, dout):
    """16-row tiles, the switch to 32-row tiles (32 rows for each of 256 CUs) and the first
    tile that a workgroup takes in a second round, against the layer-by-layer kernels and the
    emulation (tolerances as for the gradients: flips of BF16 roundings, 2e-4)."""
    import torch
    from paper_2506_05362_amd import mlp
    dims = [din, 256, 256, 256, dout]
    rng = np.random.default_rng(din)
    p = (M.init_params(dims, seed=2) + rng.normal(0, 0.02, M.n_params(dims))).astype(np.float32).astype(np.float64)
    net = mlp.Net(dims, max_batch=4096)
    net.set_params(p)
    X = rng.normal(size=(16500, din)).astype(np.float32)
    x = torch.from_numpy(X).cuda()
    emu, _ = forward_bf16(p, dims, X[:300])
    for m in (1, 15, 16, 17, 300, 8191, 8192, 8193, 16384, 16385, 16500):
        print(dims, m, flush=True)
        net.set_inference(True)
        y = net.forward(x[:m]).cpu().numpy()
        net.set_inference(False)
        yl = net.forward(x[:m]).cpu().numpy()
        assert np.linalg.norm(y - yl) <= 2e-4 * np.linalg.norm(yl)
        k = min(m, 300)
        assert np.linalg.norm(y[:k] - emu[:k]) <= 2e-4 * np.linalg.norm(emu[:k])
