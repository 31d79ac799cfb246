"""Device memory of the simulator: none is asked for and left unused, reading fields out
takes none, and goes to any."""
import numpy as np
import pytest

from paper_2506_05362_amd import inputs as I

pytestmark = pytest.mark.gpu


class Recorder:
    """PyTorch's caching allocator and a stream; holds the sizes in use, and can refuse."""

    def __init__(self):
        from paper_2506_05362_amd import pd
        base = pd.TorchPlumbing()
        self.torch, self.device, self.stream, self.stream_ptr = base.torch, base.device, base.stream, base.stream_ptr
        self.sizes, self.refuse, self.refused = {}, False, 0

        def _alloc(nbytes, user):
            if self.refuse:
                self.refused += 1
                return None
            p = self.torch.cuda.caching_allocator_alloc(int(nbytes), self.device, self.stream)
            self.sizes[p] = int(nbytes)
            return p

        def _free(ptr, user):
            del self.sizes[ptr]
            self.torch.cuda.caching_allocator_delete(int(ptr))

        self.alloc, self.free = pd.ALLOC_FN(_alloc), pd.FREE_FN(_free)

    @property
    def in_use(self):
        return sum(self.sizes.values())


def _mesh():
    wl = I.two_spheres(radius_cells=6, speed=30.0, gap=0.0)
    wl.v0[:] += np.random.default_rng(0).normal(0.0, 1.0, size=wl.v0.shape)
    return wl


def test_fields_without_device_memory():
    """State, damage and counts come out, to host and device memory, when there is no device
    memory left: the same values as where there is, and nothing is asked for."""
    import torch
    from paper_2506_05362_amd import pd
    wl = _mesh()
    mem = Recorder()
    sim, other = pd.Sim(wl, plumbing=mem), pd.Sim(wl)
    for s in (sim, other):
        s.step(25)
    mem.refuse = True
    for name in ("displacement", "velocity", "accel", "damage", "intact_count", "initial_count"):
        host = sim.get(name)
        dev = torch.zeros(host.size, dtype=getattr(torch, str(host.dtype)), device="cuda")
        sim.get_device(name, dev.data_ptr(), sim.field_bytes(name))
        assert np.array_equal(host, other.get(name)), name
        assert np.array_equal(dev.cpu().numpy(), host.ravel()), name
    assert mem.refused == 0
    for s in (sim, other):  # the read-outs left the candidates alone
        s.step(25)
    assert np.array_equal(sim.get("displacement"), other.get("displacement"))
    sim.close()


def test_fields_into_any_device_memory():
    """A destination at any byte of a device array, or in pinned host memory handed over as
    device memory, is written as a copy would: the bytes around it stay."""
    import torch
    from paper_2506_05362_amd import pd
    sim = pd.Sim(_mesh())
    sim.step(20)
    for name in ("displacement", "velocity", "damage"):
        want = sim.get(name).tobytes()
        for kind in ("device", "pinned"):
            for off in (0, 1, 4, 8):
                print(name, kind, off, flush=True)
                buf = torch.full((len(want) + 16,), 7, dtype=torch.uint8,
                                 **(dict(device="cuda") if kind == "device" else dict(pin_memory=True)))
                sim.get_device(name, buf.data_ptr() + off, len(want))
                torch.cuda.synchronize()
                b = buf.cpu().numpy().tobytes()
                assert b[:off] == b"\x07" * off and b[off + len(want):] == b"\x07" * (16 - off)
                assert b[off:off + len(want)] == want, (name, kind, off)
    sim.close()


def test_no_allocation_is_left_unused():
    """Every device array that grows with the mesh is written by a build and some steps with
    contact and walls: each is handed out full of one byte, and holds another afterwards."""
    import torch
    from paper_2506_05362_amd import pd

    class Marked(Recorder):
        def __init__(self):
            super().__init__()
            self.arrays = {}

            def _alloc(nbytes, user):
                with torch.cuda.stream(self.stream):
                    t = torch.full((int(nbytes),), 0xA5, dtype=torch.uint8, device="cuda")
                self.arrays[t.data_ptr()] = t
                return t.data_ptr()

            def _free(ptr, user):
                del self.arrays[ptr]

            self.alloc, self.free = pd.ALLOC_FN(_alloc), pd.FREE_FN(_free)

    wl = _mesh()
    lo, hi = wl.X.min(axis=1), wl.X.max(axis=1)
    h = wl.grain_h[0]
    wl.walls = [I.Wall(normal=(0.0, 0.0, 1.0), offset=lo[2] - 0.5 * h), I.Wall(normal=(0.0, 0.0, -1.0), offset=-hi[2] - 0.5 * h)]
    mem = Marked()
    sim = pd.Sim(wl, plumbing=mem)
    sim.step(25)
    torch.cuda.synchronize()
    big = [t for t in mem.arrays.values() if t.numel() >= wl.n_nodes]
    assert len(big) > 10
    unused = [t.numel() for t in big if not bool((t != 0xA5).any())]
    assert not unused, unused
    sim.close()
