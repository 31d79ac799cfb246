"""The work a user of this framework has it do, as cases that can be timed.

Two libraries stand behind the public entry points: the simulator (`pd.Sim`:
explicit peridynamic steps of grains and aggregates) and the surrogate network
(`mlp.Net`: BF16 matrix-core forward, backward and Adam).  A simulation case is
one logging interval of a running simulation - some steps, then the fields and
wall reactions read out, as scale_bench.py, shape_study.py and surrogate.py do -
and the simulation goes on from pass to pass.  A network case is one call (or a
few minibatch steps) on tensors that are already on the GPU.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2506_05362_amd import inputs as I
from paper_2506_05362_amd import mlp, pd, surrogate

DEV = "cuda"


# ----------------------------------------------------------------------------
# the cases
# ----------------------------------------------------------------------------

def listed():
    return [
        # a binary collision, the framework's smallest experiment: a few thousand nodes, so that
        # a step is launches and latency; fields read to numpy
        dict(name="spheres", kind="spheres", radius=10, speed=1.0, steps=100),
        # uneven level-set grains between platens (the batching study's kind of aggregate at a
        # size between the collision and the big volumes), default launch, sliced bond rows
        dict(name="grains", kind="grains", grains=16, n_max=2.0e4, steps=40),
        # impact on the double-notched plate of the fracture benchmark at its full size: one
        # grain, cuts, a moving wall patch, cracks after some hundred steps, LDS tiles
        dict(name="plate", kind="plate", nx=200, ny=200, nz=18, speed=32.0, steps=100),
        # the shape study's box of 125 grains under a falling lid with the whole contact model:
        # damping, self-contact, wall corners, candidates rebuilt every 5 steps, sliced rows
        dict(name="shapes", kind="shapes", shape="sphere", grid=5, self_contact=True, wall_corners=True, steps=50),
        # one logging interval of the representative volume behind the surrogate's training data:
        # servo walls, damping, early rebuilds, LDS tiles over the shared lattice
        dict(name="volume", kind="volume", grains=200, nodes_per_grain=1850, friction=0.0, steps=100),
        # the large aggregate at its full size (about 9.3 million nodes) as the scale run sets it
        # up: damping, a wide skin, a rebuild every 5 steps, LDS tiles; logged every 100 steps
        dict(name="aggregate", kind="aggregate", side=210, grains=1000, rebuild_every=5, steps=100),
        # one strain path of 100 points through the trained network: a query of one path
        dict(name="infer path", kind="forward", width=256, hidden=3, batch=100, max_batch=65536),
        # the surrogate's bulk query of 100,000 paths x 100 points as one batch
        dict(name="infer bulk", kind="forward", width=256, hidden=3, batch=10_000_000, max_batch=65536),
        # a network of another width: the layer-by-layer kernels that training uses
        dict(name="infer layers", kind="forward", width=128, hidden=2, batch=65536, max_batch=65536),
        # minibatch training as Surrogate.fit does it: 512 samples a step
        dict(name="train", kind="train", batch=512, steps=4),
        # the same with large minibatches
        dict(name="train large", kind="train", batch=16384, steps=4),
        # loss and gradient of one batch for a caller's own optimiser
        dict(name="gradients", kind="gradients", batch=4096),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["spheres", "grains", "plate", "shapes", "volume", "aggregate", "forward", "forward", "train",
                       "gradients"])
    if kind == "spheres":
        return dict(kind=kind, radius=rng.randint(4, 18), speed=round(_log(rng, 0.5, 10.0), 3), steps=rng.randint(20, 150))
    if kind == "grains":
        return dict(kind=kind, grains=rng.randint(3, 16), n_max=round(_log(rng, 2.5e3, 2.0e4), 1), steps=rng.randint(20, 60))
    if kind == "plate":
        k = rng.randint(5, 25)  # notches at a quarter and three quarters of the width, half as deep
        return dict(kind=kind, nx=8 * k, ny=rng.randint(4 * k, 8 * k) // 2 * 2, nz=rng.randint(5, 18),
                    speed=round(rng.uniform(8.0, 32.0), 2), steps=rng.randint(20, 120))
    if kind == "shapes":
        return dict(kind=kind, shape=rng.choice(list(I.SHAPES)), grid=rng.randint(1, 5), self_contact=rng.random() < 0.5,
                    wall_corners=rng.random() < 0.5, steps=rng.randint(20, 60))
    if kind == "volume":
        return dict(kind=kind, grains=rng.randint(12, 200), nodes_per_grain=rng.randint(300, 1850),
                    friction=rng.choice([0.0, 0.3]), steps=rng.randint(20, 100))
    if kind == "aggregate":
        side = int(_log(rng, 48, 150))
        return dict(kind=kind, side=side, grains=max(8, side ** 3 // rng.randint(4000, 12000)),
                    rebuild_every=rng.choice([5, 10, 20]), steps=rng.randint(20, 100))
    if kind == "forward":
        width = rng.choice([256, 256, 256, 64, 128, 200])
        hidden = 3 if width == 256 else rng.randint(1, 3)
        return dict(kind=kind, width=width, hidden=hidden, batch=int(_log(rng, 1, 4e6 if width == 256 else 2e5)),
                    max_batch=rng.choice([4096, 65536]))
    if kind == "train":
        return dict(kind=kind, batch=int(_log(rng, 64, 16384)), steps=rng.randint(1, 4))
    return dict(kind=kind, batch=int(_log(rng, 64, 16384)))


# ----------------------------------------------------------------------------
# what a program has in hand
# ----------------------------------------------------------------------------

def _aggregate(seed, side, grains, rebuild_every):
    """A Laguerre tessellation of a side^3 lattice into log-normally sized grains, confined by six
    walls, as inputs.large_aggregate lays it out (there with a host-side search that takes a minute)."""
    h, dt = 4.1e-5, 4.0e-9
    rng = np.random.default_rng(seed)
    L = side * h
    radii = rng.lognormal(0.0, 0.3, size=grains)
    radii *= L / np.sum(4.0 / 3.0 * math.pi * radii ** 3) ** (1.0 / 3.0)
    seeds = rng.uniform(0.0, L, size=(grains, 3))
    cell = np.floor(seeds / (L / 8.0)).astype(np.int64)
    perm = np.lexsort((seeds[:, 0], cell[:, 0], cell[:, 1], cell[:, 2]))
    c = torch.tensor(seeds[perm], dtype=torch.float32, device=DEV)
    r2 = torch.tensor(radii[perm] ** 2, dtype=torch.float32, device=DEV)
    ax = (torch.arange(side, device=DEV, dtype=torch.float32) + 0.5) * h
    d2 = [(ax[:, None] - c[None, :, q]) ** 2 for q in range(3)]
    gid = torch.empty((side, side, side), dtype=torch.int64, device=DEV)
    for i in range(side):
        for k0 in range(0, side, 64):
            p = (d2[0][i] - r2)[None, None, :] + d2[1][k0:k0 + 64, None, :] + d2[2][None, :, :]
            gid[i, k0:k0 + 64] = p.argmin(dim=2)
    gid = gid.reshape(-1)
    count = torch.bincount(gid, minlength=grains)
    keep = count >= 20  # slivers are left out, as the library's own generator does
    order = torch.sort(gid, stable=True).indices
    order = order[keep[gid[order]]]
    new_id = torch.cumsum(keep.long(), 0) - 1
    g = new_id[gid[order]]
    ng = int(keep.sum())
    lat = torch.stack([order // (side * side), order // side % side, order % side])
    lo = torch.full((3, ng), side, dtype=torch.int64, device=DEV).scatter_reduce(1, g.expand(3, -1), lat, "amin")
    ijk = lat - lo[:, g]
    begin = np.zeros(ng + 1, dtype=np.int64)
    begin[1:] = torch.cumsum(count[keep], 0).cpu().numpy()
    origin = 0.5 * h + h * lo.double()
    X = (origin[:, g] + h * ijk.double()).cpu().numpy()
    n = X.shape[1]
    params = I.default_params(h, dt, rebuild_every=rebuild_every)
    params.contact_damping = 2.4e23
    params.skin = 0.5 * h
    a, b = X.min(axis=1) - h, X.max(axis=1) + h
    span = b - a
    area = [span[1] * span[2], span[0] * span[2], span[0] * span[1]]
    walls = [I.Wall(normal=(0.0, 0.0, 1.0), offset=a[2], area=area[2]),
             I.Wall(normal=(0.0, 0.0, -1.0), offset=-b[2], mode=I.WALL_VELOCITY, velocity=10.0, area=area[2])]
    for q in (0, 1):
        for s in (1.0, -1.0):
            normal = [0.0, 0.0, 0.0]
            normal[q] = s
            walls.append(I.Wall(normal=tuple(normal), offset=a[q] if s > 0 else -b[q], area=area[q]))
    return I.Workload(name="aggregate", X=X, ijk=ijk.to(torch.int32).cpu().numpy(), grain_begin=begin,
                      grain_h=np.full(ng, h), grain_origin=origin.cpu().numpy(),
                      grain_material=np.zeros(ng, dtype=np.int32), materials=[I.SAND], params=params,
                      u0=np.zeros((3, n)), v0=np.zeros((3, n)), fixed=np.zeros(n, dtype=np.uint8), walls=walls, cuts=[],
                      steps=1)


MESH_SEED = 1


def _stir(wl, seed, speed):
    """Nothing is quite at rest when a run starts: small random velocities, the seed's share of the input
    (the meshes themselves are the same for every seed, so that all of a case's runs have one size)."""
    wl.v0[:] = np.random.default_rng(seed).normal(0.0, speed, size=wl.v0.shape)
    return wl


def _workload(case, seed):
    """(workload, candidate capacity, tiled bond loop)"""
    kind = case["kind"]
    if kind == "spheres":
        return I.two_spheres(seed=seed, radius_cells=case["radius"], speed=case["speed"], gap=0.0), 0, False
    if kind == "grains":
        gx = math.ceil(case["grains"] / 4)
        wl = I.grain_aggregate(n_grains=case["grains"], seed=MESH_SEED, grid=(gx, 2, 2), n_min=2e3, n_max=case["n_max"])
        return _stir(wl, seed, 0.01), 0, False
    if kind == "plate":
        h = 5e-4
        nx, ny = case["nx"], case["ny"]
        wl = I.notched_plate(nx=nx, ny=ny, nz=case["nz"], h=h, notch_x=(nx // 4 * h, nx // 4 * 3 * h),
                             notch_len=ny // 2 * h, speed=case["speed"])
        return _stir(wl, seed, 0.05), 0, True
    if kind == "shapes":
        wl = I.shape_study(case["shape"], seed=MESH_SEED, grid=case["grid"], rebuild_every=5)
        wl.params.contact_damping = 6.7e21
        wl.params.skin = 0.4 * 1e-4
        wl.params.self_contact = case["self_contact"]
        wl.params.wall_corners = case["wall_corners"]
        return _stir(wl, seed, 0.05), 48, False
    if kind == "volume":
        conf = float(np.random.default_rng(seed).uniform(0.0, 20e6))
        wl = I.rve_aggregate(seed=MESH_SEED, n_grains=case["grains"], nodes_per_grain=case["nodes_per_grain"],
                             confinement=conf, friction=case["friction"], **surrogate.RVE_DEFAULTS)
        return _stir(wl, seed, 0.02), surrogate.SIM_CAPACITY, True
    return _stir(_aggregate(MESH_SEED, case["side"], case["grains"], case["rebuild_every"]), seed, 0.02), 32, True


def _dims(case):
    return [6] + [case.get("width", 256)] * case.get("hidden", 3) + [7]


def _samples(case, seed):
    """Standardised strains (three normal ones, no shear: the rig's paths), targets and weights."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    x = torch.randn((case["batch"], 6), generator=g, device=DEV)
    x[:, 3:] = 0.0
    y = torch.tanh(x[:, [0, 1, 2, 0, 1, 2, 2]]) * 1.3 + 0.3 * torch.randn((case["batch"], 7), generator=g, device=DEV)
    return x, y, surrogate.init_params(_dims(case), seed)


def prepare(case, seed):
    if case["kind"] in ("forward", "train", "gradients"):
        x, y, p = _samples(case, seed)
        net = mlp.Net(_dims(case), max_batch=case.get("max_batch", case["batch"]))
        net.set_params(p)
        net.set_adam(weight_decay=1e-2)
        return dict(case=case, net=net, x=x, y=y)
    wl, capacity, tiles = _workload(case, seed)
    sim = pd.Sim(wl, candidate_capacity_per_node=capacity)
    if tiles:
        sim.set_launch(bond_path=pd.BONDS_TILES)
    f = lambda *shape: torch.empty(shape, dtype=torch.float64, device=DEV)  # noqa: E731
    return dict(case=case, sim=sim, n=wl.n_nodes, u=f(3, wl.n_nodes), v=f(3, wl.n_nodes), damage=f(wl.n_nodes))


# ----------------------------------------------------------------------------
# one pass
# ----------------------------------------------------------------------------

def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "forward":
        return state["net"].forward(state["x"])
    if kind == "train":
        net = state["net"]
        with torch.cuda.stream(net.stream):
            for k in range(case["steps"]):
                net.train_step(state["x"], state["y"], 2e-3, want_loss=False)
            return net.get_params()
    if kind == "gradients":
        loss, grad = state["net"].gradients(state["x"], state["y"])
        return dict(loss=np.float32(loss), grad=grad)
    sim, n = state["sim"], state["n"]
    sim.step(case["steps"])
    walls = dict(force=sim.get("wall_force"), offset=sim.get("wall_offset"), impulse=sim.get("wall_impulse"))
    if kind in ("spheres", "grains"):  # small meshes are looked at in numpy
        return dict(u=sim.get("displacement"), v=sim.get("velocity"), damage=sim.get("damage"), walls=walls)
    sim.get_device("displacement", state["u"].data_ptr(), 24 * n)
    sim.get_device("velocity", state["v"].data_ptr(), 24 * n)
    sim.get_device("damage", state["damage"].data_ptr(), 8 * n)
    return dict(u=state["u"], v=state["v"], damage=state["damage"], walls=walls)


# ----------------------------------------------------------------------------
# what a pass cannot do without
# ----------------------------------------------------------------------------

def _mesh_size(case):
    """(nodes, directed bonds), near enough: 122 neighbours at horizon factor 3 less those beyond the surface."""
    kind = case["kind"]
    ball = lambda r: 4.0 / 3.0 * math.pi * r ** 3  # noqa: E731
    if kind == "spheres":
        sizes = [ball(case["radius"])] * 2
    elif kind == "grains":
        sizes = [(case["n_max"] - 2e3) / math.log(case["n_max"] / 2e3)] * case["grains"]
    elif kind == "plate":
        n = float(case["nx"] * case["ny"] * case["nz"])
        return n, n * 122.0 * (1.0 - 1.3 / case["nz"])
    elif kind == "shapes":
        sizes = [ball(10.0) * {"sphere": 1.0, "shell": 0.875, "jack": 0.29}[case["shape"]]] * case["grid"] ** 3
    elif kind == "volume":
        sizes = [float(case["nodes_per_grain"])] * case["grains"]
    else:
        sizes = [case["side"] ** 3 / case["grains"]] * case["grains"]
    return sum(sizes), sum(122.0 * n * max(0.3, 1.0 - 2.8 * n ** (-1.0 / 3.0)) for n in sizes)


def work(case):
    kind = case["kind"]
    if kind in ("forward", "train", "gradients"):
        dims = _dims(case)
        products = 2.0 * sum(a * b for a, b in zip(dims[:-1], dims[1:]))
        weights = 4.0 * sum(a * b + b for a, b in zip(dims[:-1], dims[1:]))
        if kind == "forward":
            return dict(bytes=weights + 4.0 * case["batch"] * (dims[0] + dims[-1]), flops=products * case["batch"])
        # backward: two products for each forward one, less the input's; Adam reads p, g, m, v and writes p, m, v
        passes = case.get("steps", 1)
        flops = case["batch"] * (3.0 * products - 2.0 * dims[0] * dims[1])
        moved = 4.0 * case["batch"] * (dims[0] + dims[-1]) + weights * (7.0 if kind == "train" else 2.0)
        return dict(bytes=passes * moved, flops=passes * flops)
    # a step reads and writes u, v and a of every node and one bit of bond memory for each directed bond; a
    # bond's force takes about 45 operations and serves both of its ends; the read-out writes u, v and damage
    n, bonds = _mesh_size(case)
    return dict(bytes=case["steps"] * (144.0 * n + bonds / 8.0) + 56.0 * n, flops=case["steps"] * 45.0 * bonds / 2.0)


# ----------------------------------------------------------------------------
# the same in 64 bits, without the framework's code
# ----------------------------------------------------------------------------

def _layers(p, dims):
    out, o = [], 0
    for a, b in zip(dims[:-1], dims[1:]):
        out.append((p[o:o + a * b].view(a, b), p[o + a * b:o + a * b + b]))
        o += a * b + b
    return out


def _net(p, dims, x):
    layers = _layers(p, dims)
    for k, (w, b) in enumerate(layers):
        x = x @ w + b
        if k < len(layers) - 1:
            x = torch.nn.functional.gelu(x)
    return x


def _loss(p, dims, x, y):
    return ((_net(p, dims, x) - y) ** 2).mean()


def _exact_steps(wl, steps):
    """Velocity Verlet of bonds, contact between two grains and planar walls, in plain torch."""
    f64 = dict(dtype=torch.float64, device=DEV)
    n, h, mat, prm = wl.n_nodes, float(wl.grain_h[0]), wl.materials[0], wl.params
    m, V, Rc = prm.horizon_factor, h ** 3, prm.contact_radius
    delta = m * h
    c = 18.0 * mat.bulk_modulus / (math.pi * delta ** 4)
    s0 = math.sqrt(5.0 * mat.fracture_energy / (9.0 * mat.bulk_modulus * delta))
    Kn = 18.0 * mat.bulk_modulus / (math.pi * prm.contact_horizon ** 5)
    X, u, v = (torch.tensor(a, **f64) for a in (wl.X, wl.u0, wl.v0))
    ijk = torch.tensor(wl.ijk, dtype=torch.int64, device=DEV)
    # neighbours and intact bonds of each horizon offset
    offsets = [(a, b, d) for a in range(-m, m + 1) for b in range(-m, m + 1) for d in range(-m, m + 1)
               if 0 < a * a + b * b + d * d <= m * m]
    g = torch.tensor(wl.grain_of_node().astype(np.int64), device=DEV)
    ext = [int(e) + 1 + 2 * m for e in wl.ijk.max(axis=1)]
    table = torch.full((wl.n_grains, *ext), -1, dtype=torch.int64, device=DEV)
    table[g, ijk[0] + m, ijk[1] + m, ijk[2] + m] = torch.arange(n, device=DEV)
    nbr, alive = [], []
    for d in offsets:
        j = table[g, ijk[0] + m + d[0], ijk[1] + m + d[1], ijk[2] + m + d[2]]
        ok = j >= 0
        for cut in wl.cuts:  # notch planes x = const, half-lattice units, down to a largest y
            A, B = 2 * ijk, 2 * (ijk + torch.tensor(d, device=DEV)[:, None])
            fa, fb = A[0] + cut.plane[3], B[0] + cut.plane[3]
            t = fa.double() / torch.where(fa == fb, 1, fa - fb).double()
            ok &= ~((fa * fb < 0) & (A[1] + t * (B[1] - A[1]) <= cut.hi[1]))
        nbr.append(torch.where(ok, j, torch.arange(n, device=DEV)))
        alive.append(ok)
    initial = sum(a.long() for a in alive)
    split = int(wl.grain_begin[1])

    def force(step):
        F = torch.zeros_like(u)
        for k, d in enumerate(offsets):
            xi = h * torch.tensor(d, **f64)[:, None]
            e = u[:, nbr[k]] - u
            y = xi + e
            l0 = h * math.sqrt(d[0] ** 2 + d[1] ** 2 + d[2] ** 2)
            dd = (e * (y + xi)).sum(0)
            l = torch.sqrt(l0 * l0 + dd)
            s = dd / (l0 * (l0 + l))
            alive[k] &= s <= s0
            F += torch.where(alive[k], c * V * s / l, 0.0) * y
        if wl.n_grains == 2:
            p = X + u
            # only nodes near the other grain's box can touch it
            a, b = torch.arange(split, device=DEV), torch.arange(split, n, device=DEV)
            for q in range(3):
                lo, hi = p[q, b].min() - Rc, p[q, b].max() + Rc
                a = a[(p[q, a] >= lo) & (p[q, a] <= hi)] if len(b) else a
                if len(a):
                    lo, hi = p[q, a].min() - Rc, p[q, a].max() + Rc
                    b = b[(p[q, b] >= lo) & (p[q, b] <= hi)]
            if len(a) and len(b):
                r = p[:, b][:, None, :] - p[:, a][:, :, None]
                dist = r.square().sum(0).sqrt()
                f = torch.where(dist < Rc, Kn * (Rc - dist) * V / dist, 0.0) * r
                F[:, a] -= f.sum(2)
                F[:, b] += f.sum(1)
        for w in wl.walls:
            p = X + u
            nrm = torch.tensor(w.normal, **f64)[:, None]
            inside = torch.ones(n, dtype=torch.bool, device=DEV)
            for q in range(3):
                inside &= (p[q] >= w.lo[q]) & (p[q] <= w.hi[q])
            d = (nrm * p).sum(0) - (w.offset + w.velocity * step * prm.dt)
            ell = 0.75 * (Rc + d) ** 2 / (2.0 * Rc + d)
            cap = math.pi / 3.0 * (Rc - d) ** 2 * (2.0 * Rc + d)
            F += torch.where(inside & (d < Rc), Kn * (Rc - ell) * cap, 0.0) * nrm
        return F / mat.density

    a = force(0)
    for s in range(1, steps + 1):
        u = u + prm.dt * v + 0.5 * prm.dt ** 2 * a
        new = force(s)
        v = v + 0.5 * prm.dt * (a + new)
        a = new
    left = sum(x.long() for x in alive)
    damage = torch.where(initial > 0, 1.0 - left.double() / initial.clamp(min=1).double(), 0.0)
    return dict(u=u, v=v, damage=damage, walls=None)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("spheres", "plate"):
        wl, _, _ = _workload(case, seed)
        if wl.n_nodes * case["steps"] > 100_000_000:
            return None  # more than 20 seconds
        return _exact_steps(wl, case["steps"])
    if kind not in ("forward", "train", "gradients"):
        return None
    x, y, p = _samples(case, seed)
    dims = _dims(case)
    p = torch.tensor(p, device=DEV).double()
    if kind == "forward":
        out = torch.empty((case["batch"], dims[-1]), dtype=torch.float64, device=DEV)
        for k in range(0, case["batch"], 1 << 20):
            out[k:k + (1 << 20)] = _net(p, dims, x[k:k + (1 << 20)].double())
        return out
    x, y = x.double(), y.double()
    m, v = torch.zeros_like(p), torch.zeros_like(p)
    for t in range(1, case.get("steps", 1) + 1):
        q = p.clone().requires_grad_(True)
        loss = _loss(q, dims, x, y)
        (grad,) = torch.autograd.grad(loss, q)
        if kind == "gradients":
            return dict(loss=loss.detach(), grad=grad)
        m = 0.9 * m + 0.1 * grad
        v = 0.999 * v + 0.001 * grad * grad
        p = p - 2e-3 * (m / (1 - 0.9 ** t) / ((v / (1 - 0.999 ** t)).sqrt() + 1e-8) + 1e-2 * p)
    return p
