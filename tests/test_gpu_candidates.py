"""Contact-candidate rows against brute force, where the search changes its way:
rows longer than a thread sorts in registers (16) or holds in LDS (24), cells
hashed into buckets because the box has too many, a box far from the origin,
grains with nothing near, self-contact, and workgroups that read four records a
thread.  The distance is formed as the library documents it, so rows are equal."""
import numpy as np
import pytest

from paper_2506_05362_amd import inputs as I

pytestmark = pytest.mark.gpu
H = 1e-4


def blocks(at, n=6, jitter=0.3, seed=0, skin=0.25, self_contact=False):
    """Cubes of n^3 nodes at the given places (in spacings), every node displaced a little."""
    off = I.box_offsets(n, n, n)
    bl = []
    for c in at:
        ijk, origin = I.grain_block(off, np.asarray(c, dtype=np.float64) * H, H)
        bl.append((ijk, origin, H, 0))
    params = I.default_params(H, 1e-8)
    params.skin = skin * H
    params.self_contact = self_contact
    wl = I.assemble("blocks", bl, [I.SAND], params, [], [], 1)
    wl.u0[:] = np.random.default_rng(seed).uniform(-jitter * H, jitter * H, size=wl.u0.shape)
    return wl


def brute_force(wl):
    g = wl.grain_of_node()
    cut = wl.params.contact_radius + wl.params.skin
    rows = []
    for i in range(wl.n_nodes):
        p = (wl.X - wl.X[:, i:i + 1]) + (wl.u0 - wl.u0[:, i:i + 1])
        d2 = p[0] * p[0] + p[1] * p[1] + p[2] * p[2]
        ok = d2 < cut * cut
        ok &= (np.arange(wl.n_nodes) != i) if wl.params.self_contact else (g != g[i])
        rows.append(np.flatnonzero(ok))
    return rows


CASES = {
    "touching": dict(at=[(0, 0, 0), (6, 0, 0), (0, 6, 0.5)]),
    "long_rows": dict(at=[(0, 0, 0), (6, 0, 0)], skin=2.0),
    "interpenetrating": dict(at=[(0, 0, 0), (0.5, 0.5, 0.5), (0.2, 0.3, 0.1)], skin=1.0),
    "hashed": dict(at=[(0, 0, 0), (6, 0, 0), (9e4, 7e4, 0), (9e4, 7e4 + 6, 0)]),
    "far_from_origin": dict(at=[(1e6, -2e6, 3e6), (1e6 + 6, -2e6, 3e6)]),
    "one_isolated": dict(at=[(0, 0, 0), (6, 0, 0), (40, 0, 0)]),
    "all_isolated": dict(at=[(0, 0, 0), (20, 0, 0), (40, 0, 0)]),
    "self_contact": dict(at=[(0, 0, 0), (6.2, 0, 0)], self_contact=True, skin=0.4, jitter=0.02),
    "single_grain_self_contact": dict(at=[(0, 0, 0)], self_contact=True, skin=0.4, jitter=0.02),
    "single_grain": dict(at=[(0, 0, 0)]),
}


@pytest.mark.parametrize("name", list(CASES))
def test_candidates_equal_brute_force(name):
    from paper_2506_05362_amd import pd
    wl = blocks(**CASES[name])
    print(name, wl.n_nodes, flush=True)
    sim = pd.Sim(wl, candidate_capacity_per_node=150)
    ptr, col = sim.candidates()
    rows = brute_force(wl)
    assert np.array_equal(np.diff(ptr), [len(r) for r in rows])
    assert np.array_equal(col, np.concatenate(rows))
    if name == "long_rows":
        assert np.diff(ptr).max() > 24
    sim.close()


def test_large_workgroups():
    """2.2 million nodes in one lattice: four records a thread."""
    from paper_2506_05362_amd import pd
    n = 130
    r = np.arange(n)
    gid = (np.add.outer(np.add.outer(r // 33 * 16, r // 27 * 4), r // 41)).ravel()
    lat = I.box_offsets(n, n, n)
    bl = []
    for g in np.unique(gid):
        ijk, origin = I.grain_block(lat[:, gid == g], np.zeros(3), H, axes=(0, 1, 2))
        bl.append((ijk, origin, H, 0))
    wl = I.assemble("lattice", bl, [I.SAND], I.default_params(H, 1e-8), [], [], 1)
    assert wl.n_nodes >= 256 * 4 * 2048
    sim = pd.Sim(wl)
    ptr, col = sim.candidates()
    sim.close()
    # on an undeformed lattice a row is the face neighbours of other grains
    # (R_c + skin = 1.2 spacings)
    node = np.full((n + 2, n + 2, n + 2), -1, dtype=np.int64)
    own = np.full((n + 2, n + 2, n + 2), -1, dtype=np.int64)
    q = np.rint(wl.X / H).astype(np.int64) + 1
    node[tuple(q)] = np.arange(wl.n_nodes)
    own[tuple(q)] = wl.grain_of_node()
    nb = []
    for d in ((1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1)):
        at = tuple(q[k] + d[k] for k in range(3))
        nb.append(np.where((own[at] >= 0) & (own[at] != own[tuple(q)]), node[at], wl.n_nodes))
    nb = np.sort(np.stack(nb, axis=1), axis=1)
    assert np.array_equal(np.diff(ptr), (nb < wl.n_nodes).sum(axis=1))
    assert np.array_equal(col, nb[nb < wl.n_nodes])
