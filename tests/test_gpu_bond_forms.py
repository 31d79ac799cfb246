"""One bond at the edges of the ranges of the bond law's forms and beyond them, down to a
hundredth of its length, against the law in extended precision."""
import dataclasses

import numpy as np
import pytest

from paper_2506_05362_amd import inputs as I

pytestmark = pytest.mark.gpu
EDGES = [s * e * (1.0 + t) for e in (0.0055, 0.08) for s in (1.0, -1.0) for t in (-1e-9, 1e-9)]


@pytest.mark.parametrize("x", [1e-9, -1e-4, *EDGES, 0.02, -0.05, 0.3, 3.0, -0.3, -0.9, -0.99, -0.9999])
def test_one_bond(x):
    """Two nodes a spacing apart, |y|^2 / |xi|^2 = 1 + x, without breaking.  The force goes
    through the constants (some 14 roundings of 2^-53), x, the form and the density (another
    10): 32 * 2^-53 relative."""
    from paper_2506_05362_amd import pd
    h, L = 1e-4, np.longdouble
    m = dataclasses.replace(I.SAND, fracture_energy=np.inf)
    ijk, o = I.grain_block(I.box_offsets(2, 1, 1), np.zeros(3), h)
    wl = I.assemble("pair", [(ijk, o, h, 0)], [m], I.default_params(h, 1e-12), [], [], 1)
    e = float(h * (np.sqrt(1.0 + x) - 1.0))
    wl.u0[0, 1] = e
    eta = L(e)
    y = L(h) + eta
    g = eta * (2 * L(h) + eta) / (y * (y + L(h)))  # 1 - |xi| / |y|, without a difference of lengths
    c = 18 * L(m.bulk_modulus) / (L("3.14159265358979323846264338327950288") * (3 * L(h)) ** 4)
    want = c * L(h) ** 3 / L(h) * g * y / L(m.density)
    for path in (pd.BONDS_SLICES, pd.BONDS_TILES):
        sim = pd.Sim(wl)
        sim.set_launch(bond_path=path)
        if path == pd.BONDS_TILES:
            sim.step(1)  # evaluates one drift of dt later: the force changes by far less
        a = sim.get("accel")
        tol = 32 * 2.0 ** -53 if path == pd.BONDS_SLICES else 1e-9
        assert abs(L(a[0, 0]) - want) <= tol * abs(want), (path, a[0, 0], want)
        assert a[0, 1] == -a[0, 0] and not a[1:].any()
        sim.close()
