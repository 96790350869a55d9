"""Macroscopic fields and mass on widths around the strip and unit limits of their
kernels (62, 126 and 254 columns; units of 64), the smallest lattices and heights
that leave a short last chunk, against the oracle on the same populations."""
import numpy as np
import pytest

from oracle import lbm as olbm
from tests.gpu_common import CS, PR, pair

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    import torch
    from paper_1204_4098_amd import lbm
    assert torch.cuda.is_available()
    lbm.lib()
    return lbm


@pytest.mark.parametrize("prec", [0, 1, 2, 3])
@pytest.mark.parametrize("nx,ny", [(3, 3), (5, 4), (62, 5), (63, 6), (64, 7), (65, 3), (126, 9), (127, 8),
                                   (254, 17), (255, 16), (508, 5), (509, 33), (700, 301)])
def test_fields_and_mass_at_edges(L, nx, ny, prec):
    eos = PR if (nx + ny) % 2 else CS
    gp, op = pair(L, nx, ny, t=0.9, tau=0.9, scheme=2, sigma=0.05, eos=eos, precision=prec)
    rng = np.random.default_rng(nx * 1000 + ny)
    base = 0.1 if eos is CS else 2.0
    rho0 = np.ascontiguousarray(base * (1 + 0.2 * rng.random((ny, nx))))
    u0 = [np.ascontiguousarray(0.05 * (rng.random((ny, nx)) - 0.5)) for _ in range(2)]
    lat = L.Lattice(gp, rho0, *u0)
    f = lat.get_populations()[0]
    rho, vx, vy, p = lat.moments()
    ref = olbm.moments(op, f)
    # FP64: a few roundings of sums of order rho, and of psi, whose cancellation in p - rho/3
    # costs about one digit; FP32 arithmetic: the velocity is a quotient of FP32 sums of nine
    # stored deviations (9 half-ulps of about rho, over rho)
    tol = 1e-12 if prec in (0, 3) else 1e-5
    assert np.max(np.abs(rho / ref[0] - 1)) < (1e-13 if prec in (0, 3) else 1e-6)
    assert np.max(np.abs(vx - ref[1])) < tol and np.max(np.abs(vy - ref[2])) < tol
    assert np.max(np.abs(p - ref[3])) < (1e-12 if prec in (0, 3) else 1e-4) * np.max(np.abs(ref[3]))
    # the integer mass is exact: the direction-ordered sums, scaled and rounded to even
    s = np.zeros((ny, nx))
    for a in range(9):
        s = s + f[a]
    m, fixed = lat.mass()
    assert fixed == int(np.sum(np.rint(s * 2.0 ** 40).astype(np.int64)))
    assert abs(m / s.sum() - 1) < 1e-13
    lat.close()
