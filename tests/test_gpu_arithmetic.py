"""The node arithmetic: FP16 lattices keep their populations bit for bit, and psi^2 outside
the range of FP32 or 0 spoils nothing else."""
import hashlib
import json
import os

import numpy as np
import pytest

from tests.gpu_common import CS, PR, pair, slab_rho, temperature

pytestmark = pytest.mark.gpu
GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "fp16_states.json")


@pytest.fixture(scope="module")
def L():
    import torch
    from paper_1204_4098_amd import lbm
    assert torch.cuda.is_available()
    lbm.lib()
    return lbm


def _golden():
    with open(GOLDEN) as f:
        return json.load(f)["states"]


@pytest.mark.parametrize("case", _golden(), ids=lambda c: "{nx}x{ny}-eos{eos}-scheme{scheme}".format(**c))
def test_fp16_states_keep_their_bits(L, case):
    # digests of the raw storage after 101 steps, made with single steps per launch by the
    # library before it had kernels of several steps per wave group
    eos = CS if case["eos"] == 0 else PR
    gp, _ = pair(L, case["nx"], case["ny"], t=case["t"], tau=case["tau"], scheme=case["scheme"],
                 sigma=case["sigma"], eos=eos, precision=L.LBM_PREC_F16DEV)
    rho0 = slab_rho(case["nx"], case["ny"], eos, case["t"], seed=7)
    for tile in [(2, 8, 1, 1), (4, 0, 1, 2), (4, 0, 1, 4), (1, 0, 1, 4)]:
        lat = L.Lattice(gp, rho0)
        lat.set_tile(*tile)
        lat.step(101)
        assert lat.status()[0] == L.LBM_OK
        assert hashlib.sha256(lat.save_state()[56:]).hexdigest() == case["sha256"], tile
        lat.close()


@pytest.mark.parametrize("prec,scheme,mrt", [(p, s, False) for p in (1, 2) for s in (0, 1, 2, 4)] + [(1, 2, True)])
@pytest.mark.parametrize("power", [150, -150])
def test_psi2_outside_fp32_range(L, prec, scheme, mrt, power):
    # psi^2 = 2 (p - rho/3)/G: with G times 2^150 it is below the least FP32 number, with G
    # times 2^-150 above the largest.  psi scales by 2^(-+75), and the force G psi grad psi and
    # all that follows keep their bits; sigma = 0, so 1/psi^2 is not used
    nx, ny = 96, 40
    rho0 = slab_rho(nx, ny, CS, 0.9, seed=3)
    gp, _ = pair(L, nx, ny, t=0.9, tau=0.9, scheme=scheme, sigma=0.0, precision=prec)

    def run(G, tile):
        gp.G = G
        lat = L.Lattice(gp, rho0)
        if mrt:
            lat.set_mrt((1.3, 1.1, 1.2))
        lat.set_tile(*tile)
        lat.step(22)
        st = lat.status()
        raw = lat.save_state()[56:]
        lat.close()
        assert st == (L.LBM_OK, 22, -1), (tile, st)
        return raw

    want = run(-1.0, (2, 8, 1, 1))
    for tile in [(2, 8, 1, 1), (4, 0, 1, 2), (4, 0, 1, 4), (1, 0, 1, 3)]:
        assert run(-2.0 ** power, tile) == want, tile


@pytest.mark.parametrize("prec", [0, 1, 2, 3])
@pytest.mark.parametrize("nx,ny", [(9, 7), (130, 45)])
def test_fields_around_a_node_of_no_density(L, nx, ny, prec):
    # psi of an empty node is 0 (psi^2 = 2 (p - rho/3)/G = 0): its neighbours have a force and
    # a velocity.  Equilibrium at rest elsewhere, so v = F/(2 rho), F of psi(rho)
    T, _ = temperature(0, 0.9)
    gp, _ = pair(L, nx, ny, t=0.9, tau=0.9, scheme=2, sigma=0.1, precision=prec, rho_ref=0.0)
    rho0 = np.full((ny, nx), 0.125)
    lat = L.Lattice(gp, rho0)
    w = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4)[:, None, None]
    f = w * rho0
    f[:, 3, 4] = 0.0
    lat.set_populations(np.ascontiguousarray(f), 0)
    rho, vx, vy, p = lat.moments()
    lat.close()
    e = rho
    psi = np.sqrt(-2 * (rho * T * (1 + e + e * e - e ** 3) / (1 - e) ** 3 - rho * rho - rho / 3))
    assert rho[3, 4] == 0 and p[3, 4] == 0 and psi[3, 4] == 0
    F = np.zeros((2, ny, nx))
    for ex, ey in [(1, 0), (0, 1), (-1, 0), (0, -1), (1, 1), (-1, 1), (-1, -1), (1, -1)]:
        n = np.roll(psi, (-ey, -ex), (0, 1)) * (1 / 3 if ex * ey == 0 else 1 / 12)
        F[0] += ex * n
        F[1] += ey * n
    v = psi * F / (2 * np.where(rho > 0, rho, 1.0))
    full = rho > 0
    # FP64 sums of at most 8 numbers of 0.1, F and psi to 1e-15 each
    assert np.abs(vx - v[0])[full].max() < 1e-14 and np.abs(vy - v[1])[full].max() < 1e-14
    assert np.abs(v[:, 3, 3]).max() > 0.01
