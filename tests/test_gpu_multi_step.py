"""The multi-step kernels where their strips change in number, with the MRT collision in
batches and in the index-checked build, on the largest benchmarked lattice and past 2^31
elements."""
import ctypes as C

import numpy as np
import pytest

from oracle import lbm as olbm
from tests.gpu_common import CS, mirror_tile, pair, slab_rho
from tests.test_gpu_mrt import _batch_runs

pytestmark = pytest.mark.gpu
RATES = (1.3, 1.1, 1.2)


@pytest.fixture(scope="module")
def L():
    import torch
    from paper_1204_4098_amd import lbm
    assert torch.cuda.is_available()
    lbm.lib()
    return lbm


def _after(L, gp, rho0, tile, n, graph=0):
    lat = L.Lattice(gp, rho0)
    lat.set_tile(*tile)
    if graph:
        lat.set_graph_steps(graph)
    lat.step(n)
    assert lat.status() == (L.LBM_OK, n, -1)
    raw = lat.save_state()[56:]
    lat.close()
    return raw


# FP64 arithmetic has three waves per step: strips of 64*3 - (4*steps - 2) columns, FP64
# storage's edges rounded down to 8 (a strip fewer 7 columns wide); two steps take six waves
# (378 columns) unless that leaves a quarter more lanes idle
@pytest.mark.parametrize("nx", [174, 175, 176, 182, 183, 184, 349, 350, 351, 364, 365, 524, 525, 526, 527])
@pytest.mark.parametrize("prec", [0, 3])
def test_three_steps_where_the_strips_change(L, nx, prec):
    gp, _ = pair(L, nx, 9, t=0.8, tau=0.8, scheme=2, sigma=0.1, precision=prec)
    rho0 = slab_rho(nx, 9, CS, 0.8, seed=nx)
    ref = _after(L, gp, rho0, (2, 8, 1, 1), 11)
    for tile in [(4, 0, 1, 3), (4, 3, 1, 3)]:
        assert _after(L, gp, rho0, tile, 11) == ref, tile


@pytest.mark.parametrize("nx", [178, 179, 180, 185, 186, 187, 188, 357, 358, 359, 372, 373, 378, 379, 380])
@pytest.mark.parametrize("prec", [0, 3])
def test_two_steps_where_the_strips_change(L, nx, prec):
    gp, _ = pair(L, nx, 9, t=0.8, tau=0.8, scheme=2, sigma=0.1, precision=prec)
    rho0 = slab_rho(nx, 9, CS, 0.8, seed=nx)
    ref = _after(L, gp, rho0, (2, 8, 1, 1), 11)
    for tile in [(4, 0, 2, 2), (4, 3, 1, 2)]:
        assert _after(L, gp, rho0, tile, 11) == ref, tile


@pytest.mark.parametrize("tile,graph", [((2, 0, 1, 4), 0), ((4, 0, 1, 4), 10), ((2, 4, 1, 4), 6), ((4, 32, 1, 4), 0)])
@pytest.mark.parametrize("prec", [0, 1])
def test_mrt_batch_of_four_steps_equals_single_lattices(L, prec, tile, graph):
    # 3, then 34 steps: one and two left over, also in the graphs
    gps, rhos, rates = _batch_runs(L, prec)
    b = L.Batch(gps, rhos)
    b.set_tile(*tile)
    b.set_mrt(rates)
    if graph:
        b.set_graph_steps(graph)
    b.step(3)
    b.step(34)
    for i, (gp, rho, r) in enumerate(zip(gps, rhos, rates)):
        lat = L.Lattice(gp, rho)
        lat.set_mrt(r)
        lat.set_tile(2, 8, 1, 1)
        lat.step(37)
        assert np.array_equal(b.get_populations(i), lat.get_populations()[0]), (tile, i)
        lat.close()
    b.close()


@pytest.mark.parametrize("prec", [0, 1])
def test_mrt_tiles_in_bounds(monkeypatch, prec):
    import torch
    from paper_1204_4098_amd import lbm as L
    assert torch.cuda.is_available()
    monkeypatch.setattr(L, "_lib", L.load(L.LIB_CHECK_PATH))
    n = C.c_uint64()
    assert L.lib().lbm_debug_index_faults(C.byref(n)) == L.LBM_OK
    for nx, ny in [(3, 3), (5, 4), (130, 7), (179, 5), (300, 70)]:
        gp, _ = pair(L, nx, ny, t=0.9, tau=0.9, scheme=2, sigma=0.05, precision=prec)
        lat = L.Lattice(gp, np.full((ny, nx), 0.11))
        lat.set_mrt(RATES)
        for tile in [(4, 0, 1, 4), (2, 0, 1, 4), (4, 5, 1, 4), (2, 1, 1, 4), (4, 0, 1, 2), (1, 0, 1, 4), (1, 0, 1, 3),
                     (1, 0, 1, 2)]:
            lat.set_tile(*tile)
            lat.step(7)
        lat.close()
    gps, rhos, rates = _batch_runs(L, prec)
    b = L.Batch(gps, rhos)
    b.set_mrt(rates)
    for tile in [(2, 0, 1, 4), (4, 0, 1, 4), (2, 4, 1, 4), (4, 16, 1, 4), (2, 5, 1, 2)]:
        b.set_tile(*tile)
        b.step(7)
    b.close()
    assert L.lib().lbm_debug_index_faults(C.byref(n)) == L.LBM_OK and n.value == 0


def test_full_size_four_steps_bitwise(L):
    # the tile that the benchmark's tuner picks, against single steps, eager and replayed
    gp, _ = pair(L, 4096, 4096, t=0.7, tau=0.8, scheme=2, sigma=0.105)
    rho0 = slab_rho(4096, 4096, CS, 0.7, seed=9)
    ref = _after(L, gp, rho0, (16, 0, 1, 1), 11)
    for tile, graph in [((4, 0, 1, 4), 0), ((4, 0, 1, 4), 4)]:
        assert _after(L, gp, rho0, tile, 11, graph) == ref, (tile, graph)


def test_four_steps_and_patches_beyond_2_31_elements(L):
    # as the other tile families: windows near the first and last rows against the oracle
    nx, ny, half = 4096, 70000, 20
    gp, op = pair(L, nx, ny, t=0.8, tau=0.8, scheme=2, sigma=0.1)
    rho0 = slab_rho(nx, ny, CS, 0.8, seed=51)
    pts = [(0, ny - 1), (nx - 1, ny - 3), (1024, 0), (3000, 66000), (2048, 40000)]
    wins = {}
    for cx, cy in pts:
        ys, xs = np.arange(cy - half, cy + half) % ny, np.arange(cx - half, cx + half) % nx
        wins[(cx, cy)] = mirror_tile(olbm.init_equilibrium(np.ascontiguousarray(rho0[np.ix_(ys, xs)])))
    wp = olbm.Params(**{**op.__dict__, "nx": 4 * half, "ny": 4 * half})
    lat = L.Lattice(gp, rho0)
    del rho0
    done = 0
    for tile in [(4, 0, 1, 4), (1, 0, 1, 4)]:
        lat.set_tile(*tile)
        lat.step(4)
        done += 4
        assert lat.status()[0] == L.LBM_OK
        rho = lat.moments()[0]
        m = 2 * done + 1                            # light cone of `done` steps
        for cx, cy in pts:
            win = wins[(cx, cy)]
            assert olbm.step(wp, win, 4)[0] == olbm.OK
            ref = olbm.moments(wp, win)[0][m:2 * half - m, m:2 * half - m]
            ys, xs = np.arange(cy - half + m, cy + half - m) % ny, np.arange(cx - half + m, cx + half - m) % nx
            err = float(np.max(np.abs(rho[np.ix_(ys, xs)] - ref) / ref))
            assert err < 1e-12, (tile, (cx, cy), err)
        del rho
    lat.close()
