"""The multi-step kernels (one group of waves per time step): every storage type
and step count bitwise equal to single steps on widths around the strip limits,
the smallest lattices, ragged rows, remainders, graphs, frozen runs and batches,
and within bounds in the index-checked build."""
import ctypes as C

import numpy as np
import pytest

import synth
from tests.gpu_common import CS, PR, pair, slab_rho

pytestmark = pytest.mark.gpu

# widest strip of a tile: 64 k - (4 steps - 2) columns, k = 4 (FP32 arithmetic) or 3, 2 for
# the narrow class; FP64 strip edges are rounded down to 8 columns
FOUR = [(4, 0, 1, 4), (2, 0, 1, 4), (4, 5, 1, 4), (2, 1, 1, 4), (8, 16, 1, 4)]
# patches of 22 x 22 (four steps: 8 x 8 stored) and 32 x 32 nodes (26 and 22 square)
PATCH = [(1, 0, 1, 4), (1, 0, 1, 3), (1, 0, 1, 2)]


@pytest.fixture(scope="module")
def L():
    import torch
    from paper_1204_4098_amd import lbm
    assert torch.cuda.is_available()
    lbm.lib()
    return lbm


def _rho(nx, ny, seed):
    return np.ascontiguousarray(0.1 + 0.02 * np.random.default_rng(seed).random((ny, nx)))


def _run(L, gp, rho0, tile, n, graph=0, rates=None):
    lat = L.Lattice(gp, rho0)
    if rates:
        lat.set_mrt(rates)
    lat.set_tile(*tile)
    if graph:
        lat.set_graph_steps(graph)
    lat.step(n)
    st, done, div = lat.status()
    f = lat.get_populations()[0]
    lat.close()
    assert (st, done, div) == (L.LBM_OK, n, -1)
    return f


@pytest.mark.parametrize("prec", [0, 1, 2, 3])
@pytest.mark.parametrize("nx,ny", [(3, 3), (5, 4), (64, 7), (107, 9), (108, 9), (114, 5), (115, 6),
                                   (171, 11), (172, 11), (178, 9), (179, 9), (235, 13), (242, 9),
                                   (243, 9), (485, 10)])
def test_four_steps_bitwise_at_strip_edges(L, nx, ny, prec):
    gp, _ = pair(L, nx, ny, t=0.9, tau=0.9, scheme=2, sigma=0.05, precision=prec)
    rho0 = _rho(nx, ny, nx + ny)
    # 4 + 4 + 3: the remainder is one launch of three steps, or two and one
    ref = _run(L, gp, rho0, (2, 8, 1), 11)
    for tile in FOUR:
        assert np.array_equal(_run(L, gp, rho0, tile, 11), ref), tile


@pytest.mark.parametrize("prec", [0, 3])
@pytest.mark.parametrize("nx,ny", [(371, 9), (378, 7), (379, 7), (756, 6), (757, 40), (1100, 5)])
def test_two_steps_with_six_waves(L, nx, ny, prec):
    # strips of up to 378 columns (FP64 arithmetic); 2 + 2 + 2 + 1 steps
    gp, _ = pair(L, nx, ny, t=0.9, tau=0.9, scheme=2, sigma=0.05, precision=prec)
    rho0 = _rho(nx, ny, nx + ny)
    ref = _run(L, gp, rho0, (2, 8, 1), 7)
    for tile in [(4, 0, 1, 2), (4, 5, 1, 2), (8, 0, 2, 2)]:
        assert np.array_equal(_run(L, gp, rho0, tile, 7), ref), tile


@pytest.mark.parametrize("prec", [0, 1, 2, 3])
@pytest.mark.parametrize("nx,ny", [(3, 3), (5, 4), (8, 8), (9, 7), (22, 23), (26, 27), (64, 32), (130, 45)])
def test_patches_bitwise(L, nx, ny, prec):
    gp, _ = pair(L, nx, ny, t=0.9, tau=0.9, scheme=2, sigma=0.05, precision=prec)
    rho0 = _rho(nx, ny, nx + ny)
    ref = _run(L, gp, rho0, (2, 8, 1), 23)
    for tile in PATCH:
        assert np.array_equal(_run(L, gp, rho0, tile, 23), ref), tile
        assert np.array_equal(_run(L, gp, rho0, tile, 23, graph=10), ref), tile


@pytest.mark.parametrize("prec,rates", [(0, None), (0, (1.3, 1.1, 1.2)), (1, (1.3, 1.1, 1.2)), (2, None)])
@pytest.mark.parametrize("k", [6, 10, 12])
def test_four_step_graphs_bitwise(L, k, prec, rates):
    # replays of graphs with remainders of two steps (k = 6, 10: two and three launches) and none
    gp, _ = pair(L, 300, 70, t=0.8, tau=0.8, scheme=2, sigma=0.105, precision=prec)
    rho0 = slab_rho(300, 70, CS, 0.8, seed=6)
    ref = _run(L, gp, rho0, (2, 8, 1), 5 * k + 7, rates=rates)
    for tile in [(4, 0, 1, 4), (2, 0, 1, 4), (1, 0, 1, 4), (1, 0, 1, 3)]:
        assert np.array_equal(_run(L, gp, rho0, tile, 5 * k + 7, graph=k, rates=rates), ref), tile


@pytest.mark.parametrize("scheme,eos,t", [(0, CS, 0.85), (1, CS, 0.85), (3, CS, 0.85), (4, CS, 0.95),
                                          (2, PR, 0.8)])
def test_four_step_schemes_bitwise(L, scheme, eos, t):
    gp, _ = pair(L, 300, 70, t=t, tau=0.7, scheme=scheme, sigma=0.105, eos=eos)
    rho0 = slab_rho(300, 70, eos, t, seed=8)
    ref = _run(L, gp, rho0, (2, 8, 1), 41)
    for tile in [(4, 0, 1, 4), (1, 0, 1, 4)]:
        assert np.array_equal(_run(L, gp, rho0, tile, 41), ref), tile


@pytest.mark.parametrize("tile", [(4, 0, 1, 4), (2, 16, 1, 4), (4, 0, 1, 3), (1, 0, 1, 4), (1, 0, 1, 3)])
def test_multi_step_divergence_step_and_freeze(L, tile):
    # the step reported is the first with a bad node, whichever step of a launch it is,
    # and the state stays what the diverging launch wrote
    from oracle import thermo as th
    gp, _ = pair(L, 96, 80, t=0.6, tau=1.0, scheme=2, sigma=0.105, eos=PR)
    c = th.maxwell_pr(0.6)
    rho0 = synth.droplet(96, 80, c.rho_l, c.rho_g, 20, 4.0, 0.005)
    one = L.Lattice(gp, rho0)
    one.step(200)
    lat = L.Lattice(gp, rho0)
    lat.set_tile(*tile)
    lat.step(200)
    assert lat.status()[0] == L.LBM_EDIVERGED and lat.status()[2] == one.status()[2]
    snap = lat.save_state()[56:]              # raw storage after the header
    for extra in (1, 2, 5):
        lat.step(extra)
        assert lat.save_state()[56:] == snap
    one.close(); lat.close()


@pytest.mark.parametrize("tile", [(2, 0, 1, 4), (4, 0, 1, 4), (8, 16, 1, 4), (2, 4, 1, 4), (4, 0, 1, 2)])
@pytest.mark.parametrize("prec", [0, 1, 2, 3])
def test_batch_four_steps_bitwise(L, tile, prec):
    # uneven runs, one lower than four rows (more strips than chunks), two models, 4 k + 3 steps
    specs = [(64, 16, 0.8, 2, CS), (211, 33, 0.75, 2, CS), (97, 17, 0.9, 1, CS), (130, 20, 0.8, 2, PR),
             (513, 3, 0.85, 2, CS), (3, 3, 0.9, 2, CS)]
    gps, rhos = [], []
    for i, (nx, ny, t, scheme, eos) in enumerate(specs):
        gps.append(pair(L, nx, ny, t=t, tau=0.8, scheme=scheme, sigma=0.1, eos=eos, precision=prec,
                        rho_ref=0.0)[0])
        rhos.append(slab_rho(nx, ny, eos, t, stream=i) if nx > 3 else _rho(nx, ny, 5))
    a, b = L.Batch(gps, rhos), L.Batch(gps, rhos)
    a.set_tile(1, 16, 2)
    b.set_tile(*tile)
    b.set_graph_steps(10)
    for n in (7, 24):
        a.step(n)
        b.step(n)
    for i in range(len(gps)):
        assert np.array_equal(a.get_populations(i, check=False), b.get_populations(i, check=False)), i
    assert np.array_equal(a.coexistence()[3], b.coexistence()[3])
    a.close(); b.close()


@pytest.mark.parametrize("tile", [(2, 5, 1, 4), (4, 4, 1, 4), (4, 0, 1, 4), (2, 4, 1, 2), (4, 7, 1, 2)])
@pytest.mark.parametrize("prec", [0, 1, 2, 3])
def test_blocks_with_many_pieces(L, tile, prec):
    # up to 2,000 pieces of 1 to 7 rows (a block marches several without draining), or
    # whole strips; a run in the middle diverges, so its pieces become copies
    from oracle import thermo as th
    gps, rhos = [], []
    for i in range(28):
        nx, ny = 64 + 37 * (i % 11), 80 + 13 * (i % 5)
        gps.append(pair(L, nx, ny, t=0.85, tau=0.7 + 0.02 * i, scheme=2, sigma=0.1, precision=prec)[0])
        rhos.append(slab_rho(nx, ny, CS, 0.85, stream=i))
    c = th.maxwell_pr(0.6)
    gps.insert(9, pair(L, 96, 80, t=0.6, tau=1.0, scheme=2, sigma=0.105, eos=PR, precision=prec)[0])
    rhos.insert(9, synth.droplet(96, 80, c.rho_l, c.rho_g, 20, 4.0, 0.005))
    a, b = L.Batch(gps, rhos), L.Batch(gps, rhos)
    a.set_tile(1, 16, 2)
    b.set_tile(*tile)
    a.step(203)
    b.step(203)
    st = b.coexistence()[2]
    assert st[9] == L.LBM_EDIVERGED and np.array_equal(a.coexistence()[2], st)
    for i in range(len(gps)):
        if i != 9:
            assert np.array_equal(a.get_populations(i), b.get_populations(i)), i
    a.close(); b.close()


@pytest.mark.parametrize("prec", [0, 1, 2, 3])
def test_four_steps_in_bounds(monkeypatch, prec):
    import torch
    from paper_1204_4098_amd import lbm as L
    assert torch.cuda.is_available()
    monkeypatch.setattr(L, "_lib", L.load(L.LIB_CHECK_PATH))
    n = C.c_uint64()
    assert L.lib().lbm_debug_index_faults(C.byref(n)) == L.LBM_OK
    gps, rhos = [], []
    for nx, ny in [(3, 3), (5, 4), (115, 7), (179, 5), (300, 70)]:
        gp, _ = pair(L, nx, ny, t=0.9, tau=0.9, scheme=2, sigma=0.05, precision=prec)
        gps.append(gp)
        rhos.append(_rho(nx, ny, nx + ny))
        for tile in FOUR + PATCH:
            lat = L.Lattice(gp, rhos[-1])
            lat.set_tile(*tile)
            lat.step(9)
            lat.close()
    for tile in [(2, 0, 1, 4), (4, 0, 1, 4), (2, 4, 1, 4)]:
        b = L.Batch(gps, rhos)
        b.set_tile(*tile)
        b.step(7)
        b.close()
    assert L.lib().lbm_debug_index_faults(C.byref(n)) == L.LBM_OK and n.value == 0


def test_four_step_tiles_rejected_where_unsupported(L):
    gp, _ = pair(L, 64, 32, t=0.8, tau=0.8, scheme=2, sigma=0.1)
    lat = L.Lattice(gp, slab_rho(64, 32, CS, 0.8, seed=1))
    for tile in [(1, 4, 1, 4), (1, 0, 2, 2), (16, 0, 1, 4), (4, 0, 2, 4), (4, 0, 1, 5), (2, 0, 1, 3),
                 (2, 0, 1, 2)]:
        with pytest.raises(L.LbmError):
            lat.set_tile(*tile)
    lat.set_tile(2, 0, 1, 4)
    assert lat.get_tile() == (2, 0, 1, 4)
    lat.close()
