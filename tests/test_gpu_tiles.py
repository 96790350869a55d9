"""Tiles kept from a tuner for later lattices and batches, and what runs the steps that a
tile leaves over."""
import numpy as np
import pytest

from tests.gpu_common import CS, pair, slab_rho

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    import torch
    from paper_1204_4098_amd import lbm
    assert torch.cuda.is_available()
    lbm.lib()
    return lbm


@pytest.mark.parametrize("prec", [0, 1])
def test_batch_takes_no_tile_of_a_lattice(L, prec):
    # a tuned MRT lattice of 864 x 72 and a BGK batch of one run of 72 x 12 = 864 nodes have the
    # same numbers in their cache keys; the lattice's tile (a patch of several steps) is none
    # of a batch
    gp, _ = pair(L, 864, 72, t=0.85, tau=0.9, scheme=2, sigma=0.1, precision=prec)
    big = L.Lattice(gp, slab_rho(864, 72, CS, 0.85, seed=2))
    big.set_mrt((1.3, 1.1, 1.2))
    big.tune()
    big.close()
    gp, _ = pair(L, 72, 12, t=0.85, tau=0.9, scheme=2, sigma=0.1, precision=prec)
    rho0 = slab_rho(72, 12, CS, 0.85, seed=2)
    b = L.Batch([gp], [rho0])
    assert b.get_tile() == (1, 16, 2, 1)          # an untuned batch's
    lat = L.Lattice(gp, rho0)
    for n in (1, 3, 4, 5):
        b.step(n)
        lat.step(n)
    assert np.array_equal(b.get_populations(0), lat.get_populations()[0])
    b.close(); lat.close()


def _us(lat, n, reps=60):
    """Shortest of several means, so that a clock or a neighbour does not decide."""
    import torch
    best = float("inf")
    for _ in range(5):
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        e[0].record(lat.stream)
        for _ in range(reps):
            lat.step(n)
        e[1].record(lat.stream)
        e[1].synchronize()
        best = min(best, e[0].elapsed_time(e[1]) * 1e3 / reps)
    return best


@pytest.mark.parametrize("nx,ny,prec", [(64, 8192, 0), (100, 3000, 3), (24, 4096, 0)])
def test_tuned_single_steps_cost_what_a_tile_of_one_step_does(L, nx, ny, prec):
    # a program that reads its lattice after each step: the tuned tile takes several steps
    # per launch, and with its strips of several waves one step took 1.5 to 2.4 times as long
    # as strips of one wave
    gp, _ = pair(L, nx, ny, t=0.85, tau=0.8, scheme=2, sigma=0.1, precision=prec)
    lat = L.Lattice(gp, slab_rho(nx, ny, CS, 0.85, seed=3))
    lat.tune()
    tuned = _us(lat, 1)
    lat.set_tile(1, 4 if ny > 5000 else 2, 1, 1)
    one = _us(lat, 1)
    lat.close()
    assert tuned < 1.3 * one, (tuned, one)


@pytest.mark.parametrize("prec", [0, 1, 2, 3])
@pytest.mark.parametrize("nx,ny", [(64, 32), (300, 200), (90, 3000)])
def test_tuned_steps_of_any_number_are_single_steps(L, nx, ny, prec):
    # whatever the tuner puts in for the steps left over, eager and in graphs
    gp, _ = pair(L, nx, ny, t=0.85, tau=0.8, scheme=2, sigma=0.1, precision=prec)
    rho0 = slab_rho(nx, ny, CS, 0.85, seed=4)
    a, b = L.Lattice(gp, rho0), L.Lattice(gp, rho0)
    a.set_tile(2, 8, 1, 1)
    b.tune()
    for graph, n in [(0, 1), (0, 2), (0, 3), (0, 7), (6, 25), (10, 33), (2, 5), (0, 5)]:
        b.set_graph_steps(graph)
        a.step(n)
        b.step(n)
        assert np.array_equal(a.get_populations()[0], b.get_populations()[0]), (graph, n)
    b.tune()                                      # other remainders perhaps, the same states
    a.step(11)
    b.step(11)
    assert np.array_equal(a.get_populations()[0], b.get_populations()[0])
    a.close(); b.close()


def _sweep(L, prec, n=256):
    import synth
    from paper_1204_4098_amd import surrogate
    runs = synth.sweep_runs(n, seed=5, lx=(64, 256, 32), ly=(16, 64, 16), t_range=(0.7, 0.95),
                            sigma_range=(0.05, 0.15))
    return surrogate.slab_runs(runs, prec, seed=5, rho_ref=0.0)


@pytest.mark.parametrize("prec", [0, 1, 2])
def test_steps_left_over_by_a_batch_tile_have_their_own_blocks(L, prec):
    # one step of a four-step tile (FP64: one block per CU) against a tile of one step with
    # strips of the same class; with the four-step list and its blocks it took 1.7 to 2.5 times
    # as long
    ps, rhos = _sweep(L, prec)
    b = L.Batch(ps, rhos)
    b.set_tile(2, 0, 1, 1)
    one = _us(b, 1, reps=30)
    b.set_tile(2, 0, 1, 4)
    left = _us(b, 1, reps=30)
    b.close()
    assert left < 1.3 * one, (left, one)


@pytest.mark.parametrize("prec,mrt", [(0, False), (0, True), (1, True), (2, False), (3, False)])
def test_tuned_batch_steps_of_any_number_are_single_steps(L, prec, mrt):
    ps, rhos = _sweep(L, prec, 30)
    a, b = L.Batch(ps, rhos), L.Batch(ps, rhos)
    a.set_tile(1, 16, 2, 1)
    b.tune()
    if mrt:                                       # after tuning: other kernels, other blocks
        a.set_mrt((1.3, 1.1, 1.2))
        b.set_mrt((1.3, 1.1, 1.2))
    for graph, n in [(0, 1), (0, 2), (0, 3), (0, 7), (6, 25), (10, 33), (2, 5), (0, 5)]:
        b.set_graph_steps(graph)
        a.step(n)
        b.step(n)
        for i in range(0, len(ps), 7):
            assert np.array_equal(a.get_populations(i), b.get_populations(i)), (graph, n, i)
    for tile in [(2, 0, 1, 4), (4, 32, 1, 4), (2, 5, 1, 4), (4, 16, 2, 2), (1, 8, 2, 1)]:
        b.set_tile(*tile)
        for n in (1, 2, 3, 4, 6):
            a.step(n)
            b.step(n)
        for i in range(0, len(ps), 7):
            assert np.array_equal(a.get_populations(i), b.get_populations(i)), (tile, i)
    a.close(); b.close()


def test_tuning_a_narrow_lattice_times_no_wide_tiles(L):
    # 3 columns: strips of 192 lanes took 0.3 s of the tuner's time and more, strips of one
    # wave take 20 ms
    import time
    gp, _ = pair(L, 3, 200000, t=0.85, tau=0.8, scheme=2, sigma=0.1)
    lat = L.Lattice(gp, np.full((200000, 3), 0.12))
    t0 = time.perf_counter()
    tile = lat.tune()
    took = time.perf_counter() - t0
    lat.close()
    assert tile[0] == 1 and took < 0.15, (tile, took)
