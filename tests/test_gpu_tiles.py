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
