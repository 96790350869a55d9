"""The node arithmetic: FP16 lattices keep their populations bit for bit."""
import hashlib
import json
import os

import pytest

from tests.gpu_common import CS, PR, pair, slab_rho

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
