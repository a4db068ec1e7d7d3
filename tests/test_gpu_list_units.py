"""The neighbour list in other units of length: scaled by a power of two every
operation of the definition scales exactly, so that the lists are the same,
entry for entry, also where FP32 products of the coordinates would not be."""
import numpy as np
import pytest

import mdinputs
from conftest import gpu_device, split_dev

pytestmark = pytest.mark.gpu


def _pairs(m, scale, precision):
    from paper_1704_03329_amd.sim import LJSim

    box = np.full(3, m * mdinputs.LJ_RHO ** (-1.0 / 3.0))
    g = (np.arange(m) + 0.5) * box[0] / m
    zz, yy, xx = np.meshgrid(g, g, g, indexing="ij")
    pos = mdinputs.perturb(np.stack([xx.ravel(), yy.ravel(), zz.ravel()], 1), 0.2, 89) % box
    sim = LJSim(pos.shape[0], box * scale, rc=2.5 * scale, skin=0.3 * scale, sigma=scale, precision=precision, max_nb=160)
    sim.build(*split_dev(pos * scale))
    assert sim.check(raise_on_error=False)[0] == 0
    return sim.pairs().numpy()


@pytest.mark.parametrize("m", [10, 32, 48])
def test_lists_in_other_units(m):
    gpu_device()
    want = _pairs(m, 1.0, "fp64")
    for e in (-58, -54, -50, -48, -30, 30, 46, 48, 55, 58):
        print(m, e, flush=True)
        assert np.array_equal(_pairs(m, 2.0 ** e, "fp64"), want), e
