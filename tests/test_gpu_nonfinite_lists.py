"""Particles with a NaN or infinite coordinate have no neighbours, not even
each other (every comparison of the definition's test is false), and the
lists of all others are as without them: in each kernel of the list build."""
import numpy as np
import pytest

import mdinputs
from conftest import gpu_device, split_dev

pytestmark = pytest.mark.gpu

# lattice sites per axis: a lane per particle; waves per stencil row and per cell of few bricks
CASES = {"lanes": 48, "three_rows": 32, "one_row": 10}


def _pairs(pos, box):
    from paper_1704_03329_amd.sim import LJSim

    sim = LJSim(pos.shape[0], box, rc=2.5, skin=0.3, precision="fp32", max_nb=256)
    sim.build(*split_dev(pos))
    assert sim.check(raise_on_error=False)[0] == 0
    p = sim.pairs().numpy()
    return p[:, 0].astype(np.int64) * pos.shape[0] + p[:, 1]


@pytest.mark.parametrize("axes", [(0,), (1,), (2,), (0, 1), (0, 2), (1, 2), (0, 1, 2)])
@pytest.mark.parametrize("name", list(CASES))
def test_particles_without_a_position(name, axes):
    gpu_device()
    print(name, axes, flush=True)
    m = CASES[name]
    box = np.full(3, m * mdinputs.LJ_RHO ** (-1.0 / 3.0))
    g = (np.arange(m) + 0.5) * box[0] / m
    zz, yy, xx = np.meshgrid(g, g, g, indexing="ij")
    pos = mdinputs.perturb(np.stack([xx.ravel(), yy.ravel(), zz.ravel()], 1), 0.2, 83) % box
    n = pos.shape[0]
    # the 24 nearest to a point, seen along the axes that they lose: one neighbourhood
    kept = [k for k in range(3) if k not in axes]
    near = np.argsort(((pos[:, kept] - 0.3 * box[kept]) ** 2).sum(1) if kept else np.arange(n), kind="stable")[:24]
    lost = pos.copy()
    for q, k in enumerate(axes):
        lost[near, k] = np.array([np.nan, np.inf, -np.inf])[(np.arange(24) + q) % 3]
    finite = np.setdiff1d(np.arange(n), near)
    want = _pairs(pos[finite], box)
    i, j = finite[want // finite.size], finite[want % finite.size]
    assert np.array_equal(np.sort(_pairs(lost, box)), np.sort(i * n + j))
