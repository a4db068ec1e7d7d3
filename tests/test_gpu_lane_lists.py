"""The list build with a lane per particle (large systems): a periodic cell
of few bricks, whose list another kernel builds, against the same cell
repeated, entry for entry in list order; the small list's pairs against the
oracle."""
import numpy as np
import pytest
import torch

import mdinputs
from conftest import gpu_device, split_dev
from oracle import lj as olj

pytestmark = pytest.mark.gpu

# cells of side 2.85 per axis; sites per axis; repeats per axis
CASES = {
    # 18 - 20 per cell (K = 3): 216 bricks of 3^3
    "liquid": ((6, 6, 6), (16, 16, 16), (3, 3, 3)),
    # 8 - 27 per cell (K = 2 .. 8), partial bricks along x and z in the repeated cell
    "lattice_ragged": ((5, 6, 4), (13, 16, 11), (4, 3, 5)),
    # about 11 per cell: many with fewer than 8, whose bricks take the general kernel
    "thin": ((6, 6, 6), (13, 13, 14), (3, 3, 3)),
    # 30 - 45 per cell (K = 1, 2): bricks of 2^3 and 1
    "dense": ((4, 4, 5), (13, 13, 16), (3, 3, 2)),
    # 100 bricks of 3^3, each shared by two workgroups; 216 of 2^3 likewise
    "shared": ((5, 5, 4), (13, 13, 11), (3, 3, 3)),
    "shared_small": ((4, 4, 4), (13, 13, 12), (3, 3, 3)),
}


def _pairs(pos, box, max_nb=256):
    from paper_1704_03329_amd.sim import LJSim

    sim = LJSim(pos.shape[0], box, rc=2.5, skin=0.3, precision="fp32", max_nb=max_nb)
    sim.build(*split_dev(pos))
    return sim, sim.check(raise_on_error=False)


def _check_repeated(pos, box, reps, max_nb=256):
    n = pos.shape[0]
    shifts = np.stack(np.meshgrid(*[np.arange(r) for r in reps], indexing="ij"), -1).reshape(-1, 3) * box
    big = (pos[None] + shifts[:, None]).reshape(-1, 3)
    print(n, big.shape[0], flush=True)
    sim, status = _pairs(pos, box, max_nb)
    assert status[0] == 0
    p = sim.pairs().numpy()
    want = olj.neighbour_pairs(olj.wrap(pos, box), box, olj.ext_radius_sq(2.5, 0.3))
    assert np.array_equal(np.sort(p[:, 0] * n + p[:, 1]), want[:, 0] * n + want[:, 1])
    sim_big, status = _pairs(big, box * reps, max_nb)
    assert status[0] == 0
    q = sim_big.pairs().numpy()
    # a particle's neighbours in list order, by its own index in the cell
    order = np.argsort(p[:, 0], kind="stable")
    count = np.bincount(p[:, 0], minlength=n)
    assert np.array_equal(np.bincount(q[:, 0], minlength=big.shape[0]).reshape(-1, n),
                          np.broadcast_to(count, (len(shifts), n)))
    lists = p[order, 1]
    order = np.argsort(q[:, 0], kind="stable")
    got = (q[order, 1] % n).reshape(len(shifts), -1)
    assert np.array_equal(got, np.broadcast_to(lists, got.shape))


@pytest.mark.parametrize("jitter", [0.05, 0.3])
@pytest.mark.parametrize("name", list(CASES))
def test_lists_of_a_repeated_cell(name, jitter):
    gpu_device()
    cells, sites, reps = CASES[name]
    print(name, jitter, flush=True)
    box = 2.85 * np.array(cells, dtype=float)
    g = [(np.arange(s) + 0.5) * L / s for s, L in zip(sites, box)]
    zz, yy, xx = np.meshgrid(g[2], g[1], g[0], indexing="ij")
    pos = mdinputs.perturb(np.stack([xx.ravel(), yy.ravel(), zz.ravel()], 1), jitter, 37) % box
    _check_repeated(pos, box, reps)


@pytest.mark.parametrize("extra", [150, 168, 176, 184, 192, 200, 208, 216, 260])
def test_row_lengths_about_the_tables_end(extra):
    """A crowded cell: stencil rows of about 40 + 20 + extra candidates beside
    cells of 18 - 20, up to and past the longest row that a lane takes."""
    gpu_device()
    print("extra", extra, flush=True)
    box = np.full(3, 2.85 * 6)
    g = (np.arange(16) + 0.5) * box[0] / 16
    zz, yy, xx = np.meshgrid(g, g, g, indexing="ij")
    pos = mdinputs.perturb(np.stack([xx.ravel(), yy.ravel(), zz.ravel()], 1), 0.2, 43) % box
    spot = 2.85 * (2.0 + np.random.default_rng(extra).uniform(0.02, 0.98, (extra, 3)))
    _check_repeated(np.concatenate([pos, spot]), box, (3, 3, 3), 512)


def test_capacity_of_the_last_word():
    """A capacity that is no multiple of four: exactly enough, and one short."""
    gpu_device()
    box = 2.85 * np.array([18.0, 18.0, 18.0])
    g = (np.arange(48) + 0.5) * box[0] / 48
    zz, yy, xx = np.meshgrid(g, g, g, indexing="ij")
    pos = mdinputs.perturb(np.stack([xx.ravel(), yy.ravel(), zz.ravel()], 1), 0.12, 41) % box
    x, y, z = split_dev(pos)
    wide, status = _pairs(pos, box)
    assert status[0] == 0
    p = wide.pairs().numpy()
    most = int(np.bincount(p[:, 0]).max())
    ref = torch.stack(wide.forces(x, y, z)[:3], 1)
    for cap in (most, most + 1, most + 2):
        print("capacity", cap, flush=True)
        sim, status = _pairs(pos, box, max_nb=cap)
        assert status[0] == 0
        assert np.array_equal(sim.pairs().numpy(), p)
        assert torch.equal(torch.stack(sim.forces(x, y, z)[:3], 1), ref)
    for cap in (most - 1, most - 2, most - 3):
        sim, status = _pairs(pos, box, max_nb=cap)
        assert status[0] != 0
