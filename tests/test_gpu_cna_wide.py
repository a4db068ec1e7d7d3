"""Common-neighbour signatures of particles with more candidates than a lane
holds: 33 to 64 bonds (a wave per particle, in several components of the
common neighbours), more than the capacity (counted by lanes or waves, for
systems of few and of many waves), and positions up to and beyond a quarter of
the box outside it."""
import numpy as np
import pytest

import mdinputs
from conftest import gpu_device, split_dev
from oracle import boa as oboa
from oracle import cna as ocna

pytestmark = pytest.mark.gpu


def _compare(pos, box, rc, max_nb, atoms):
    from paper_1704_03329_amd.sim import cna, unpack_triplets

    atoms = [int(a) for a in atoms]
    got = {k: v.cpu().numpy() for k, v in cna(*split_dev(pos), box, rc, max_nb).items()}
    nu = oboa.bond_order(pos, box, rc, ls=(4,), rows=np.array(atoms))["nu"]
    assert np.array_equal(got["nnb"][atoms], nu)
    assert int(got["max_count"][0]) == got["nnb"].max()
    sigs, labels = ocna.cna_sampled(pos, box, rc, [i for i, k in zip(atoms, nu) if k <= max_nb])
    for i, k in zip(atoms, nu):
        if k <= max_nb:
            assert unpack_triplets(got["trip"][i][:k]) == sigs[i], i
            assert got["label"][i] == labels[i] and not got["trip"][i][k:].any(), i
        else:
            assert got["label"][i] == 0 and not got["trip"][i].any(), i
    return nu


def _wheels(spokes, size, spread, seed):
    """Two bonded particles and about their middle `spokes` clumps of `size`, each bonded to
    both, neighbouring clumps here and there: common neighbours in up to `spokes` parts."""
    r = mdinputs.rng(seed)
    a = 2.0 * np.pi * np.arange(spokes) / spokes
    hubs = np.array([[-0.25, 0.0, 0.0], [0.25, 0.0, 0.0]])
    rim = 0.8 * np.stack([np.zeros(spokes), np.cos(a), np.sin(a)], 1)
    pos = []
    for k in range(27):
        c = 4.0 * np.array([k % 3, k // 3 % 3, k // 9]) + 2.0
        arms = (rim[:, None] + r.normal(0.0, spread, (spokes, size, 3))).reshape(-1, 3)
        pos.append(c + np.concatenate([hubs, arms]) @ mdinputs.random_rotation(r).T)
    return np.concatenate(pos), np.full(3, 12.0)


BOX = np.array([9.3, 10.2, 12.1])
DENSE = mdinputs.random_box(1100, BOX, 3)
# positions, box, cutoff, capacity
CASES = {
    "about_45": (DENSE, BOX, 2.3, 64), "capacity_40": (DENSE, BOX, 2.3, 40), "counted": (DENSE, BOX, 2.3, 20),
    "capacity_32": (mdinputs.random_box(1100, BOX, 4), BOX, 1.95, 32),
    "wheels_2": (*_wheels(2, 17, 0.05, 5), 1.0, 64), "wheels_4": (*_wheels(4, 9, 0.04, 6), 1.0, 64),
    "wheels_4_wide": (*_wheels(4, 14, 0.05, 7), 1.0, 64),
}


@pytest.mark.parametrize("name", list(CASES))
def test_small_system(name):
    gpu_device()
    pos, box, rc, max_nb = CASES[name]
    print(name, len(pos), flush=True)
    nu = _compare(pos, box, rc, max_nb, range(0, len(pos), 3 if name[0] == "w" else 11))
    assert nu.max() > 32


@pytest.mark.parametrize("max_nb", [16, 32, 50, 64])
def test_many_waves(max_nb):
    """70,000 atoms: 64 of a wave; capacities on both sides of a lane's column."""
    gpu_device()
    print(max_nb, flush=True)
    box = BOX * 4.0
    pos = mdinputs.random_box(70000, box, 7)
    nu = _compare(pos, box, 2.25, max_nb, mdinputs.rng(8).choice(len(pos), 100, replace=False))
    assert nu.max() > 50 and nu.min() < 50


@pytest.mark.parametrize("rc", [1.4, 2.2])
@pytest.mark.parametrize("reach", [0.2, 0.3, 0.6])
def test_positions_outside_the_box(reach, rc):
    """Images of random positions in [-reach, 1 + reach] box edges."""
    gpu_device()
    print(reach, rc, flush=True)
    r = mdinputs.rng(int(10 * reach))
    pos = mdinputs.random_box(1100, BOX, 9)
    for k in range(3):
        up = (pos[:, k] < reach * BOX[k]) & (r.integers(0, 2, len(pos)) == 1)
        down = ~up & (pos[:, k] > (1.0 - reach) * BOX[k]) & (r.integers(0, 2, len(pos)) == 1)
        pos[:, k] += BOX[k] * (up.astype(float) - down)
    _compare(pos, BOX, rc, 64, range(0, len(pos), 3 if rc < 2 else 12))
