"""Bond screen, bond order and common-neighbour signatures on irregular
configurations against the oracle: particle counts around a wave, bond
counts from none to beyond every capacity (12, 14, 18 and 24 candidates in
registers, 64 by a wave, more only counted), positions outside the box, and
neighbours of an atom within 1e-8 of the cutoff from each other."""
import numpy as np
import pytest

import mdinputs
from conftest import gpu_device, split_dev
from oracle import boa as oboa
from oracle import cna as ocna

pytestmark = pytest.mark.gpu


def _random(n, seed, spread=False):
    L = 9.3
    pos = mdinputs.random_box(n, [L, L * 1.1, L * 1.3], seed)
    if spread:  # every third position one box further along some axis
        r = mdinputs.rng(seed + 1)
        sh = r.integers(0, 2, (n, 3)) * (np.arange(n) % 3 == 0)[:, None]
        pos = pos + sh * np.array([L, L * 1.1, L * 1.3])
    return pos, np.array([L, L * 1.1, L * 1.3])


def _at_cutoff(rc):
    """Triples (i, a, b): a and b bonded to i, |a - b| = rc (1 +- 1e-8), also
    across the faces."""
    box = np.array([24.0, 24.0, 24.0])
    r = mdinputs.rng(8)
    pos = []
    for k in range(216):
        c = 4.0 * np.array([k % 6, (k // 6) % 6, k // 36]) + 0.1
        u = mdinputs.random_rotation(r)
        d = rc * (1.0 + (1e-8 if k % 2 else -1e-8))
        h = np.sqrt((0.9 * rc) ** 2 - (0.5 * d) ** 2)
        pos += [c, c + u @ [h, 0.5 * d, 0.0], c + u @ [h, -0.5 * d, 0.0]]
    pos = np.array(pos)
    return pos - box * np.floor(pos / box), box


CASES = {
    "one": (*_random(1, 1), 2.0, 16), "63": (*_random(63, 2), 3.0, 16), "64": (*_random(64, 3), 3.0, 32),
    "65": (*_random(65, 4), 3.0, 16), "few_bonds": (*_random(1200, 5), 1.0, 14),
    "about_12": (*_random(1100, 6), 1.5, 32), "capacity_5": (*_random(1100, 6), 1.5, 5),
    "about_22": (*_random(1100, 7), 1.8, 64), "capacity_21": (*_random(1100, 7), 1.8, 21),
    "beyond_64": (*_random(1300, 8), 2.6, 64), "outside": (*_random(1000, 9, True), 1.5, 32),
    "at_cutoff": (*_at_cutoff(1.4), 1.4, 16),
}


@pytest.mark.parametrize("name", list(CASES))
def test_bonds_against_oracle(name):
    from paper_1704_03329_amd.sim import boa, cna, unpack_triplets

    gpu_device()
    pos, box, rc, max_nb = CASES[name]
    n = pos.shape[0]
    print(name, n, rc, max_nb, flush=True)
    cols = split_dev(pos)
    ref = oboa.bond_order(pos, box, rc, ls=(4, 5, 6))
    for q5 in (True, False):
        got = {k: (v.cpu().numpy() if v is not None else None) for k, v in boa(*cols, box, rc, q5=q5).items()}
        assert np.array_equal(got["nnb"], ref["nu"])
        for l, key in ((4, "q4"), (5, "q5"), (6, "q6")):
            if got[key] is not None:
                assert np.max(np.abs(got[key] - ref[l])) <= 1e-5, (l, q5)
    got = {k: v.cpu().numpy() for k, v in cna(*cols, box, rc, max_nb).items()}
    nnb = ref["nu"]
    assert np.array_equal(got["nnb"], nnb)
    assert int(got["max_count"][0]) == nnb.max()
    # the oracle's sets take their time: a sample of the atoms with many bonds
    atoms = list(range(0, n, 1 if nnb.mean() < 4 else (4 if nnb.mean() < 18 else 40)))
    sigs, labels = ocna.cna(pos, box, rc, atoms=atoms)
    for i in atoms:
        if nnb[i] <= max_nb:
            assert unpack_triplets(got["trip"][i][: nnb[i]]) == sigs[i], i
            assert not got["trip"][i][nnb[i]:].any(), i
        else:
            assert not got["trip"][i].any(), i
        if nnb[i] <= max_nb or max_nb >= 14:
            assert got["label"][i] == labels[i], i
