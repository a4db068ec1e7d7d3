"""Bonds where FP32 copies of the positions cannot screen the candidates:
positions 10^10 boxes away, whose folding rounds by more than the FP32 copy
does, and cutoffs whose squares FP32 does not hold.  The definition's FP64
test decides, as everywhere."""
import numpy as np
import pytest

import mdinputs
from conftest import gpu_device, split_dev
from oracle import boa as oboa
from oracle import cna as ocna

pytestmark = pytest.mark.gpu


def _check(pos, box, rc, max_nb=64):
    from paper_1704_03329_amd.sim import boa, cna, unpack_triplets

    n = pos.shape[0]
    nu = oboa.bond_order(pos, box, rc, ls=(4,))["nu"]
    assert nu.max() > 0
    cols = split_dev(pos)
    for q5 in (True, False):
        assert np.array_equal(boa(*cols, box, rc, q5=q5)["nnb"].cpu().numpy(), nu)
    got = {k: v.cpu().numpy() for k, v in cna(*cols, box, rc, max_nb).items()}
    assert np.array_equal(got["nnb"], nu)
    atoms = list(range(0, n, max(1, n // 300)))
    sigs, labels = ocna.cna(pos, box, rc, atoms=atoms)
    for i in atoms:
        assert unpack_triplets(got["trip"][i][: nu[i]]) == sigs[i], i
        assert got["label"][i] == labels[i], i


@pytest.mark.parametrize("axis", [0, 1, 2])
def test_positions_far_outside_the_box(axis):
    """Pairs just inside the cutoff, one on either side of a face of a far image."""
    gpu_device()
    L = 17.0 + 0.95 * 2.0 ** -14  # L k is rounded to multiples of 2^-14
    box = np.full(3, L)
    k = np.arange(2 ** 34, 2 ** 34 + 200, dtype=np.float64)
    widened = L - (L * k - L * (k - 1.0))  # by which folding parts the two
    k = k[np.argmax(widened)]
    ulp = np.spacing(L * k)
    d = 6000 * ulp  # 0.37
    assert widened.max() > 0.9 * ulp
    rc = d * (1.0 + 1e-9)
    r = mdinputs.rng(97)
    grid = np.stack(np.meshgrid(np.arange(17), np.arange(17), indexing="ij"), -1).reshape(-1, 2) + 0.5
    m = grid.shape[0]
    pos = np.empty((2 * m, 3))
    a = L * k - ulp * r.integers(1000, 5000, m)
    other = [q for q in range(3) if q != axis]
    pos[0::2, axis], pos[1::2, axis] = a, a + d
    pos[0::2, other] = pos[1::2, other] = grid
    _check(pos, box, rc)


@pytest.mark.parametrize("scale", [1e-22, 1e-18, 1e-10, 1e17, 1e20])
def test_units_beyond_fp32(scale):
    gpu_device()
    print(scale, flush=True)
    box = np.array([9.3, 10.2, 12.1])
    pos = mdinputs.random_box(1100, box, 98)
    _check(pos * scale, box * scale, 1.5 * scale)
