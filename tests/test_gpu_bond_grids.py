"""Bonds in the largest grid that the analyses take: 2^30 cells, whose table of
first slots is one entry longer than 32-bit byte offsets reach."""
import numpy as np
import pytest

import mdinputs
from conftest import gpu_device, split_dev
from oracle import boa as oboa
from oracle import cna as ocna

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sides", [(1024, 1024, 1024), (4096, 512, 512)])
def test_bonds_in_the_last_cells(sides):
    """A cluster about the box corner (the last row of cells, its images
    across the faces among them) in a sparse background."""
    from paper_1704_03329_amd.sim import boa, cna, unpack_triplets

    gpu_device()
    print(sides, flush=True)
    box, rc = np.array(sides, dtype=float), 1.0 - 1e-5
    assert np.array_equal(np.floor(box / (rc * (1 + 1e-10))), sides)
    r = mdinputs.rng(29)
    m = 300
    pos = np.concatenate([r.uniform(-2.0, 1.5, (m, 3)) % box, r.uniform(0.0, 1.0, (30000, 3)) * box])
    rows = np.arange(m)
    ref = oboa.bond_order(pos, box, rc, ls=(4, 6), rows=rows)
    last = np.all(pos[:m] >= box - 1.0, axis=1)
    assert last.sum() > 3 and ref["nu"][last].min() > 0
    cols = split_dev(pos)
    got = {k: v.cpu().numpy() for k, v in boa(*cols, box, rc).items() if v is not None}
    assert np.array_equal(got["nnb"][:m], ref["nu"])
    assert np.max(np.abs(got["q4"][:m] - ref[4])) <= 1e-5 and np.max(np.abs(got["q6"][:m] - ref[6])) <= 1e-5
    got = {k: v.cpu().numpy() for k, v in cna(*cols, box, rc, 64).items()}
    assert np.array_equal(got["nnb"][:m], ref["nu"])
    sigs, labels = ocna.cna_sampled(pos, box, rc, rows.tolist())
    for i in range(m):
        assert unpack_triplets(got["trip"][i][: ref["nu"][i]]) == sigs[i], i
        assert got["label"][i] == labels[i], i
