"""Cells of thousands of particles (no list holds them, but the sorts and the
analyses take them): the sorted order is that of a stable numpy sort, exactly,
and the bond-order sums, whose last bits follow it, are those of every repeat."""
import numpy as np
import pytest
import torch

import mdinputs
from conftest import gpu_device, split_dev
from oracle import lj as olj

pytestmark = pytest.mark.gpu

BOX = np.array([30.0, 33.0, 29.0])  # cells of side >= 2.8
# particles, crowds as (cell, particles); particles decide the radix passes
CASES = {
    "one_workgroup": (8192, {(3, 4, 5): 5000}),
    "at_the_limit": (20000, {(0, 0, 0): 4096, (1, 0, 0): 4097}),
    "two_passes": (20000, {(4, 4, 4): 9000, (5, 4, 4): 4500}),
    "three_passes": (70000, {(9, 10, 9): 60000}),
    "all_in_one": (33000, {(2, 1, 0): 33000}),
}


def _positions(n, crowds, seed):
    """Random order; the crowds anywhere in their cells, the rest anywhere in the box."""
    nc = np.floor(BOX / (2.8 * (1 + 1e-10))).astype(int)
    r = mdinputs.rng(seed)
    parts = [(np.array(c) + r.uniform(0.001, 0.999, (m, 3))) * (BOX / nc) for c, m in crowds.items()]
    parts.append(r.uniform(0.0, 1.0, (n - sum(crowds.values()), 3)) * BOX)
    pos = np.concatenate(parts)
    return pos[r.permutation(n)], nc


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("name", list(CASES))
def test_order_inside_crowded_cells(name, precision):
    """A run of no steps: the lower x half of a cell first, the caller's order inside that."""
    from paper_1704_03329_amd.sim import LJSim

    gpu_device()
    n, crowds = CASES[name]
    print(name, n, flush=True)
    pos, nc = _positions(n, crowds, 71)
    sim = LJSim(n, BOX, rc=2.5, skin=0.3, precision=precision, max_nb=64)
    vel = np.arange(3 * n, dtype=np.float64).reshape(n, 3)
    st = sim.new_state(torch.from_numpy(pos), torch.from_numpy(vel))
    sim.run(st, 0)
    q = olj.wrap(pos, BOX) * (nc / BOX)
    c = np.minimum(q.astype(int), nc - 1)
    upper = q[:, 0] - c[:, 0] >= 0.5
    key = (c[:, 2] * nc[1] + c[:, 1]) * nc[0] + c[:, 0]
    ids = st["ids"].cpu().numpy()
    assert np.array_equal(np.sort(ids), np.arange(n))
    k = key[ids]
    starts = np.concatenate([[0], np.nonzero(np.diff(k))[0] + 1])
    assert np.unique(k).size == starts.size
    cell = np.repeat(np.arange(starts.size), np.diff(np.append(starts, n)))[np.argsort(ids)]
    assert np.array_equal(ids, np.lexsort((np.arange(n), upper, cell)))
    assert np.array_equal(st["vy"].cpu().numpy(), vel[ids, 1])


@pytest.mark.parametrize("name", ["one_workgroup", "two_passes", "three_passes"])
def test_bond_order_of_crowded_cells_repeats(name):
    from paper_1704_03329_amd.sim import boa

    gpu_device()
    n, crowds = CASES[name]
    print(name, n, flush=True)
    pos, _ = _positions(n, crowds, 72)
    cols = split_dev(pos)
    # cells of the same count per axis as above
    first = boa(*cols, BOX, 2.8, q5=True)
    for _ in range(4):
        again = boa(*cols, BOX, 2.8, q5=True)
        for k in first:
            assert torch.equal(first[k], again[k]), k
