"""The sorts by cell: one workgroup (with and without its own move), the
general counting sort (its scan in one workgroup and in several) and the
radix path of sparse grids, against a stable numpy sort of the same keys.
The order is exact: cells in key order, the lower half of a cell along x
first, the caller's order inside that."""
import numpy as np
import pytest
import torch

import mdinputs
from conftest import gpu_device, split_dev
from oracle import lj as olj

pytestmark = pytest.mark.gpu

# particles, box sides (cells of side >= 2.8)
SIZES = {
    "one": (1, (9.0, 9.0, 9.0)), "small_move": (2048, (12.0, 15.0, 20.0)),
    "small_two_launches": (2049, (12.0, 15.0, 20.0)), "small_last": (8192, (20.0, 23.0, 30.0)),
    "general": (8193, (20.0, 23.0, 30.0)), "general_scan4": (40000, (40.0, 40.0, 40.0)),
    "general_scan16": (70000, (100.0, 80.0, 60.0)), "three_launch_scan": (60000, (130.0, 130.0, 120.0)),
    "radix": (300, (60.0, 60.0, 60.0)), "radix_large": (20000, (190.0, 190.0, 160.0)),
}


@pytest.mark.parametrize("name", list(SIZES))
def test_run_sorts_particles_by_cell(name):
    """A run of no steps bins and reorders the state in place."""
    from paper_1704_03329_amd.sim import LJSim

    gpu_device()
    n, box = SIZES[name]
    box = np.array(box)
    print(name, n, flush=True)
    pos = mdinputs.random_box(n, box, 61)
    pos[:: 7] += box * np.array([1.0, -1.0, 0.0])  # unfolded images
    sim = LJSim(n, box, rc=2.5, skin=0.3, precision="fp64", max_nb=256)
    vel = np.arange(3 * n, dtype=np.float64).reshape(n, 3)
    st = sim.new_state(torch.from_numpy(pos), torch.from_numpy(vel))
    sim.run(st, 0)
    w = olj.wrap(pos, box)
    nc = np.floor(box / (2.8 * (1 + 1e-10))).astype(int)
    q = w * (nc / box)
    c = np.minimum(q.astype(int), nc - 1)
    ids = st["ids"].cpu().numpy()
    assert np.array_equal(np.sort(ids), np.arange(n))
    # runs of equal cells, each cell once
    key = (c[:, 2] * nc[1] + c[:, 1]) * nc[0] + c[:, 0]
    k = key[ids]
    starts = np.concatenate([[0], np.nonzero(np.diff(k))[0] + 1])
    assert np.unique(k).size == starts.size
    # inside a cell: lower x half first, then the caller's order
    upper = q[:, 0] - c[:, 0] >= 0.5
    order = np.lexsort((np.arange(n), upper, np.repeat(np.arange(starts.size), np.diff(np.append(starts, n)))[np.argsort(ids)]))
    assert np.array_equal(ids, order)
    got = np.stack([st[a].cpu().numpy() for a in ("x", "y", "z")], 1)
    assert np.array_equal(got, w[ids])
    assert np.array_equal(st["vy"].cpu().numpy(), vel[ids, 1])


@pytest.mark.parametrize("name", ["small_last", "general", "radix", "radix_large"])
def test_build_and_analysis_after_each_sort(name):
    from paper_1704_03329_amd.sim import LJSim, boa

    gpu_device()
    n, box = SIZES[name]
    n = min(n, 8193)
    pos = mdinputs.random_box(n, box, 62)
    sim = LJSim(n, box, rc=2.5, skin=0.3, precision="fp64", max_nb=256)
    cols = split_dev(pos)
    sim.build(*cols)
    p = sim.pairs().numpy()
    want = olj.neighbour_pairs(pos, np.array(box), olj.ext_radius_sq(2.5, 0.3))
    assert np.array_equal(np.sort(p[:, 0] * n + p[:, 1]), want[:, 0] * n + want[:, 1])
    near = olj.neighbour_pairs(pos, np.array(box), 1.2 ** 2)
    got = boa(*cols, list(box), 1.2)["nnb"].cpu().numpy()
    assert np.array_equal(got, np.bincount(near[:, 0], minlength=n))
