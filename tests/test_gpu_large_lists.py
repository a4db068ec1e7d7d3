"""List builds of 1.0 to 2.1 * 10^6 particles (a lane per particle): word
rows that 32-bit offsets just take, and longer ones; and a crowded spot where
lanes find more entries than any list holds."""
import numpy as np
import pytest
import torch

import mdinputs
from conftest import gpu_device, split_dev

pytestmark = pytest.mark.gpu


def _export(sim):
    """The pairs in list order on the GPU (int64, a 2^21-particle list does not travel)."""
    from paper_1704_03329_amd import mdpl as C

    total = C.mdpl_nlist_export(sim.handle, None, None, 0)
    i, j = (torch.empty(total, dtype=torch.int32, device="cuda") for _ in range(2))
    C.mdpl_nlist_export(sim.handle, i, j, total)
    return i.long(), j.long()


def _runs(i):
    """Of every pair its rank in the list of its first particle."""
    start = torch.ones_like(i, dtype=torch.bool)
    start[1:] = i[1:] != i[:-1]
    first = torch.nonzero(start)[:, 0]
    return torch.arange(i.numel(), device="cuda") - first[torch.cumsum(start, 0) - 1]


# particles of the cell that is repeated 512 times, its sides in cells of 2.85
CELLS = {"last_32_bit": (2076, (6, 6, 3)), "first_64_bit": (2077, (6, 6, 3)), "rows_of_2^24": (4096, (6, 6, 6))}


@pytest.mark.parametrize("name", list(CELLS))
def test_lists_on_both_sides_of_the_offset_rule(name):
    from paper_1704_03329_amd.sim import LJSim

    gpu_device()
    n, cells = CELLS[name]
    print("particles", 512 * n, flush=True)
    box = 2.85 * np.array(cells, dtype=float)
    g = [(np.arange(m) + 0.5) * s / m for m, s in zip((16, 16, 16 if cells[2] == 6 else 9), box)]
    zz, yy, xx = np.meshgrid(g[2], g[1], g[0], indexing="ij")
    pos = mdinputs.perturb(np.stack([xx.ravel(), yy.ravel(), zz.ravel()], 1)[:n], 0.25, 47) % box
    small = LJSim(n, box, max_nb=256)
    small.build(*split_dev(pos))
    assert small.check(raise_on_error=False)[0] == 0
    i, j = _export(small)
    lists = torch.full((n, 256), -1, dtype=torch.int64, device="cuda")
    lists[i, _runs(i)] = j
    r = [torch.arange(8, device="cuda", dtype=torch.float64) * L for L in box]
    shift = torch.stack(torch.meshgrid(*r, indexing="ij"), -1).reshape(-1, 1, 3)
    big = (torch.from_numpy(pos).cuda()[None] + shift).reshape(-1, 3)
    sim = LJSim(512 * n, 8 * box, max_nb=256)
    sim.build(*[big[:, k].contiguous() for k in range(3)])
    assert sim.check(raise_on_error=False)[0] == 0
    p, q = _export(sim)
    assert p.numel() == 512 * i.numel()
    assert torch.equal(lists[p % n, _runs(p)], q % n)


@pytest.mark.parametrize("nc", [(44, 45, 44), (56, 56, 55)])
def test_more_entries_than_any_list_holds(nc):
    """27 cells of 64 particles huddled about the middle one, the other cells
    with 12 each: 1727 neighbours where a list holds 1024 at most.  The flag
    and the largest count say so, and the lists of all others are whole (a
    pair is in the lists of both its particles)."""
    from paper_1704_03329_amd import mdpl as C
    from paper_1704_03329_amd.sim import LJSim

    gpu_device()
    side, mid = 2.85, 30
    site = np.stack(np.meshgrid([0.25, 0.75], [0.25, 0.75], [1 / 6, 0.5, 5 / 6], indexing="ij"), -1).reshape(-1, 3)
    c = np.stack(np.meshgrid(*[np.arange(k) for k in nc], indexing="ij"), -1).reshape(-1, 1, 3)
    crowded = np.all(np.abs(c[:, 0] - mid) <= 1, axis=1)
    rng = np.random.default_rng(53)
    pos = (c[~crowded] + site + rng.uniform(-0.05, 0.05, (np.count_nonzero(~crowded), 12, 3))).reshape(-1, 3) * side
    off = c[crowded, 0] - mid
    at = (mid + 0.5) * side + off * (0.5 * side + 0.05)
    spot = at[:, None] + rng.uniform(-0.02, 0.02, (27, 64, 3))
    full = np.repeat(np.abs(off).sum(1) <= 1, 64)  # the middle and its face neighbours: more than 1024
    n0 = pos.shape[0]
    pos = np.concatenate([pos, spot.reshape(-1, 3)])
    n = pos.shape[0]
    print("particles", n, flush=True)
    sim = LJSim(n, np.array(nc) * side, max_nb=1024)
    sim.build(*split_dev(pos))
    status, flags, most = sim.check(raise_on_error=False)
    assert status == C.MDPL_ECAPACITY and flags & C.FLAG_NL_OVERFLOW and most == 27 * 64 - 1
    cut = torch.zeros(n, dtype=torch.bool, device="cuda")
    cut[n0:] = torch.from_numpy(full).cuda()
    i, j = _export(sim)
    keep = ~(cut[i] | cut[j])
    i, j = i[keep], j[keep]
    g = torch.Generator(device="cuda").manual_seed(3)
    a, b = (torch.randint(-2**62, 2**62, (n,), device="cuda", generator=g) for _ in range(2))
    assert int((a[i] * b[j] - a[j] * b[i]).sum()) == 0
    assert int(torch.bincount(i, minlength=n)[:n0].min()) > 12
