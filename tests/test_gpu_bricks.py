"""Bricks shared by several workgroups (small systems): the list build with
9, 3 and 1 waves per home cell and the force and descriptor passes with 8,
2 and 1 parts per brick, against the oracle at the bars of test_gpu_lj.py
and test_gpu_potential.py."""
import numpy as np
import pytest
import torch

import mdinputs
from conftest import force_errors, gpu_device, split_dev
from oracle import descriptor as OD
from oracle import lj as olj

pytestmark = pytest.mark.gpu

# jittered grids (sites per axis, spacing): cells of side >= 2.8 per axis -> bricks
GRIDS = {
    "5x5x4_cells": ((14, 14, 12), 1.03),     # 2^3 bricks, 18 of them: 8 parts, 9 waves per cell
    "10x10x10_cells": ((14, 14, 14), 2.05),  # 64 bricks of 3^3: 8 parts, 4 cells of 3 waves each
    "13x7x10_cells": ((18, 10, 14), 2.05),   # 60 bricks, partial ones along x and z
    "17x17x17_cells": ((24, 24, 24), 2.05),  # 216 bricks: 2 parts, one wave per cell
}


@pytest.mark.parametrize("name", list(GRIDS))
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_shared_bricks(name, precision):
    from paper_1704_03329_amd.sim import LJSim

    gpu_device()
    reps, a = GRIDS[name]
    g = [(np.arange(r) + 0.5) * a for r in reps]
    zz, yy, xx = np.meshgrid(g[2], g[1], g[0], indexing="ij")
    pos = mdinputs.perturb(np.stack([xx.ravel(), yy.ravel(), zz.ravel()], 1), 0.06 * a, 31)
    box = np.array(reps, dtype=float) * a
    n = pos.shape[0]
    print(name, precision, n, flush=True)
    sim = LJSim(n, box, rc=2.5, skin=0.3, precision=precision, shift="cutoff")
    x, y, z = split_dev(pos)
    sim.build(x, y, z)
    assert sim.check(raise_on_error=False)[0] == 0
    p = sim.pairs().numpy()
    key = np.sort(p[:, 0] * n + p[:, 1])
    want = olj.neighbour_pairs(olj.wrap(pos, box), box, olj.ext_radius_sq(2.5, 0.3))
    assert np.array_equal(key, want[:, 0] * n + want[:, 1])
    ref = olj.lj_forces(pos, box, 2.5, shift="cutoff")
    fx, fy, fz, pe_w, e = sim.forces(x, y, z, energy=True, per_atom=True)
    plain = torch.stack(sim.forces(x, y, z)[:3], 1)
    F = torch.stack([fx, fy, fz], 1)
    assert torch.equal(F, plain)  # the energy pass forms the plain pass's forces
    assert max(force_errors(F.double().cpu().numpy(), ref["F"])) <= 1e-5
    assert abs(pe_w[0].item() - ref["pe"]) <= 1e-9 * abs(ref["pe"])
    assert abs(pe_w[1].item() - ref["w"]) <= 1e-9 * abs(ref["w"]) + 1e-9 * abs(ref["pe"])
    assert np.max(np.abs(e.cpu().numpy() - ref["e"])) <= 1e-9 * np.max(np.abs(ref["e"]))
    # descriptors of sampled particles, and the sum rule of the backward's forces
    from paper_1704_03329_amd import potential as P

    G = torch.empty((n, 24), dtype=torch.float32, device="cuda")
    mom = torch.empty((n, 50), dtype=torch.float32, device="cuda")
    P.mdpl_desc_fwd(sim, x, y, z, G, mom)
    rows = np.arange(0, n, max(1, n // 60))
    want = OD.descriptors(pos, box, rows)
    got = G.double().cpu().numpy()[rows]
    assert np.linalg.norm(got - want) <= 1e-5 * np.linalg.norm(want)
    dEdG = torch.sin(torch.arange(n * 24, device="cuda", dtype=torch.float32)).view(n, 24).contiguous()
    f = [torch.empty(n, dtype=torch.float32, device="cuda") for _ in range(3)]
    P.mdpl_desc_bwd(sim, x, y, z, dEdG, mom, *f)
    if n <= 3000:
        _, table, grads = OD.descriptors(pos, box, with_grad=True)
        Fd = OD.forces_from_feature_grad(n, np.arange(n), table, grads, dEdG.double().cpu().numpy())
        got = torch.stack(f, 1).double().cpu().numpy()
        assert np.linalg.norm(got - Fd) <= 1e-4 * np.linalg.norm(Fd)


# (sites per axis, spacing): a wave per particle in the descriptor passes
WAVES = {
    "up_to_130_in_range": ((10, 10, 12), 0.85),     # several rounds of 64 neighbours
    "several_batches": ((23, 23, 23), 1.12),         # 27 bricks in 8 parts of about 56
    "one_part_per_brick": ((23, 22, 27), 1.9),       # 150 bricks of about 90
    "6_sites_per_part": ((9, 10, 9), 1.07),          # 8 bricks in 32 parts, the last ones empty
}


@pytest.mark.parametrize("name", list(WAVES))
def test_wave_per_particle(name):
    from paper_1704_03329_amd import potential as P
    from paper_1704_03329_amd.sim import LJSim

    gpu_device()
    reps, a = WAVES[name]
    g = [(np.arange(r) + 0.5) * a for r in reps]
    zz, yy, xx = np.meshgrid(g[2], g[1], g[0], indexing="ij")
    pos = mdinputs.perturb(np.stack([xx.ravel(), yy.ravel(), zz.ravel()], 1), 0.06 * a, 33)
    box = np.array(reps, dtype=float) * a
    n = pos.shape[0]
    print(name, n, flush=True)
    sim = LJSim(n, box, rc=2.5, skin=0.3, precision="fp32", max_nb=256)
    x, y, z = split_dev(pos)
    sim.build(x, y, z)
    assert sim.check(raise_on_error=False)[0] == 0
    G = torch.empty((n, 24), dtype=torch.float32, device="cuda")
    mom = torch.empty((n, 50), dtype=torch.float32, device="cuda")
    P.mdpl_desc_fwd(sim, x, y, z, G, mom)
    # sampled rows against the oracle at the bars above; the forces of a
    # gradient that only these rows have, with their neighbours' reactions
    rows = np.arange(0, n, max(1, n // 400))
    want, table, grads = OD.descriptors(pos, box, rows, with_grad=True)
    got = G.double().cpu().numpy()[rows]
    assert np.linalg.norm(got - want) <= 1e-5 * np.linalg.norm(want)
    dEdG = torch.zeros((n, 24), dtype=torch.float32, device="cuda")
    dEdG[torch.as_tensor(rows, device="cuda")] = torch.sin(
        torch.arange(len(rows) * 24, device="cuda", dtype=torch.float32)).view(-1, 24)
    f = [torch.empty(n, dtype=torch.float32, device="cuda") for _ in range(3)]
    P.mdpl_desc_bwd(sim, x, y, z, dEdG, mom, *f)
    Fd = OD.forces_from_feature_grad(n, rows, table, grads, dEdG.double().cpu().numpy()[rows])
    got = torch.stack(f, 1).double().cpu().numpy()
    assert np.linalg.norm(got - Fd) <= 1e-4 * np.linalg.norm(Fd)
