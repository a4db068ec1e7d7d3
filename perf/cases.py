"""Timed cases of the library: what a program that uses it spends its time on.

The cases go through the public entry points (LJSim, lj_energy, MLPPotential,
boa, cna) at the sizes of the tests, the benchmark and the README, from the
1000-particle check to the 10^6-particle fluid and the 4*10^6-atom
polycrystal, with box shapes and particle counts that do not divide evenly
among the drawn ones.  Kinds:

  md        velocity Verlet from a lattice with thermal motion (LJSim.run)
  energy    lj_energy and its gradient through torch autograd
  snapshot  training targets of one configuration: list, FP64 forces and
            per-atom energies, then list and descriptors
  potential one force evaluation of the learned potential on new positions
  train     Adam steps on random batches (MLPPotential.train)
  boa, cna  structure analysis of a polycrystal

`exact` evaluates the same quantities with plain torch in float64.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import mdinputs
from paper_1704_03329_amd import potential as P
from paper_1704_03329_amd.autograd import lj_energy
from paper_1704_03329_amd.sim import LJSim, boa, cna

DEV = "cuda"
RHO = mdinputs.LJ_RHO
RC, SKIN = 2.5, 0.3
BOND = 1.2684 * (math.sqrt(2.0)) ** (1.0 / 3.0)  # first-shell cutoff of the crystals at density 1
GRAINS = 50
ROWS = 80_000  # rows of the training set of a "train" case
LR = 1e-3


# ------------------------------------------------------------------ cases
def listed():
    def cube(name, kind, side, **kw):
        return {"name": name, "kind": kind, "nx": side, "ny": side, "nz": side, **kw}

    return [
        # the README's small check: a short FP64 run, launches and latency count
        cube("md_n1000_fp64", "md", 10, precision="fp64", steps=100, sample=10),
        # a stretch of training-data generation (FP64, N about 4000, thermo every 10 steps)
        cube("md_n4096_fp64", "md", 16, precision="fp64", steps=50, sample=10),
        # the crystallisation run: 125,000 particles, rc 3, Andersen bath, lists kept 18 steps
        cube("md_andersen_n125k", "md", 50, precision="fp32", steps=36, sample=18, andersen=True),
        # the benchmark fluid: 10^6 particles, FP32 pair forces, energies every 10 steps
        cube("md_n1m_fp32", "md", 100, precision="fp32", steps=20, sample=10),
        # energy and gradient behind a torch optimiser or a loss
        cube("energy_grad_n32k_fp64", "energy", 32, precision="fp64"),
        # one labelled training configuration
        cube("snapshot_n4096", "snapshot", 16),
        # the learned potential on a training-sized and on the benchmark's evaluation configuration
        cube("potential_n4096", "potential", 16),
        cube("potential_n262k", "potential", 64),
        # training: 16 Adam steps at the benchmark's batch size
        {"name": "train_b4096", "kind": "train", "batch": 4096, "steps": 16},
        # bond order while a run proceeds, and of the benchmark's polycrystal
        {"name": "boa_n125k", "kind": "boa", "n": 125_000, "q5": True},
        {"name": "boa_n4m", "kind": "boa", "n": 4_000_000, "q5": False},
        # common-neighbour analysis of the benchmark's polycrystal
        {"name": "cna_n4m", "kind": "cna", "n": 4_000_000, "max_nb": 32},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _sides(rng, lo, hi):
    """Lattice sides of about lo^3 .. hi^3 particles, not always a cube."""
    s = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    a, b = rng.choice([(1.0, 1.0), (0.8, 1.2), (1.15, 0.95), (0.9, 0.9)])
    return {"nx": min(hi, max(9, round(s * a))), "ny": min(hi, max(9, round(s * b))), "nz": min(hi, max(9, round(s / (a * b))))}


def draw(rng):
    kind = rng.choice(["md", "md", "md", "energy", "snapshot", "potential", "train", "boa", "cna"])
    if kind == "md":
        how = rng.choice(["fp64", "fp32", "andersen"])
        if how == "andersen":
            return {"kind": kind, **_sides(rng, 16, 50), "precision": "fp32", "steps": rng.randint(18, 36), "sample": 18,
                    "andersen": True}
        steps = rng.randint(10, 100)
        side = _sides(rng, 10, 40 if how == "fp64" else 64)
        return {"kind": kind, **side, "precision": how, "steps": steps, "sample": rng.choice([0, 5, 10])}
    if kind == "energy":
        return {"kind": kind, **_sides(rng, 10, 40), "precision": rng.choice(["fp64", "fp32"])}
    if kind == "snapshot":
        return {"kind": kind, **_sides(rng, 10, 24)}
    if kind == "potential":
        return {"kind": kind, **_sides(rng, 12, 56)}
    if kind == "train":
        return {"kind": kind, "batch": _log_int(rng, 256, 8192), "steps": rng.randint(4, 16)}
    if kind == "boa":
        return {"kind": kind, "n": _log_int(rng, 8_000, 2_000_000), "q5": rng.random() < 0.5}
    return {"kind": kind, "n": _log_int(rng, 8_000, 2_000_000), "max_nb": rng.choice([16, 32])}


# ------------------------------------------------------------------ inputs
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 7919 + 11)


def _fluid(case, seed):
    """Positions and velocities (N, 3): simple-cubic sites at the fluid's
    density with a thermal displacement of about 0.08 sigma per component
    (bounded, so that no pair overlaps), T* = 1."""
    g = _gen(seed)
    side = (case["nx"], case["ny"], case["nz"])
    a = RHO ** (-1.0 / 3.0)
    axes = [(torch.arange(s, device=DEV, dtype=torch.float64) + 0.5) * a for s in side]
    zz, yy, xx = torch.meshgrid(axes[2], axes[1], axes[0], indexing="ij")
    pos = torch.stack([xx.reshape(-1), yy.reshape(-1), zz.reshape(-1)], 1)
    n = pos.shape[0]
    pos = pos + (torch.rand(n, 3, device=DEV, dtype=torch.float64, generator=g) - 0.5) * 0.28
    vel = torch.randn(n, 3, device=DEV, dtype=torch.float64, generator=g)
    vel = vel - vel.mean(0, keepdim=True)
    return pos, vel, [s * a for s in side]


def _lattice(phase, half):
    """Points of one crystal phase (fcc, hcp, bcc at density 1) around the origin."""
    d = math.sqrt(2.0) ** (1.0 / 3.0)
    if phase == 0:
        cell = [d * math.sqrt(2.0)] * 3
        basis = [[0, 0, 0], [0.5, 0.5, 0], [0.5, 0, 0.5], [0, 0.5, 0.5]]
    elif phase == 1:
        cell = [d, d * math.sqrt(3.0), d * math.sqrt(8.0 / 3.0)]
        basis = [[0, 0, 0], [0.5, 0.5, 0], [0.5, 1 / 6, 0.5], [0, 2 / 3, 0.5]]
    else:
        cell = [2.0 ** (1.0 / 3.0)] * 3
        basis = [[0, 0, 0], [0.5, 0.5, 0.5]]
    m = [int(math.ceil(half / c)) + 1 for c in cell]
    ax = [torch.arange(-k, k + 1, device=DEV, dtype=torch.float64) for k in m]
    g = torch.stack(torch.meshgrid(*ax, indexing="ij"), -1).reshape(-1, 1, 3)
    b = torch.tensor(basis, device=DEV, dtype=torch.float64)
    return ((g + b).reshape(-1, 3)) * torch.tensor(cell, device=DEV, dtype=torch.float64)


def _polycrystal(n, seed):
    """Exactly n atoms of a periodic Voronoi polycrystal (fcc, hcp and bcc
    grains, random orientations, thermal jitter, about 1 % vacancies)."""
    g = _gen(seed)
    ng = max(4, min(GRAINS, n // 2000))
    L = n ** (1.0 / 3.0)
    while True:
        full = 1.02 * n
        scale = L / full ** (1.0 / 3.0)  # generated at density 1 in a larger box, then scaled
        Lg = L / scale
        seeds = torch.rand(ng, 3, device=DEV, dtype=torch.float64, generator=g) * Lg
        q, r = torch.linalg.qr(torch.randn(ng, 3, 3, dtype=torch.float64, device=DEV, generator=g).cpu())
        rot = (q * torch.sign(torch.diagonal(r, dim1=1, dim2=2))[:, None, :]).to(DEV)

        def owner(p):
            best, own = None, None
            for k in range(ng):
                d = p - seeds[k]
                d = d - Lg * torch.round(d / Lg)
                d2 = (d * d).sum(1)
                if best is None:
                    best, own = d2, torch.zeros(p.shape[0], dtype=torch.int64, device=DEV)
                else:
                    own = torch.where(d2 < best, k, own)
                    best = torch.minimum(best, d2)
            return own, best

        m = 32
        ax = (torch.arange(m, device=DEV, dtype=torch.float64) + 0.5) * (Lg / m)
        probe = torch.stack(torch.meshgrid(ax, ax, ax, indexing="ij"), -1).reshape(-1, 3)
        own, d2 = owner(probe)
        reach = torch.zeros(ng, dtype=torch.float64, device=DEV).scatter_reduce_(0, own, d2.sqrt(), "amax")
        reach = (reach + 2.0 * Lg / m + 2.5).cpu().tolist()
        parts = []
        for k in range(ng):
            p = _lattice(k % 3, reach[k])
            p = p[(p * p).sum(1) <= reach[k] ** 2] @ rot[k].T + seeds[k]
            p = p - Lg * torch.floor(p / Lg)
            parts.append(p[owner(p)[0] == k])
        pos = torch.cat(parts)
        if pos.shape[0] >= n:
            break
    keep = torch.randperm(pos.shape[0], device=DEV, generator=g)[:n].sort().values
    pos = pos[keep] * scale
    pos = pos + torch.randn(n, 3, device=DEV, dtype=torch.float64, generator=g) * (0.05 * 1.1225)
    pos = pos - L * torch.floor(pos / L)
    return torch.where(pos >= L, pos - L, pos), [L, L, L]


def _sample_stats():
    """Mean and spread of the descriptors and the energies of a small fluid
    configuration (the standardisation a trained model carries)."""
    pos, _, box = _fluid({"nx": 9, "ny": 9, "nz": 9}, 0)
    G = _features(*_neighbours(pos, box, RC, 0, pos.shape[0], 128))
    return G.mean(0).float(), G.std(0).float() + 1e-6


_STATS = []


def _model(seed):
    if not _STATS:
        _STATS.append(_sample_stats())
    model = P.MLPPotential(seed=int(seed) % 1_000_003, device=DEV)
    model.mu.copy_(_STATS[0][0])
    model.sd.copy_(_STATS[0][1])
    model.e_mean, model.e_sd = -5.2, 0.6
    return model


def _training(case, seed):
    """Features and energies of a training set, and a model some way into
    its training (Adam moments of the gradients' size)."""
    g = _gen(seed)
    mu, sd = _model(seed).mu, _STATS[0][1]
    z = torch.randn(ROWS, 24, device=DEV, generator=g)
    z = z + 0.7 * torch.randn(ROWS, 1, device=DEV, generator=g)
    G = (mu + sd * z).contiguous()
    w = torch.randn(24, device=DEV, generator=g)
    e = (-5.2 + 0.1 * (z @ w) + 0.02 * (z[:, :12] ** 2).sum(1)).double()
    m = 1e-3 * torch.randn(P.NPARAM, device=DEV, generator=g)
    v = 1e-5 * (0.5 + torch.rand(P.NPARAM, device=DEV, generator=g))
    pad = torch.zeros(64, 32, dtype=torch.bool, device=DEV)
    pad[:, 24:] = True
    m[:2048][pad.reshape(-1)] = 0
    v[:2048][pad.reshape(-1)] = 0
    return G, e, m, v


def prepare(case, seed):
    kind = case["kind"]
    if kind == "train":
        G, e, m, v = _training(case, seed)
        model = _model(seed)
        model.m.copy_(m)
        model.v.copy_(v)
        model.step = 100
        return {"case": case, "model": model, "G": G, "e": e, "seed": int(seed) % 100_003}
    if kind in ("boa", "cna"):
        pos, box = _polycrystal(case["n"], seed)
        return {"case": case, "x": pos[:, 0].contiguous(), "y": pos[:, 1].contiguous(), "z": pos[:, 2].contiguous(),
                "box": box}
    pos, vel, box = _fluid(case, seed)
    n = pos.shape[0]
    if kind == "md":
        cryst = case.get("andersen", False)
        sim = LJSim(n, box, rc=3.0 if cryst else RC, skin=SKIN, dt=0.001, reuse_every=18 if cryst else 10,
                    shift="cutoff", precision=case["precision"], max_nb=256 if cryst else 128, rebuild="vmax")
        bath = {"temperature": 0.01, "collision_rate": 10.0, "seed": 1, "step0": 0} if cryst else None
        return {"case": case, "sim": sim, "st": sim.new_state(pos, vel), "bath": bath}
    if kind == "energy":
        sim = LJSim(n, box, rc=RC, skin=SKIN, shift="cutoff", precision=case["precision"])
        return {"case": case, "sim": sim, "pos": pos.requires_grad_(True)}
    if kind == "snapshot":
        return {"case": case, "sim": LJSim(n, box, rc=RC, skin=SKIN, precision="fp64"), "pos": pos}
    model = _model(seed)
    return {"case": case, "sim": LJSim(n, box, rc=RC, skin=SKIN, precision="fp32"), "model": model,
            "x": pos[:, 0].contiguous(), "y": pos[:, 1].contiguous(), "z": pos[:, 2].contiguous(),
            "buf": model.buffers(n)}


# ------------------------------------------------------------------ one pass
def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "md":
        st, bath = state["st"], state["bath"]
        thermo = state["sim"].run(st, case["steps"], case["sample"], andersen=bath)
        if bath is not None:
            bath["step0"] += case["steps"]
        return {**st, "thermo": thermo}
    if kind == "energy":
        e = lj_energy(state["pos"], state["sim"])
        (g,) = torch.autograd.grad(e, state["pos"])
        return {"e": e, "grad": g}
    if kind == "snapshot":
        e, F = P.lj_snapshot_targets(state["sim"], state["pos"])
        return {"e": e, "F": F, "G": P.descriptors(state["sim"], state["pos"])}
    if kind == "potential":
        x, y, z = state["x"], state["y"], state["z"]
        state["sim"].build(x, y, z)
        e, fx, fy, fz = state["model"].forces(state["sim"], x, y, z, state["buf"])
        return {"e": e, "fx": fx, "fy": fy, "fz": fz}
    if kind == "train":
        model = state["model"]
        model.train(state["G"], state["e"], case["steps"], batch=case["batch"], lr=LR, seed=state["seed"])
        return {"params": model.params, "m": model.m, "v": model.v}
    if kind == "boa":
        return boa(state["x"], state["y"], state["z"], state["box"], BOND, q5=case["q5"])
    return cna(state["x"], state["y"], state["z"], state["box"], BOND, max_nb=case["max_nb"])


# ------------------------------------------------------------------ least work
def work(case):
    kind = case["kind"]
    if kind == "train":
        b, s = case["batch"], case["steps"]
        # features, index and target of the batch; parameters and both moments read and written
        return {"bytes": s * (b * (96 + 4 + 8) + P.NPARAM * 4 * 6), "flops": s * b * 6 * (24 * 64 + 64 * 64 + 64)}
    if kind == "boa":
        n, nb = case["n"], 13.0
        return {"bytes": n * (24 + 4 * (4 if case["q5"] else 3)), "flops": n * nb * (10 + (150 if case["q5"] else 110))}
    if kind == "cna":
        n, nb = case["n"], 13.0
        return {"bytes": n * (24 + 4 * nb + 4 + 1), "flops": n * (nb * 10 + 0.5 * nb * nb * 8)}
    n = case["nx"] * case["ny"] * case["nz"]
    nb = RHO * 4.0 / 3.0 * math.pi * (3.0 if case.get("andersen") else RC) ** 3
    fb = 8 if case.get("precision", "fp64") == "fp64" else 4
    if kind == "md":  # every step: positions and velocities read and written; each pair once
        steps = case["steps"]
        return {"bytes": n * (steps * 96 + 2 * 3 * fb + 8), "flops": n * steps * (0.5 * nb * 22 + 18)}
    if kind == "energy":
        return {"bytes": n * (24 + 24) + 8, "flops": n * 0.5 * nb * 25}
    if kind == "snapshot":
        return {"bytes": n * (24 + 24 + 8 + 96), "flops": n * (0.5 * nb * 25 + nb * 130)}
    # descriptors and their backward per ordered pair, the network per atom
    return {"bytes": n * (24 + 12 + 4), "flops": n * (nb * (130 + 220) + 2 * 2 * (24 * 64 + 64 * 64 + 64))}


# ------------------------------------------------------------------ 64-bit values
class _Cells:
    """Padded cell table of a periodic configuration (cells of side >= r)."""

    def __init__(self, pos, box, r):
        self.pos, self.L = pos, torch.tensor(box, device=DEV, dtype=torch.float64)
        self.nc = [max(1, int(math.floor(b / (r * (1 + 1e-9))))) for b in box]
        if min(self.nc) < 3:
            self.nc = [1, 1, 1]
        nct = torch.tensor(self.nc, device=DEV)
        w = pos - self.L * torch.floor(pos / self.L)
        self.c = torch.minimum((w / self.L * nct).long(), nct - 1)
        key = (self.c[:, 2] * self.nc[1] + self.c[:, 1]) * self.nc[0] + self.c[:, 0]
        order = torch.argsort(key, stable=True)
        count = torch.bincount(key, minlength=math.prod(self.nc))
        start = torch.cumsum(count, 0) - count
        self.table = torch.full((math.prod(self.nc), int(count.max())), -1, dtype=torch.int64, device=DEV)
        self.table[key[order], torch.arange(pos.shape[0], device=DEV) - start[key[order]]] = order

    def candidates(self, i0, i1):
        """(i1 - i0, M) candidate partners, -1 for none."""
        out = []
        for oz in (-1, 0, 1):
            for oy in (-1, 0, 1):
                for ox in (-1, 0, 1):
                    if self.nc == [1, 1, 1] and (ox or oy or oz):
                        continue
                    c = [(self.c[i0:i1, k] + o) % self.nc[k] for k, o in enumerate((ox, oy, oz))]
                    out.append(self.table[(c[2] * self.nc[1] + c[1]) * self.nc[0] + c[0]])
        return torch.cat(out, 1)


def _neighbours(pos, box, rc, i0, i1, most, cells=None):
    """Padded separations u = r_j - r_i, partners j and mask of atoms i0 .. i1 within rc."""
    cells = cells or _Cells(pos.detach(), box, rc)
    cand = cells.candidates(i0, i1)
    ri = pos.detach()[i0:i1, None, :]
    d = pos.detach()[cand.clamp(min=0)] - ri
    d = d - cells.L * torch.round(d / cells.L)
    d2 = (d * d).sum(2)
    ok = (cand >= 0) & (cand != torch.arange(i0, i1, device=DEV)[:, None]) & (d2 < rc * rc)
    k = min(most, cand.shape[1])
    _, at = torch.topk(torch.where(ok, d2, math.inf), k, dim=1, largest=False)
    j, ok = cand.gather(1, at).clamp(min=0), ok.gather(1, at)
    u = pos[j] - pos[i0:i1, None, :]
    u = u - cells.L * torch.round(u.detach() / cells.L)
    return torch.where(ok[..., None], u, torch.ones_like(u)), j, ok


def _features(u, j, ok):
    r = (u * u).sum(-1).sqrt()
    fc = torch.where(ok, 0.5 * (torch.cos(math.pi * r / RC) + 1.0), torch.zeros_like(r))
    out = [(torch.exp(-((r - (0.85 + 0.11 * k)) ** 2) / (2 * 0.11 ** 2)) * fc).sum(1) for k in range(16)]
    uh = u / r[..., None]
    cos = uh @ uh.transpose(1, 2)
    off = 1.0 - torch.eye(u.shape[1], dtype=torch.float64, device=DEV)
    for zeta in (1, 4):
        for lam in (1.0, -1.0):
            t = 2.0 ** (1 - zeta) * (1.0 + lam * cos) ** zeta * off
            for eta in (0.5, 2.0):
                w = torch.exp(-eta * r * r) * fc
                out.append(((t @ w[..., None])[..., 0] * w).sum(1))
    return torch.stack(out, 1)


def _network(d, g):
    """y of standardised features g (N, 24)."""
    silu = torch.nn.functional.silu
    return silu(silu(g @ d["W1"][:, :24].T + d["b1"]) @ d["W2"].T + d["b2"]) @ d["w3"] + d["b3"]


def _unpack(params):
    """The network's parameters as the kernels use them: BF16 weights, FP32 biases, in float64."""
    d = {k: params[o:o + math.prod(s)].reshape(s) for k, (o, s) in P.OFF.items()}
    return {k: (v.to(torch.bfloat16) if k in ("W1", "W2", "w3") else v).double() for k, v in d.items()}


def _lj(pos, box, rc, shift):
    """(per-atom energy, force) in float64."""
    cells = _Cells(pos, box, rc)
    n, step = pos.shape[0], 16384
    E, F = [], []
    vc = 4.0 * (rc ** -12 - rc ** -6) if shift else 0.0
    for i0 in range(0, n, step):
        i1 = min(n, i0 + step)
        cand = cells.candidates(i0, i1)
        d = pos[i0:i1, None, :] - pos[cand.clamp(min=0)]
        d = d - cells.L * torch.round(d / cells.L)
        d2 = (d * d).sum(2)
        ok = (cand >= 0) & (cand != torch.arange(i0, i1, device=DEV)[:, None]) & (d2 < rc * rc)
        s6 = torch.where(ok, 1.0 / torch.where(ok, d2, torch.ones_like(d2)) ** 3, torch.zeros_like(d2))
        E.append(0.5 * torch.where(ok, 4.0 * (s6 * s6 - s6) - vc, torch.zeros_like(s6)).sum(1))
        F.append(((48.0 * s6 * (s6 - 0.5) / torch.where(ok, d2, torch.ones_like(d2)))[..., None] * d).sum(1))
    return torch.cat(E), torch.cat(F)


def _exact_md(case, seed):
    """The thermo rows of a short FP64 run (the state comes back in the
    library's cell order, so its arrays have no value here)."""
    if case["precision"] != "fp64" or not case["sample"] or case["nx"] * case["ny"] * case["nz"] > 5000:
        return None
    pos, vel, box = _fluid(case, seed)
    dt, every, rows = 0.001, case["sample"], []
    e, F = _lj(pos, box, RC, True)
    ref, last, moved, since, bound = pos, pos, 0.0, 0, 0.0

    def row():
        L = torch.tensor(box, device=DEV, dtype=torch.float64)
        cells = _Cells(pos, box, RC)
        cand = cells.candidates(0, pos.shape[0])
        d = pos[:, None, :] - pos[cand.clamp(min=0)]
        d = d - L * torch.round(d / L)
        d2 = (d * d).sum(2)
        ok = (cand >= 0) & (cand != torch.arange(pos.shape[0], device=DEV)[:, None]) & (d2 < RC * RC)
        s6 = torch.where(ok, 1.0 / torch.where(ok, d2, torch.ones_like(d2)) ** 3, torch.zeros_like(d2))
        return [0.5 * float((vel * vel).sum()), float(e.sum()), float(0.5 * (48.0 * s6 * (s6 - 0.5)).sum()), moved]

    rows.append(row())
    for k in range(1, case["steps"] + 1):
        vel = vel + 0.5 * dt * F
        last, pos = pos, pos + dt * vel
        since, bound = since + 1, bound + dt * float((vel * vel).sum(1).max().sqrt())
        if since >= 10 or 2.0 * bound >= SKIN:
            moved = max(moved, float(((last - ref) ** 2).sum(1).max().sqrt()))
            ref, since, bound = pos, 0, 0.0
        e, F = _lj(pos, box, RC, True)
        vel = vel + 0.5 * dt * F
        if k % every == 0:
            rows.append(row())
    none = {k: None for k in ("x", "y", "z", "vx", "vy", "vz", "fx", "fy", "fz", "ids")}
    return {**none, "thermo": torch.tensor(rows, dtype=torch.float64)}


def _exact_train(case, seed):
    G, e, m, v = _training(case, seed)
    model = _model(seed)
    mu, sd = model.mu.double(), model.sd.double()
    idx = torch.from_numpy(mdinputs.batch_indices(ROWS, case["batch"], case["steps"], int(seed) % 100_003)).to(DEV).long()
    p, m, v = model.params.double(), m.double(), v.double()
    pad = torch.zeros(64, 32, dtype=torch.bool, device=DEV)
    pad[:, 24:] = True
    for k in range(case["steps"]):
        d = {q: t.requires_grad_(True) for q, t in _unpack(p.float()).items()}
        rows = idx[k]
        y = _network(d, (G[rows].double() - mu) / sd)
        loss = ((y - (e[rows] + 5.2) / 0.6) ** 2).mean()
        loss.backward()
        g = torch.zeros_like(p)
        for q, (o, s) in P.OFF.items():
            g[o:o + math.prod(s)] = d[q].grad.reshape(-1)
        g[:2048][pad.reshape(-1)] = 0
        t = 101 + k
        m = 0.9 * m + 0.1 * g
        v = 0.999 * v + 0.001 * g * g
        p = p - LR * (m / (1 - 0.9 ** t)) / ((v / (1 - 0.999 ** t)).sqrt() + 1e-8)
        p[:2048][pad.reshape(-1)] = 0
    return {"params": p, "m": m, "v": v}


def _exact_boa(case, seed):
    pos, box = _polycrystal(case["n"], seed)
    cells = _Cells(pos, box, BOND)
    out, step = {4: [], 5: [], 6: []}, 65536
    for i0 in range(0, case["n"], step):
        u, _, ok = _neighbours(pos, box, BOND, i0, min(case["n"], i0 + step), 32, cells)
        uh = torch.where(ok[..., None], u / (u * u).sum(-1, keepdim=True).sqrt(), torch.zeros_like(u))
        c = uh @ uh.transpose(1, 2)
        both = (ok[:, :, None] & ok[:, None, :]).double()
        nu = ok.sum(1).double()
        c2 = c * c
        pl = {4: (35 * c2 * c2 - 30 * c2 + 3) / 8, 5: c * (63 * c2 * c2 - 70 * c2 + 15) / 8,
              6: (231 * c2 * c2 * c2 - 315 * c2 * c2 + 105 * c2 - 5) / 16}
        for l, t in pl.items():  # addition theorem: Q_l^2 = sum_jk P_l(cos_jk) / nu^2
            out[l].append((t * both).sum((1, 2)).clamp(min=0).sqrt() / nu.clamp(min=1))
    q = {l: torch.cat(t) for l, t in out.items()}
    return {"q4": q[4], "q5": q[5] if case["q5"] else None, "q6": q[6], "nnb": None}


def exact(case, seed):
    kind = case["kind"]
    if kind == "cna":  # whole numbers only
        return None
    if kind == "boa":
        return _exact_boa(case, seed)
    if kind == "train":
        return _exact_train(case, seed)
    if kind == "md":
        return _exact_md(case, seed)
    pos, _, box = _fluid(case, seed)
    if kind == "energy":
        e, F = _lj(pos, box, RC, True)
        return {"e": e.sum(), "grad": -F}
    n, step = pos.shape[0], 1024
    cells = _Cells(pos, box, RC)
    if kind == "snapshot":
        e, F = _lj(pos, box, RC, False)
        G = [_features(*_neighbours(pos, box, RC, i, min(n, i + step), 128, cells)) for i in range(0, n, step)]
        return {"e": e, "F": F, "G": torch.cat(G)}
    model = _model(seed)
    d, mu, sd = _unpack(model.params), model.mu.double(), model.sd.double()
    pos = pos.requires_grad_(True)
    es = []
    for i in range(0, n, step):
        G = _features(*_neighbours(pos, box, RC, i, min(n, i + step), 128, cells))
        e = model.e_mean + model.e_sd * _network(d, (G - mu) / sd)
        e.sum().backward()
        es.append(e.detach())
    F = -pos.grad
    return {"e": torch.cat(es), "fx": F[:, 0], "fy": F[:, 1], "fz": F[:, 2]}
