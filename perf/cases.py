"""Performance cases of the polyethylene MD library: what a simulation program has it do.

Every case goes through ``paper_1001_3764_amd.md.MDSystem`` as a program does:

  step         advance the boxes some steps, read the energies (a program's log line), hand back
               the frame (positions and velocities; in single precision where the forces are,
               as a trajectory file holds them);
  single       forces and energies of a configuration just placed in the buffers;
  observables  the structural observables of the current positions and the end-to-end
               autocorrelation.

Melts are grown by ``pe_melt`` from the seed (a base of a few thousand atoms), relaxed here with
plain torch in FP64 (no code of the library takes part, so the inputs follow from the seed alone),
copied over a lattice of tiles, and given Maxwell velocities for the whole system.  ``exact`` runs
the same physics in FP64 with plain torch operations.
"""

import math

import numpy as np
import torch

from pe_melt import make_melt, polyethylene_forcefield

DEV = "cuda:0"
ACC = 4.184e-4          # (kcal/mol/A) / (g/mol) -> A/fs^2
RGAS = 1.987204259e-3   # kcal/mol/K
RC = 10.5

BASE = {
    "kind": "step", "chains": 10, "chain_len": 300, "tx": 1, "ty": 1, "tz": 1, "density": 0.80, "T": 300.0,
    "T0": 300.0, "tau": 100.0, "dt": 1.0, "steps": 20, "precision": "mixed", "cell_div": 0, "lj_kernel": 0,
    "graph": True, "skin": 0.0, "integrator": "verlet", "com": False, "unequal": False, "boxes": 1,
}


def _case(name, **kw):
    return dict(BASE, name=name, **kw)


def listed():
    return [
        # a small melt watched step by step: one step and its log line, the smallest call
        _case("monitor_3k_fp64", steps=1, precision="fp64", T0=0.0, cell_div=1, lj_kernel=1, graph=False),
        # the 3,000-atom FP64 NVE preset (100 steps), constructor defaults for grid and kernel
        _case("nve_3k_fp64", T=500.0, steps=100, precision="fp64", T0=0.0, cell_div=1, lj_kernel=1, graph=False),
        # the same melt in production: mixed precision, graph replay, thermostatted
        _case("nvt_3k_mixed", steps=100, cell_div=2, lj_kernel=2),
        # everything at the constructor's defaults (27-cell grid, lane per atom, no graph), a mid-size melt of
        # shorter chains
        _case("defaults_33k", chains=17, chain_len=180, tx=3, ty=2, tz=2, T=400.0, T0=0.0, cell_div=1, lj_kernel=1,
              graph=False),
        # the benchmark's melt: 300,000 atoms, tuned, quench from 500 K towards 300 K
        _case("quench_300k_mixed", tx=5, ty=5, tz=4, T=500.0, T0=300.0, steps=20),
        # the same melt in plain FP64
        _case("nvt_300k_fp64", tx=5, ty=5, tz=4, precision="fp64", steps=10, graph=False),
        # the paper's integrator (leap-frog, Nose-Hoover, centre-of-mass removal) on a ragged size
        _case("nose_hoover_127k", chains=13, chain_len=233, tx=7, ty=3, tz=2, integrator="leapfrog", com=True, T=350.0,
              T0=350.0, cell_div=2, lj_kernel=2),
        # the paper's force path: Verlet neighbour lists, rebuilt on displacement
        _case("lists_300k", tx=5, ty=5, tz=4, skin=1.0),
        # the large melt of the throughput presets
        _case("nvt_3M_mixed", tx=10, ty=10, tz=10, density=0.85, steps=5, cell_div=2, lj_kernel=2),
        # a batch of independent boxes of 2,100 to 75,600 atoms at their own temperatures, as replica runs use
        _case("ensemble_24_mixed", chains=7, steps=10, boxes=24, T=250.0, cell_div=2, lj_kernel=2),
        # forces and energies of a given configuration, the two united atoms with different LJ parameters
        _case("single_48k_unequal", kind="single", chains=16, chain_len=250, tx=3, ty=2, tz=2, steps=1, unequal=True,
              cell_div=2, lj_kernel=2, graph=False),
        # analysis of a frame: radial distribution, dihedrals, chain shapes, autocorrelation
        _case("observables_300k", kind="observables", tx=5, ty=5, tz=4, steps=1, cell_div=2, lj_kernel=2, graph=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the ranges above: 1,500 to about 1.5 million atoms, chains of 12 to 300 sites, either
    precision and integrator, the tuned, explicit and default set-ups, one box or a batch."""
    c = dict(BASE)
    chain_len = _log_int(rng, 12, 300)
    chains = max(1, int(round(_log_int(rng, 1700, 6000) / chain_len)))
    chains += 1 if chains * chain_len < 1600 else 0
    base = chains * chain_len
    c.update(chain_len=chain_len, chains=chains, density=round(rng.uniform(0.72, 0.86), 3),
             T=round(rng.uniform(250.0, 500.0), 1))
    form = rng.choice(["step", "step", "step", "step", "fp64", "lists", "batch", "single", "observables", "defaults"])
    most = {"step": 1.5e6, "fp64": 4e5, "lists": 6e5, "batch": 3e4, "single": 3e5, "observables": 4e5,
            "defaults": 1.2e5}[form]
    copies = _log_int(rng, 1, max(1, int(most / base)))
    c["tx"] = max(1, int(round(copies ** (1 / 3) * rng.uniform(0.8, 1.5))))
    c["ty"] = max(1, int(round((copies / c["tx"]) ** 0.5 * rng.uniform(0.8, 1.25))))
    c["tz"] = max(1, copies // (c["tx"] * c["ty"]))
    atoms = base * c["tx"] * c["ty"] * c["tz"]
    c["T0"] = rng.choice([0.0, c["T"], 300.0])
    c["steps"] = int(min(60, max(3, 6e6 // atoms)))
    if form == "step":
        c.update(integrator=rng.choice(["verlet", "leapfrog"]), com=rng.random() < 0.4, graph=rng.random() < 0.7,
                 cell_div=2, lj_kernel=2)
    elif form == "fp64":
        c.update(precision="fp64", graph=rng.random() < 0.5, steps=max(3, c["steps"] // 3), cell_div=2, lj_kernel=2)
    elif form == "lists":
        c.update(skin=round(rng.uniform(0.6, 1.4), 2), cell_div=2, lj_kernel=5)
    elif form == "batch":
        c.update(boxes=rng.randrange(5, 30), cell_div=2, lj_kernel=2)
        c["steps"] = int(min(30, max(2, 6e6 // _atoms(c))))
    elif form == "single":
        c.update(kind="single", steps=1, unequal=rng.random() < 0.6, graph=False, cell_div=rng.choice([1, 2]),
                 lj_kernel=2, precision=rng.choice(["mixed", "fp64"]))
    elif form == "observables":
        c.update(kind="observables", steps=1, cell_div=2, lj_kernel=2, graph=False)
    else:
        c.update(cell_div=1, lj_kernel=1, graph=False, T0=0.0, precision=rng.choice(["mixed", "fp64"]))
    return c


# ---- inputs ----

def _forcefield(case):
    ff = polyethylene_forcefield(RC)
    if case["unequal"]:
        ff.update(sigma=(3.47, 3.70), epsilon=(0.0951, 0.1200))
    return ff


def _tiles(case, b):
    """Tile counts of box b (a batch cycles through small multiples of the first box's)."""
    t = (case["tx"], case["ty"], case["tz"])
    if case["boxes"] == 1:
        return t
    k = ((1, 1, 1), (2, 1, 1), (2, 2, 1), (3, 1, 1), (3, 2, 1), (2, 2, 2), (3, 2, 2), (4, 3, 3))[b % 8]
    return tuple(a * s for a, s in zip(t, k))


def _maxwell(types, ff, T, gen):
    m = torch.tensor(ff["mass"], dtype=torch.float64, device=DEV)[types.long()]
    n = types.numel()
    v = torch.randn((3, n), dtype=torch.float64, device=DEV, generator=gen) * (RGAS * T * ACC / m).sqrt()
    v -= (v * m).sum(1, keepdim=True) / m.sum()
    t_now = (m * v * v).sum() / ACC / ((3 * n - 3) * RGAS)
    return v * (T / t_now).sqrt()


def _base_melt(case, seed):
    """The grown base melt with its contacts resolved: a capped descent, then a short isokinetic run."""
    ff = polyethylene_forcefield(RC)
    m = make_melt(case["chains"], case["chain_len"], case["density"], case["T"], 10007 * seed + 1, 10007 * seed + 2)
    box = torch.tensor(m.box, dtype=torch.float64, device=DEV)
    pos = torch.tensor(m.pos, dtype=torch.float64, device=DEV)
    types = torch.tensor(m.types, device=DEV)
    mass = torch.tensor(ff["mass"], dtype=torch.float64, device=DEV)[types.long()]
    for _ in range(50):
        f, _ = _forces(pos, box, types, case["chain_len"], ff)
        pos = torch.remainder(pos + (4e-4 * f).clamp(-0.05, 0.05), box[:, None])
    vel = _maxwell(types, ff, case["T"], torch.Generator(device=DEV).manual_seed(seed + 77))
    f, _ = _forces(pos, box, types, case["chain_len"], ff)
    for _ in range(60):
        vel = vel + 0.5 * ACC * f / mass
        pos = torch.remainder(pos + vel, box[:, None])
        f, _ = _forces(pos, box, types, case["chain_len"], ff)
        vel = vel + 0.5 * ACC * f / mass
        vel = vel * (case["T"] * (3 * pos.shape[1] - 3) * RGAS / ((mass * vel * vel).sum() / ACC)).sqrt()
    return pos, box, types


def _unwrap(pos, box, chain_len):
    p = pos.reshape(3, -1, chain_len)
    d = p[:, :, 1:] - p[:, :, :-1]
    d = d - box[:, None, None] * torch.round(d / box[:, None, None])
    return torch.cat([p[:, :, :1], p[:, :, :1] + d.cumsum(2)], 2).reshape(3, -1)


def _inputs(case, seed):
    """(positions, velocities, types, boxes, chains per box, T0 per box), device tensors, box after box."""
    ff = _forcefield(case)
    pos0, box0, types0 = _base_melt(case, seed)
    flat = _unwrap(pos0, box0, case["chain_len"])
    gen = torch.Generator(device=DEV).manual_seed(seed + 1234567)
    P, V, Y, boxes, chains, T0 = [], [], [], [], [], []
    for b in range(case["boxes"]):
        t = _tiles(case, b)
        temp = case["T"] if case["boxes"] == 1 else 250.0 + 200.0 * b / (case["boxes"] - 1)
        n = t[0] * t[1] * t[2]
        cell = torch.arange(n, device=DEV)
        at = torch.stack([cell // (t[1] * t[2]), cell // t[2] % t[1], cell % t[2]]).double()
        box = box0 * torch.tensor(t, dtype=torch.float64, device=DEV)
        p = (flat[:, None, :] + (at * box0[:, None])[:, :, None]).reshape(3, -1)
        p = torch.remainder(p, box[:, None])
        p = torch.where(p >= box[:, None], torch.zeros_like(p), p)
        y = types0.repeat(n)
        P.append(p)
        V.append(_maxwell(y, ff, temp, gen))
        Y.append(y)
        boxes.append(box)
        chains.append(case["chains"] * n)
        T0.append(case["T0"] if case["boxes"] == 1 or case["T0"] <= 0 else temp)
    return torch.cat(P, 1), torch.cat(V, 1), torch.cat(Y), torch.stack(boxes), chains, T0


def _displaced(case, pos, boxes, seed):
    """Other positions of the same melt: small seeded displacements, as some steps later."""
    gen = torch.Generator(device=DEV).manual_seed(seed + 424242)
    out, a = [], 0
    for b in range(case["boxes"]):
        n = case["chains"] * case["chain_len"] * math.prod(_tiles(case, b))
        d = 0.04 * torch.randn((3, n), dtype=torch.float64, device=DEV, generator=gen)
        p = torch.remainder(pos[:, a:a + n] + d, boxes[b][:, None])
        out.append(torch.where(p >= boxes[b][:, None], torch.zeros_like(p), p))
        a += n
    return torch.cat(out, 1)


def prepare(case, seed):
    from paper_1001_3764_amd.md import MDSystem

    pos, vel, types, boxes, chains, T0 = _inputs(case, seed)
    kw = {}
    if case["skin"] > 0:
        kw = dict(nl_skin=case["skin"], nl_every=0)
    s = MDSystem(_forcefield(case), chains, boxes.cpu().numpy(), T0, pos.cpu().numpy(), vel.cpu().numpy(),
                 types.cpu().numpy(), chain_len=case["chain_len"], dt=case["dt"], tau=case["tau"],
                 precision=case["precision"], cell_div=case["cell_div"], lj_kernel=case["lj_kernel"],
                 use_graph=case["graph"], device=DEV, integrator=case["integrator"], remove_com=case["com"], **kw)
    state = {"case": case, "system": s}
    if case["kind"] != "step":
        state["pos"] = _displaced(case, pos, boxes, seed)
        if case["kind"] == "observables":
            s.pos.copy_(state["pos"])
            s.rebuild_bins()
    return state


ENERGIES = ("e_lj", "e_lj_shifted", "e_bond", "e_angle", "e_dih", "e_kin", "temperature", "virial")


def _real(case):
    return np.float32 if case["precision"] == "mixed" else np.float64


def _log_line(case, energies):
    keys = ENERGIES if case["kind"] == "step" else tuple(k for k in ENERGIES if k not in ("e_kin", "temperature"))
    return np.array([[e[k] for k in keys] for e in energies], dtype=np.float64).astype(_real(case))


def run(state):
    case, s = state["case"], state["system"]
    if case["kind"] == "observables":
        got = s.observables(rdf_bins=210, rdf_rmax=RC, dih_bins=72)
        got["pair_counts"] = got["pair_counts"].astype(np.int64)
        got["dihedral_hist"] = got["dihedral_hist"].astype(np.int64)
        got["dihedral_classes"] = got["dihedral_classes"].astype(np.int64)
        got["ree_acf"] = s.ree_acf()
        return got
    if case["kind"] == "single":
        s.pos.copy_(state["pos"])
        s.rebuild_bins()
        s.compute_forces(True)
        return {"energies": _log_line(case, s.energies()), "forces": s.forces().astype(_real(case))}
    s.step(case["steps"])
    energies = _log_line(case, s.energies())
    if case["precision"] == "mixed":
        return {"energies": energies, "pos": s.pos.float(), "vel": s.vel.float()}
    return {"energies": energies, "pos": s.pos, "vel": s.vel}


def _atoms(case):
    return sum(case["chains"] * case["chain_len"] * math.prod(_tiles(case, b)) for b in range(case["boxes"]))


def work(case):
    """A pass reads its state (positions, velocities, types) once and writes it once; each step
    evaluates every unordered pair inside the cutoff once (24 flops: difference, r^2, reciprocal,
    force factor, both sums) and about 230 flops per atom of bonded terms and update."""
    n = _atoms(case)
    per_chain = (case["chain_len"] - 2) * 14.027 + 2 * 15.035
    rho = case["density"] * 0.602214076 / per_chain * case["chain_len"]
    pairs = 0.5 * n * rho * 4.0 / 3.0 * math.pi * RC ** 3
    if case["kind"] == "observables":
        return {"bytes": 24.0 * n + 32.0 * n / case["chain_len"], "flops": 12.0 * pairs + 150.0 * n}
    if case["kind"] == "single":
        return {"bytes": (25.0 + (12 if case["precision"] == "mixed" else 24)) * n, "flops": 24.0 * pairs + 200.0 * n}
    return {"bytes": 97.0 * n, "flops": case["steps"] * (24.0 * pairs + 230.0 * n)}


# ---- the same physics in plain torch, FP64 ----

def _lj(pos, box, types, chain_len, ff):
    """Truncated LJ over a 27-cell grid: forces [3, N], energy, shifted energy, virial."""
    rc, excl, n = ff["rc"], ff["excl_depth"], pos.shape[1]
    M = [int(math.floor(float(box[d]) / rc)) for d in range(3)]
    k = [(pos[d] * (M[d] / box[d])).floor().long().clamp(0, M[d] - 1) for d in range(3)]
    cell = k[0] + M[0] * (k[1] + M[1] * k[2])
    C = M[0] * M[1] * M[2]
    order = torch.argsort(cell, stable=True)
    count = torch.bincount(cell, minlength=C)
    start = count.cumsum(0) - count
    cap = int(count.max())
    slot = torch.full((C, cap), n, dtype=torch.long, device=DEV)
    slot[cell[order], torch.arange(n, device=DEV) - start[cell[order]]] = order
    # the sentinel atom n lies far from everything
    padded = torch.cat([pos, torch.full((3, 1), 1e6, dtype=torch.float64, device=DEV)], 1)
    ty = torch.cat([types.long(), torch.zeros(1, dtype=torch.long, device=DEV)])
    c = torch.arange(C, device=DEV)
    ck = [c % M[0], c // M[0] % M[1], c // (M[0] * M[1])]
    nb, shift = [], []
    for o in range(27):
        u = [ck[d] + (o // 3 ** d % 3 - 1) for d in range(3)]
        w = [torch.div(u[d], M[d], rounding_mode="floor") for d in range(3)]
        nb.append((u[0] - w[0] * M[0]) + M[0] * ((u[1] - w[1] * M[1]) + M[1] * (u[2] - w[2] * M[2])))
        shift.append(torch.stack([w[d] * box[d] for d in range(3)]))
    nb, shift = torch.stack(nb, 1), torch.stack(shift, 2)                    # [C, 27], [3, C, 27]
    sig, eps = ff["sigma"], ff["epsilon"]
    uniform = sig[0] == sig[1] and eps[0] == eps[1]
    s6 = torch.tensor([(0.5 * (sig[a] + sig[b])) ** 6 for a in (0, 1) for b in (0, 1)], dtype=torch.float64, device=DEV)
    e4 = torch.tensor([4.0 * math.sqrt(eps[a] * eps[b]) for a in (0, 1) for b in (0, 1)], dtype=torch.float64,
                      device=DEV)
    f = torch.zeros((3, n + 1), dtype=torch.float64, device=DEV)
    sums = torch.zeros(3, dtype=torch.float64, device=DEV)
    chunk = max(1, int(1.2e7 // (cap * cap * 27)))
    for c0 in range(0, C, chunk):
        I, Jc = slot[c0:c0 + chunk], nb[c0:c0 + chunk]
        J = slot[Jc].reshape(I.shape[0], -1)                                 # [c, 27 cap]
        d = []
        for q in range(3):
            xj = padded[q][J] + shift[q, c0:c0 + chunk].repeat_interleave(cap, dim=1)
            d.append(padded[q][I][:, :, None] - xj[:, None, :])
        r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2]
        Ib, Jb = I[:, :, None], J[:, None, :]
        same = (torch.div(Ib, chain_len, rounding_mode="floor") == torch.div(Jb, chain_len, rounding_mode="floor"))
        on = (r2 < rc * rc) & ~(same & ((Ib - Jb).abs() <= excl)) & (Ib < n) & (Jb < n)
        r2i = torch.where(on, 1.0 / r2, torch.zeros_like(r2))
        if uniform:
            a6, e = s6[0], e4[0]
        else:
            t = ty[I][:, :, None] * 2 + ty[J][:, None, :]
            a6, e = s6[t], e4[t]
        u6 = r2i * r2i * r2i * a6
        g = e * u6 * (12.0 * u6 - 6.0)
        ffs = g * r2i
        for q in range(3):
            f[q, I.reshape(-1)] = (ffs * d[q]).sum(2).reshape(-1)
        uc = a6 / rc ** 6
        en = e * u6 * (u6 - 1.0)
        cut = torch.where(on, e * uc * (uc - 1.0) + torch.zeros_like(r2), torch.zeros_like(r2))
        sums += 0.5 * torch.stack([en.sum(), (en - cut).sum(), g.sum()])
    return f[:, :n], sums


def _bonded(pos, box, chain_len, ff):
    """Bond, angle and dihedral terms as functions of the bond vectors: forces [3, N], the three
    energies and the virial -sum b . dE/db."""
    p = pos.reshape(3, -1, chain_len)
    b = p[:, :, 1:] - p[:, :, :-1]
    b = (b - box[:, None, None] * torch.round(b / box[:, None, None])).detach().requires_grad_(True)
    cross = lambda a, c: torch.stack([a[1] * c[2] - a[2] * c[1], a[2] * c[0] - a[0] * c[2], a[0] * c[1] - a[1] * c[0]])
    dot = lambda a, c: (a * c).sum(0)
    e_bond = (0.5 * ff["kb"] * (dot(b, b).sqrt() - ff["b0"]) ** 2).sum()
    u, w = -b[:, :, :-1], b[:, :, 1:]
    x = cross(u, w)
    theta = torch.atan2(dot(x, x).sqrt(), dot(u, w))
    e_angle = (0.5 * ff["ka"] * (theta - math.radians(ff["theta0_deg"])) ** 2).sum()
    m, k = cross(b[:, :, :-2], b[:, :, 1:-1]), cross(b[:, :, 1:-1], b[:, :, 2:])
    cos1 = dot(m, k)
    sin1 = dot(b[:, :, 1:-1], b[:, :, 1:-1]).sqrt() * dot(b[:, :, :-2], k)
    phi = torch.atan2(sin1, cos1)
    e_dih = (ff["kphi"] * (1.0 + torch.cos(ff["n_dih"] * phi - math.radians(ff["phis_deg"])))).sum()
    (g,) = torch.autograd.grad(e_bond + e_angle + e_dih, b)
    f = torch.zeros_like(p)
    f[:, :, :-1] += g
    f[:, :, 1:] -= g
    virial = -(b.detach() * g).sum()
    return f.reshape(3, -1), torch.stack([e_bond.detach(), e_angle.detach(), e_dih.detach()]), virial


def _forces(pos, box, types, chain_len, ff):
    """Total force [3, N] and (e_lj, e_lj_shifted, e_bond, e_angle, e_dih, virial)."""
    f, lj = _lj(pos, box, types, chain_len, ff)
    fb, eb, wb = _bonded(pos, box, chain_len, ff)
    return f + fb, torch.stack([lj[0], lj[1], eb[0], eb[1], eb[2], lj[2] + wb])


def _simulate(case, pos, vel, types, box, T0, ff):
    """One box, case["steps"] steps: positions, velocities and the last step's log line."""
    dt, tau, n = case["dt"], case["tau"], pos.shape[1]
    m = torch.tensor(ff["mass"], dtype=torch.float64, device=DEV)[types.long()]
    dof, w2 = 3 * n - 3, (2.0 * math.pi / tau) ** 2
    a = ACC / m
    leap = case["integrator"] == "leapfrog"
    xi = 0.0
    f, e = _forces(pos, box, types, case["chain_len"], ff)
    for _ in range(case["steps"]):
        if leap:
            vel = ((1.0 - 0.5 * dt * xi) * vel + dt * a * f) / (1.0 + 0.5 * dt * xi)
        else:
            vel = vel + 0.5 * dt * a * f
        pos = torch.remainder(pos + dt * vel, box[:, None])
        pos = torch.where(pos >= box[:, None], torch.zeros_like(pos), pos)
        f, e = _forces(pos, box, types, case["chain_len"], ff)
        if not leap:
            vel = vel + 0.5 * dt * a * f
        if case["com"]:
            vel = vel - (m * vel).sum(1, keepdim=True) / m.sum()
        ke = float(0.5 * (m * vel * vel).sum() / ACC)
        T = 2.0 * ke / (dof * RGAS)
        if T0 > 0 and leap:
            xi += dt * w2 * (T / T0 - 1.0)
        elif T0 > 0:
            vel = vel * math.sqrt(1.0 + dt / tau * (T0 / T - 1.0))
    e = e.tolist()
    return pos, vel, e[:5] + [ke, T, e[5]]


def exact(case, seed):
    pos, vel, types, boxes, chains, T0 = _inputs(case, seed)
    ff, L = _forcefield(case), case["chain_len"]
    if case["kind"] == "observables":
        at = _displaced(case, pos, boxes, seed)
        m = torch.tensor(ff["mass"], dtype=torch.float64, device=DEV)[types.long()].reshape(-1, L)
        u, u0 = (_unwrap(p, boxes[0], L).reshape(3, -1, L) for p in (at, pos))
        cm = (u * m).sum(2, keepdim=True) / m.sum(1)[:, None]
        rg2 = (((u - cm) ** 2).sum(0) * m).sum(1) / m.sum(1)
        ree, ree0 = u[:, :, -1] - u[:, :, 0], u0[:, :, -1] - u0[:, :, 0]
        return {"pair_counts": None, "dihedral_hist": None, "dihedral_classes": None,
                "chain_shape": torch.cat([rg2[None], ree]).T.contiguous(),
                "ree_acf": ((ree * ree0).sum() / (ree0 * ree0).sum()).reshape(1)}
    P, V, E, a = [], [], [], 0
    if case["kind"] == "single":
        pos = _displaced(case, pos, boxes, seed)
    for b in range(case["boxes"]):
        n = chains[b] * L
        p, v, y = pos[:, a:a + n], vel[:, a:a + n], types[a:a + n]
        if case["kind"] == "single":
            f, e = _forces(p, boxes[b], y, L, ff)
            P.append(f)
            E.append(e.tolist())
        else:
            p, v, e = _simulate(case, p, v, y, boxes[b], T0[b], ff)
            P.append(p)
            V.append(v)
            E.append(e)
        a += n
    line = np.array(E, dtype=np.float64)
    if case["kind"] == "single":
        return {"energies": line, "forces": torch.cat(P, 1)}
    return {"energies": line, "pos": torch.cat(P, 1), "vel": torch.cat(V, 1)}
