"""The work this framework is timed on: one pass of each case through its public entry points.

Every case is a dict of plain values; ``kind`` says which calls a pass makes:

  run       System.step(steps), then get_state() (and props() where asked): a plain NVE run
            between two frames.  FP32 or FP64 forces, neighbour list or (shell 0) the cell
            method, soft spheres or Lennard-Jones at any cutoff.
  block     block_begin, step, block_end, get_state: averages over a block of steps.
  equil     equilibrate_run (step + adjust_temp every 20 steps) and the property trace of
            its steps: thermostatted equilibration with every step's energies kept.
  mixture   step, then get_state, of a two-species fluid.
  batch     Batch.run() x runs, then every replica's state: independent replicas together.
  evaluate  set_state, get_state, atom_energies: forces and energies of given positions.

Systems start from a lattice with jittered sites and random velocities, the start the library's
own workloads use; passes on one state continue its trajectory, as a program's frames do.
"""
import math

import numpy as np
import torch

RC_SOFT = 2.0 ** (1.0 / 6.0)


def listed():
    return [
        # the smallest call: one FP64 cell-method step and its state, as a program that
        # couples the fluid to something else makes it every step
        dict(name="one_step_2048_fp64", kind="run", lattice="fcc", edge=8, rho=0.8, temp=1.0,
             shell=0.0, rc=RC_SOFT, prec="fp64", steps=1, props=False),
        # the small reference workload: N = 2 048, cell method (a sort every step), FP64
        dict(name="cells_2048_fp64", kind="run", lattice="fcc", edge=8, rho=0.8, temp=1.0,
             shell=0.0, rc=RC_SOFT, prec="fp64", steps=200, props=True),
        # the smallest replica size of the batch workload, stepped alone
        dict(name="run_864", kind="run", lattice="fcc", edge=6, rho=0.8, temp=1.0,
             shell=0.4, rc=RC_SOFT, prec="fp32", steps=200, props=True),
        # the largest replica size, FP64 forces from a neighbour list
        dict(name="run_32000_fp64", kind="run", lattice="fcc", edge=20, rho=0.85, temp=1.2,
             shell=0.4, rc=RC_SOFT, prec="fp64", steps=200, props=False),
        # thermostatted equilibration of an odd-sized system with its property trace
        dict(name="equil_19683", kind="equil", lattice="sc", edge=27, rho=0.8, temp=1.0,
             shell=0.4, rc=RC_SOFT, prec="fp32", steps=200),
        # the paper's system S: averages over a block of steps
        dict(name="block_110592", kind="block", lattice="sc", edge=48, rho=0.8, temp=1.0,
             shell=0.6, rc=RC_SOFT, prec="fp32", steps=200),
        # the medium reference workload between two frames
        dict(name="run_256000", kind="run", lattice="fcc", edge=40, rho=0.8, temp=1.0,
             shell=0.4, rc=RC_SOFT, prec="fp32", steps=1000, props=False),
        # the headline workload between two frames
        dict(name="run_4000000", kind="run", lattice="fcc", edge=100, rho=0.8, temp=1.0,
             shell=0.4, rc=RC_SOFT, prec="fp32", steps=1000, props=False),
        # Lennard-Jones with the longest cutoff used: lists of about 90 entries
        dict(name="lj3_110592", kind="run", lattice="sc", edge=48, rho=0.38, temp=1.2,
             shell=0.8, rc=3.0, prec="fp32", steps=200, props=False),
        # a binary mixture of a ragged size
        dict(name="mixture_119164", kind="mixture", lattice="fcc", edge=31, rho=0.75, temp=1.0,
             shell=0.4, prec="fp32", steps=200),
        # independent replicas of uneven size, advanced together
        dict(name="batch_48", kind="batch", replicas=48, k_lo=6, k_hi=20, shell=0.4,
             per_run=64, runs=8),
        # forces and energies of a given configuration (odd size)
        dict(name="evaluate_103823", kind="evaluate", lattice="sc", edge=47, rho=0.8, temp=1.0,
             shell=0.4, rc=RC_SOFT, prec="fp32"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["run", "run", "run", "run", "block", "equil", "mixture", "batch",
                       "evaluate"])
    if kind == "batch":
        k_lo = rng.randint(6, 12)
        return dict(kind=kind, replicas=_log_int(rng, 2, 64), k_lo=k_lo,
                    k_hi=rng.randint(k_lo, 20), shell=round(rng.uniform(0.3, 0.5), 3),
                    per_run=rng.choice([16, 32, 64]), runs=rng.randint(1, 4))
    lattice = rng.choice(["fcc", "sc"])
    n = math.exp(rng.uniform(math.log(800), math.log(2.0e6 if kind == "run" else 3.0e5)))
    edge = max(6, round((n / 4.0) ** (1.0 / 3.0))) if lattice == "fcc" else \
        max(9, round(n ** (1.0 / 3.0)))
    n = 4 * edge ** 3 if lattice == "fcc" else edge ** 3
    case = dict(kind=kind, lattice=lattice, edge=edge, rho=round(rng.uniform(0.7, 0.9), 3),
                temp=round(rng.uniform(0.8, 1.5), 3), shell=round(rng.uniform(0.3, 0.6), 3),
                rc=RC_SOFT, prec=rng.choice(["fp32", "fp32", "fp64"]))
    if kind == "mixture":
        del case["rc"]
        case["rho"] = round(rng.uniform(0.65, 0.75), 3)
        case["prec"] = "fp32"
    elif kind == "run" and n < 3.0e5 and n > 3000:
        style = rng.choice(["soft", "soft", "lj", "cells"])
        if style == "lj":
            case.update(rc=rng.choice([2.2, 2.5, 3.0]), rho=0.38, shell=0.8)
        elif style == "cells":
            case.update(shell=0.0)
    if kind == "equil":
        case["prec"] = "fp32"
    if kind == "run":
        case["props"] = rng.random() < 0.5
    if kind != "evaluate":
        most = max(1, min(400, int(4.0e8 / n)))
        case["steps"] = _log_int(rng, 1, most)
        if kind == "equil":
            case["steps"] = max(1, case["steps"] // 20) * 20
    return case


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
_FCC = np.array([[0.0, 0.0, 0.0], [0.0, 0.5, 0.5], [0.5, 0.0, 0.5], [0.5, 0.5, 0.0]])


def _start(lattice, edge, rho, temp, seed, amplitude=0.07):
    """Positions, velocities and box edge: jittered lattice sites, |v| = sqrt(3 T) in random
    directions with the mean removed."""
    rng = np.random.default_rng(seed)
    basis = _FCC if lattice == "fcc" else np.zeros((1, 3))
    n = len(basis) * edge ** 3
    box = (n / rho) ** (1.0 / 3.0)
    a = box / edge
    g = np.arange(edge, dtype=np.float64)
    pos = np.empty((edge, edge, edge, len(basis), 3))
    off = 0.25 if lattice == "fcc" else 0.5
    pos[..., 0] = (g[None, None, :, None] + basis[:, 0] + off)
    pos[..., 1] = (g[None, :, None, None] + basis[:, 1] + off)
    pos[..., 2] = (g[:, None, None, None] + basis[:, 2] + off)
    pos = pos.reshape(-1, 3)
    pos *= a
    pos -= 0.5 * box
    pos += rng.random((n, 3)) * (2.0 * amplitude) - amplitude
    pos -= box * np.floor(pos / box + 0.5)
    pos[pos >= 0.5 * box] -= box
    cz = rng.uniform(-1.0, 1.0, n)
    phi = rng.uniform(0.0, 2.0 * math.pi, n)
    s = np.sqrt(1.0 - cz * cz)
    vel = np.stack([s * np.cos(phi), s * np.sin(phi), cz], axis=1)
    vel *= math.sqrt(3.0 * temp)
    vel -= vel.mean(axis=0, keepdims=True)
    return np.ascontiguousarray(pos), np.ascontiguousarray(vel), box


def _species(case, n, seed):
    """Half the atoms of species B; WCA pairs of diameters 1 / 1.1 / 1.2."""
    sp = (np.random.default_rng(seed + 1).permutation(n) < n // 2).astype(np.int32)
    sig = np.array([[1.0, 1.1], [1.1, 1.2]])
    eps = np.array([[1.0, 1.5], [1.5, 1.0]])
    return sp, eps, sig, RC_SOFT * sig, eps.copy()


def _sizes(case):
    """fcc cells per edge of each replica, spread over [k_lo, k_hi]."""
    span = case["k_hi"] - case["k_lo"] + 1
    return [case["k_lo"] + (7 * r + 3) % span for r in range(case["replicas"])]


def _replicas(case, seed):
    rng = np.random.default_rng(seed)
    out = []
    for r, k in enumerate(_sizes(case)):
        rho, temp = float(rng.uniform(0.7, 0.9)), float(rng.uniform(0.8, 1.5))
        out.append(_start("fcc", k, rho, temp, 1000003 * (seed % 9973) + r))
    return out


def prepare(case, seed):
    from paper_0911_5631_amd.md import Batch, System
    kind = case["kind"]
    if kind == "batch":
        b = Batch(64 << 30, case["replicas"], case["per_run"])
        slots = [b.admit(p, v, box, 1 << 40, shell=case["shell"])
                 for p, v, box in _replicas(case, seed)]
        return dict(case=case, batch=b, slots=slots)
    pos, vel, box = _start(case["lattice"], case["edge"], case["rho"], case["temp"], seed)
    if kind == "mixture":
        sp, eps, sig, rcut, shift = _species(case, len(pos), seed)
        s = System(pos, vel, box, shell=case["shell"], r_cut=float(rcut.max()),
                   precision=case["prec"])
        s.set_species(sp, eps, sig, rcut, shift)
        return dict(case=case, system=s)
    s = System(pos, vel, box, shell=case["shell"], r_cut=case["rc"], precision=case["prec"],
               trace=kind == "equil")
    state = dict(case=case, system=s, at=0)
    if kind == "evaluate":
        # the configurations to be evaluated: other positions of the same atoms
        state["pos"], state["vel"], _ = _start(case["lattice"], case["edge"], case["rho"],
                                               case["temp"], seed + 77, amplitude=0.1)
    return state


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "batch":
        b = state["batch"]
        for _ in range(case["runs"]):
            b.run()
        b.poll()
        got = [b.get_state(slot) for slot in state["slots"]]
        return dict(pos=np.concatenate([g[0] for g in got]),
                    vel=np.concatenate([g[1] for g in got]),
                    step=np.array([g[2] for g in got]))
    s = state["system"]
    if kind == "evaluate":
        s.set_state(state["pos"], state["vel"])
        pos, vel, force, _ = s.get_state()
        u, w = s.atom_energies()
        return dict(pos=pos, vel=vel, force=force, u=u, w=w)
    out = {}
    if kind == "block":
        s.block_begin()
        s.step(case["steps"])
        out["block"] = s.block_end()
    elif kind == "equil":
        s.equilibrate_run(case["steps"], case["temp"], equil_steps=1 << 40)
        rows = s.trace(state["at"] + 1, case["steps"])
        state["at"] += case["steps"]
        out["trace"] = {k: np.ascontiguousarray(rows[k]) for k in ("ke", "pe", "virial", "vmax")}
    else:
        s.step(case["steps"])
    pos, vel, force, step = s.get_state()
    out.update(pos=pos, vel=vel, force=force, step=step)
    if case.get("props"):
        out["props"] = s.props()
    return out


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def _atoms(case):
    if case["kind"] == "batch":
        return sum(4 * k ** 3 for k in _sizes(case))
    return (4 if case["lattice"] == "fcc" else 1) * case["edge"] ** 3


def work(case):
    """A step reads and writes every position and velocity (96 B per atom) and tests or adds
    every pair within the list radius (9 operations for the distance, 22 more for a force);
    a frame writes positions, velocities and forces (72 B)."""
    n = _atoms(case)
    kind = case["kind"]
    if kind == "evaluate":
        steps = 1
    elif kind == "batch":
        steps = case["runs"] * case["per_run"]
    else:
        steps = case["steps"]
    rho = case.get("rho", 0.8)
    rc = case.get("rc", RC_SOFT * (1.2 if kind == "mixture" else 1.0))
    sphere = 4.0 / 3.0 * math.pi * rho
    near = sphere * (rc + case["shell"]) ** 3
    inside = sphere * rc ** 3
    return {"bytes": n * (96.0 * steps + 72.0), "flops": n * steps * (9.0 * near + 22.0 * inside)}


# ---------------------------------------------------------------------------
# the same in 64 bits with plain torch
# ---------------------------------------------------------------------------
_DEV = "cuda" if torch.cuda.is_available() else "cpu"


def _pairs(x, box, rn):
    """Unordered pairs (i < j) of wrapped positions with r < rn, from a padded cell table."""
    n = len(x)
    G = int(box / rn)
    c = ((x + 0.5 * box) * (G / box)).long().clamp_(0, G - 1)
    cell = (c[:, 2] * G + c[:, 1]) * G + c[:, 0]
    order = torch.argsort(cell, stable=True)
    count = torch.bincount(cell, minlength=G ** 3)
    first = torch.cumsum(count, 0) - count
    table = torch.full((G ** 3, int(count.max())), -1, dtype=torch.long, device=x.device)
    sc = cell[order]
    table[sc, torch.arange(n, device=x.device) - first[sc]] = order
    me = torch.arange(n, device=x.device)
    got_i, got_j = [], []
    for dz in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                other = (((c[:, 2] + dz) % G) * G + (c[:, 1] + dy) % G) * G + (c[:, 0] + dx) % G
                j = table[other]
                d = x[:, None, :] - x[j.clamp(min=0)]
                d -= box * torch.round(d / box)
                ok = ((d * d).sum(-1) < rn * rn) & (j > me[:, None])
                i_, k_ = torch.nonzero(ok, as_tuple=True)
                got_i.append(i_)
                got_j.append(j[i_, k_])
    return torch.cat(got_i), torch.cat(got_j)


def _forces(x, box, i, j, rc2, sig2, eps, shift):
    """Forces, per-atom energies and virials (each pair on both of its atoms)."""
    d = x[i] - x[j]
    d -= box * torch.round(d / box)
    s = (d * d).sum(-1)
    inside = s < rc2
    q = torch.where(inside, sig2 / s, torch.zeros_like(s))
    q3 = q * q * q
    f = 48.0 * eps * q3 * (q3 - 0.5) / s * inside
    u = (4.0 * eps * q3 * (q3 - 1.0) + shift) * inside
    fd = f[:, None] * d
    w = f * s
    force = torch.zeros_like(x).index_add_(0, i, fd).index_add_(0, j, -fd)
    uu = torch.zeros(len(x), dtype=x.dtype, device=x.device).index_add_(0, i, u).index_add_(0, j, u)
    ww = torch.zeros_like(uu).index_add_(0, i, w).index_add_(0, j, w)
    return force, uu, ww


def _wrap(x, box):
    x = torch.where(x >= 0.5 * box, x - box, x)
    return torch.where(x < -0.5 * box, x + box, x)


def _simulate(pos, vel, box, steps, rc, shell, dt=0.005, species=None, temp=None, every=None,
              rows=None):
    """`steps` leapfrog steps in 64 bits; positions are wrapped where the displacement rule
    rebuilds (every step without a shell), as the library returns them."""
    x = _wrap(torch.from_numpy(pos).to(_DEV), box)
    v = torch.from_numpy(vel).to(_DEV)
    n = len(x)

    def pair_list():
        i, j = _pairs(_wrap(x, box), box, rc + max(shell, 0.05))
        if species is None:
            t = (rc * rc, 1.0, 1.0, 1.0 if rc == RC_SOFT else 0.0)
        else:
            sp, eps, sig, rcut, shift = species
            k = torch.from_numpy(sp).to(_DEV).long()
            k = k[i] * 2 + k[j]
            t = tuple(torch.from_numpy(np.ascontiguousarray(a).reshape(-1)).to(_DEV)[k]
                      for a in (rcut * rcut, sig * sig, eps, shift))
        return i, j, t

    i, j, t = pair_list()
    f, u, w = _forces(x, box, i, j, *t)
    disp = float((v * v).sum(-1).max()) ** 0.5 * dt
    for k in range(1, steps + 1):
        v = v + 0.5 * dt * f
        x = x + dt * v
        if shell == 0.0 or disp > 0.5 * shell:
            x = _wrap(x, box)
            i, j, t = pair_list()
            disp = 0.0
        f, u, w = _forces(x, box, i, j, *t)
        v = v + 0.5 * dt * f
        vv = (v * v).sum(-1)
        vm = vv.max()
        disp += float(vm) ** 0.5 * dt
        if rows is not None:
            rows.append(torch.stack([0.5 * vv.sum(), 0.5 * u.sum(), 0.5 * w.sum(), vm.sqrt()]))
        if temp is not None and k % every == 0:
            v = v * torch.sqrt(3.0 * (n - 1) * temp / vv.sum())
    return x.cpu().numpy(), v.cpu().numpy(), f.cpu().numpy()


#: Beyond this many steps rounding has grown, along the fluid's chaotic trajectory, to the size
#: of the velocities: there is no 64-bit value to compare with.
_LAST_STEP = 220


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        steps = case["runs"] * case["per_run"]
        if steps > _LAST_STEP:
            return None
        got = []
        for p, v, box in _replicas(case, seed):
            x, v, f = _simulate(p, v, box, steps, RC_SOFT, case["shell"])
            # a replica with steps to go holds the drift of its next step
            v = v + 0.0025 * f
            got.append((x + 0.005 * v, v))
        return dict(pos=np.concatenate([g[0] for g in got]),
                    vel=np.concatenate([g[1] for g in got]), step=None)
    n = _atoms(case)
    pos, vel, box = _start(case["lattice"], case["edge"], case["rho"], case["temp"], seed)
    if kind == "evaluate":
        pos, vel, _ = _start(case["lattice"], case["edge"], case["rho"], case["temp"], seed + 77,
                             amplitude=0.1)
        x = torch.from_numpy(pos).to(_DEV)
        i, j = _pairs(x, box, case["rc"])
        rc = case["rc"]
        f, u, w = _forces(x, box, i, j, rc * rc, 1.0, 1.0, 1.0 if rc == RC_SOFT else 0.0)
        return dict(pos=pos, vel=vel, force=f.cpu().numpy(), u=u.cpu().numpy(), w=w.cpu().numpy())
    if case["steps"] > _LAST_STEP or n * case["steps"] > 3.0e7:
        return None
    rc, species, rows = case.get("rc"), None, None
    if kind == "mixture":
        species = _species(case, len(pos), seed)
        rc = float(species[3].max())
    if kind == "equil":
        rows = []
    x, v, f = _simulate(pos, vel, box, case["steps"], rc, case["shell"], species=species,
                        temp=case["temp"] if kind == "equil" else None, every=20, rows=rows)
    out = dict(pos=x, vel=v, force=f, step=None)
    if rows is not None:
        r = torch.stack(rows).cpu().numpy()
        out["trace"] = {name: np.ascontiguousarray(r[:, k])
                        for k, name in enumerate(("ke", "pe", "virial", "vmax"))}
    return out
