"""Timed cases of the library's public entry points, and their 64-bit values.

What a user of this library has it do: evaluate the fitness of a genetic
algorithm's population on a training set (``TersoffSet.fitness``), refine its
best members with the fitness gradient (``TersoffSet.fitness_grad``), evaluate
energies, forces and virials of cells (``TersoffSet.tersoff_eval``), repeat the
force call of a large cell (``TersoffSet.eval_call``) and run molecular dynamics
(``md.MD``).  ``listed()`` holds fixed sizes, from one 64-atom cell to 500
candidates on 300 structures; ``draw()`` spreads sizes over the same ranges.

``exact()`` evaluates the same inputs in float64 with plain torch operations
(autograd for every derivative) and none of the library's code.
"""
import math

import numpy as np
import torch

from paper_1909_11474_amd import api
from paper_1909_11474_amd import md as mdlib

R1, R2 = 2.8, 3.2
A_SI = 5.43                 # diamond Si lattice constant (A)
RHO = 0.04996               # atoms / A^3 at 2.33 g/cm^3
MASS_SI = 28.0855           # u
KB = 8.617333262e-5         # eV/K
MV2 = 103.642691            # 1 u A^2/fs^2 in eV
TABLE2 = (3.21481, 1.43134, 2.23801, 0.282818, 0.602568, -0.641048)
# Boxes of the fitted parameters (the GA driver's defaults): D0, alpha, r0,
# beta, n, h, and D0, alpha, r0, S, gamma, n, c, d, h for the Tersoff form.
BOX6 = ((2.0, 1.0, 2.0, 0.1, 0.5, -1.0), (5.0, 2.0, 2.6, 1.0, 1.5, 0.0))
BOX9 = ((2.0, 1.0, 2.0, 1.5, 0.05, 0.5, 0.5, 0.5, -1.0), (5.0, 2.0, 2.6, 3.0, 1.0, 1.5, 3.0, 3.0, 0.0))
# Mean directed bonds and ordered triplets per atom, for work().
BONDS = {"cells": (4.0, 12.0), "mixed": (5.2, 24.0)}


# ----------------------------------------------------------------------------
# Cases
# ----------------------------------------------------------------------------

def listed():
    return [
        # the smallest call: one 64-atom cell, one parameter set, in float64,
        # as a property calculation or a check of a fitted set makes it
        dict(name="eval_cell_fp64", kind="eval", sets="cells", n_struct=1, reps=2, P=1, nx=6, prec="fp64",
             atom_virial=False),
        # finite-displacement phonons: the displaced 216-atom supercells of the
        # force constants, one parameter set in float64
        dict(name="eval_supercells_fp64", kind="eval", sets="cells", n_struct=12, reps=3, P=1, nx=6,
             prec="fp64", atom_virial=False),
        # fitness of a small population on a small uneven training set (odd
        # sizes, early exploration of a fit)
        dict(name="fit_small_fp32", kind="fit", sets="mixed", n_struct=18, P=37, nx=6, prec="fp32"),
        # one GA generation at the paper's population (200) on 100 strained
        # 64-atom cells
        dict(name="fit_cells_fp32", kind="fit", sets="cells", n_struct=100, reps=2, P=200, nx=6, prec="fp32"),
        # one GA generation on the full uneven training set: 300 structures of
        # 8-512 atoms, 500 candidates (the largest call)
        dict(name="fit_mixed_fp32", kind="fit", sets="mixed", n_struct=300, P=500, nx=6, prec="fp32"),
        # a population re-scored in float64 before the final choice
        dict(name="fit_mixed_fp64", kind="fit", sets="mixed", n_struct=60, P=64, nx=6, prec="fp64"),
        # one GA generation of the nine-parameter Tersoff form
        dict(name="fit_form9_fp32", kind="fit", sets="mixed", n_struct=60, P=200, nx=9, prec="fp32"),
        # fitness gradient of a whole population on the full training set
        dict(name="grad_mixed_fp32", kind="grad", sets="mixed", n_struct=300, P=64, nx=6, prec="fp32"),
        # GA refinement step: gradients of the best eight members
        dict(name="grad_refine_fp32", kind="grad", sets="cells", n_struct=100, reps=2, P=8, nx=6, prec="fp32"),
        # float64 gradient of the Tersoff form (final polishing of a fit)
        dict(name="grad_form9_fp64", kind="grad", sets="mixed", n_struct=18, P=5, nx=9, prec="fp64"),
        # the force call of molecular dynamics on a 64,000-atom cell, with
        # per-atom virials and the heat current, in the MD driver's precision
        dict(name="force_64k_fp64", kind="force", reps=20, prec="fp64", nx=6),
        # a short driven MD run (HNEMD) of an 8,000-atom cell with a Verlet
        # skin, from the positions on
        dict(name="md_8k_fp64", kind="md", reps=10, steps=100, prec="fp64", nx=6),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: fitness and gradient calls most often, as in a fit."""
    kind = rng.choice(["fit", "fit", "fit", "grad", "grad", "eval", "force", "md"])
    if kind == "force":
        return dict(kind=kind, reps=rng.randint(5, 20), prec=rng.choice(["fp32", "fp64"]), nx=rng.choice([6, 6, 9]))
    if kind == "md":
        return dict(kind=kind, reps=rng.randint(3, 10), steps=rng.randint(20, 100), prec="fp64", nx=6)
    case = dict(kind=kind, sets=rng.choice(["cells", "mixed", "mixed"]), nx=rng.choice([6, 6, 9]),
                prec=rng.choice(["fp32", "fp32", "fp64"]))
    case["n_struct"] = _log_int(rng, 1, 300)
    if case["sets"] == "cells":
        case["reps"] = rng.randint(1, 4)
    pmax = {"fit": 500, "grad": 64, "eval": 16}[kind]
    # atoms x candidates: below the largest listed call of the kind
    atoms = _atoms(case)
    budget = {"fit": 2.4e7, "grad": 3.0e6, "eval": 4.0e5}[kind] / (4.0 if case["prec"] == "fp64" else 1.0)
    if case["nx"] == 9:
        budget /= 2.0
    case["P"] = _log_int(rng, 1, max(1, min(pmax, int(budget / max(atoms, 1.0)))))
    if kind == "eval":
        case["atom_virial"] = rng.random() < 0.5
    return case


def _atoms(case):
    """Expected atoms of a case."""
    if case["kind"] in ("force", "md"):
        return 8.0 * case["reps"] ** 3
    if case["sets"] == "cells":
        return 8.0 * case["reps"] ** 3 * case["n_struct"]
    return 175.0 * case["n_struct"]


def work(case):
    """Bytes and operations of one pass: positions, reference data and
    parameters read once and outputs written once; per atom and candidate 44
    operations per directed bond and 55 per ordered triplet (the chain rule
    written out), three times that for a gradient."""
    n, nx = _atoms(case), case["nx"]
    S = case.get("n_struct", 1)
    P = case.get("P", 1)
    sets = case.get("sets", "cells")
    b, t = BONDS[sets]
    flops = n * P * (44.0 * b + 55.0 * t)
    geom = 24.0 * n + 72.0 * S + 8.0 * nx * P
    if case["kind"] == "fit":
        return {"bytes": geom + 24.0 * n + 56.0 * S + 32.0 * P, "flops": flops}
    if case["kind"] == "grad":
        return {"bytes": geom + 24.0 * n + 56.0 * S + (32.0 + 8.0 * nx) * P, "flops": 3.0 * flops}
    if case["kind"] == "eval":
        per_atom = 24.0 + (72.0 if case["atom_virial"] else 0.0)
        return {"bytes": geom + P * (per_atom * n + 56.0 * S), "flops": flops}
    if case["kind"] == "force":
        return {"bytes": geom + 24.0 * n + 96.0 * n + 80.0, "flops": flops}
    # each MD step: positions and velocities read and written, forces and
    # per-atom virials written and read
    return {"bytes": geom + case["steps"] * 288.0 * n, "flops": flops * case["steps"]}


# ----------------------------------------------------------------------------
# Inputs
# ----------------------------------------------------------------------------

_BASIS = np.array([[0, 0, 0], [0, 2, 2], [2, 0, 2], [2, 2, 0], [1, 1, 1], [1, 3, 3], [3, 1, 3], [3, 3, 1]]) / 4.0


def _diamond(reps):
    grid = np.stack(np.meshgrid(*[np.arange(n) for n in reps], indexing="ij"), -1).reshape(-1, 3)
    pos = (grid[:, None, :] + _BASIS[None]).reshape(-1, 3) * A_SI
    return pos, np.diag([n * A_SI for n in reps]).astype(np.float64)


def _strained(rng, reps, sigma, vacancies=0):
    pos, cell = _diamond(reps)
    if vacancies:
        pos = pos[np.sort(rng.permutation(len(pos))[vacancies:])]
    eps = np.diag(np.full(3, rng.uniform(-0.02, 0.02)))
    for a, b in ((0, 1), (1, 2), (2, 0)):
        eps[a, b] = eps[b, a] = rng.uniform(-0.02, 0.02)
    F = np.eye(3) + eps
    return pos @ F.T + rng.normal(0.0, sigma, pos.shape), cell @ F.T


def _packing(rng, n, dmin=2.1):
    """Random sequential packing of n atoms, minimum separation dmin."""
    L = (n / RHO) ** (1.0 / 3.0)
    kept = np.empty((n, 3))
    count = 0
    while count < n:
        # a batch of trial points; each accepted one removes the points near it
        pts = rng.uniform(0.0, L, (2 * n, 3))
        for q in range(-count, n):
            if q < 0:
                p = kept[-q - 1]
            elif len(pts) == 0:
                break
            else:
                p = kept[count] = pts[0]
                count += 1
                if count == n:
                    break
            d = np.abs(pts - p)
            d = np.minimum(d, L - d)
            pts = pts[np.einsum("ij,ij->i", d, d) >= dmin * dmin]
    return kept, np.diag([L, L, L])


def _structures(case, rng):
    """Structures of a case: the sizes belong to the case, the rest to rng."""
    sizes = np.random.Generator(np.random.PCG64(case["n_struct"]))
    out = []
    for s in range(case["n_struct"]):
        if case["sets"] == "cells":
            out.append(_strained(rng, (case["reps"],) * 3, 0.1))
            continue
        # a third each: strained supercells, supercells with vacancies, packings
        reps = tuple(int(v) for v in sizes.integers(1, 5, 3))
        vacancies, n = int(sizes.integers(1, 5)), int(sizes.integers(8, 513))
        if s % 3 == 0:
            out.append(_strained(rng, reps, 0.1))
        elif s % 3 == 1:
            out.append(_strained(rng, reps if np.prod(reps) > 1 else (2, 1, 1), 0.1, vacancies))
        else:
            out.append(_packing(rng, n))
    return out


def _joined(structs):
    off = np.concatenate([[0], np.cumsum([len(p) for p, _ in structs])]).astype(np.int64)
    return np.concatenate([p for p, _ in structs]), np.stack([c for _, c in structs]), off


def _params(rng, nx, count):
    lo, hi = (np.asarray(v) for v in (BOX6 if nx == 6 else BOX9))
    return lo + rng.uniform(0.0, 1.0, (count, nx)) * (hi - lo)


def _inputs(case, seed):
    """Host inputs of a case, from the seed alone."""
    rng = np.random.Generator(np.random.PCG64(seed))
    if case["kind"] in ("force", "md"):
        pos, cell = _diamond((case["reps"],) * 3)
        pos = pos + rng.normal(0.0, 0.08 if case["kind"] == "force" else 0.05, pos.shape)
        sig = math.sqrt(KB * 300.0 / (MASS_SI * MV2))
        vel = rng.normal(0.0, sig, pos.shape)
        vel -= vel.mean(axis=0)
        x = np.asarray([TABLE2]) if case["nx"] == 6 else _params(rng, 9, 1)
        mass = rng.choice([27.97692653, 28.97649472, 29.97377022], len(pos), p=[0.9223, 0.0467, 0.0310])
        return dict(pos=pos, cell=cell[None], off=np.array([0, len(pos)]), vel=vel, x=x, mass=mass,
                    fe=(1e-4, 0.0, 0.0))
    pos, cell, off = _joined(_structures(case, rng))
    x = _params(rng, case["nx"], case["P"])
    return dict(pos=pos, cell=cell, off=off, x=x, hidden=_params(rng, case["nx"], 1)[0])


def prepare(case, seed):
    inp = _inputs(case, seed)
    if case["kind"] == "md":
        return dict(case=case, inp=inp)
    ts = api.TersoffSet(inp["pos"], inp["cell"], inp["off"], R1, R2)
    x = torch.as_tensor(inp["x"], dtype=torch.float64, device="cuda")
    if case["kind"] == "force":
        return dict(case=case, call=ts.eval_call(x, precision=case["prec"], atom_virial=True,
                                                 velocities=inp["vel"]))
    if case["kind"] in ("fit", "grad"):
        ts.attach_reference(*_reference(inp))
    return dict(case=case, ts=ts, x=x)


def _stored(case, t):
    """A result as the program stores it.  The library returns float64 arrays
    from both paths; a program that asks for the float32 path, whose results
    carry float32's digits, keeps them in float32."""
    return t.float() if case["prec"] == "fp32" else t


def run(state):
    case = state["case"]
    if case["kind"] == "fit":
        return _stored(case, state["ts"].fitness(state["x"], precision=case["prec"]))
    if case["kind"] == "grad":
        Z, G = state["ts"].fitness_grad(state["x"], precision=case["prec"])
        return _stored(case, Z), _stored(case, G)
    if case["kind"] == "eval":
        out = state["ts"].tersoff_eval(state["x"], precision=case["prec"], atom_virial=case["atom_virial"])
        return {k: _stored(case, v) for k, v in out.items()}
    if case["kind"] == "force":
        return {k: _stored(case, v) for k, v in state["call"]().items()}
    inp = state["inp"]
    sim = mdlib.MD(inp["pos"], inp["cell"][0], inp["x"][0], inp["mass"], inp["vel"], 1.0, R1, R2,
                   precision=case["prec"], fe=inp["fe"], skin=0.5)
    records = sim.run(case["steps"])
    return {"pos": sim.positions(), "vel": sim.velocities(),
            "etot": np.array([r["etot"] for r in records]), "J": np.array([r["J"] for r in records])}


# ----------------------------------------------------------------------------
# The same quantities in plain float64 torch
# ----------------------------------------------------------------------------

def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _pairs(pos, cell, rc):
    """(i, j, shift [nb, 3]) of all pairs (with images) of one structure closer
    than rc, by enumeration."""
    inv = torch.linalg.inv(cell)
    wrap = torch.floor(pos @ inv)
    p = pos - wrap @ cell
    width = 1.0 / torch.linalg.norm(inv, dim=0)
    n = len(p)
    ii, jj, ss = [], [], []
    if bool((width > 2.0 * rc).all()):
        # every neighbour is a nearest image: round the fractional difference
        step = max(1, int(2e7) // n)
        for a in range(0, n, step):
            d = p[None, :, :] - p[a:a + step, None, :]
            sh = -torch.round(d @ inv)
            r2 = ((d + sh @ cell) ** 2).sum(-1)
            r2[torch.arange(len(r2)), torch.arange(a, a + len(r2))] = 1e30
            i, j = torch.nonzero(r2 < rc * rc, as_tuple=True)
            ii.append(i + a)
            jj.append(j)
            ss.append(sh[i, j])
    else:
        m = [int(math.ceil(rc / float(w))) for w in width]
        grid = torch.cartesian_prod(*[torch.arange(-k, k + 1, device=p.device) for k in m]).to(p.dtype)
        d = p[None, :, :] - p[:, None, :]
        for sh in grid:
            r2 = ((d + sh @ cell) ** 2).sum(-1)
            if not bool(sh.any()):
                r2.fill_diagonal_(1e30)
            i, j = torch.nonzero(r2 < rc * rc, as_tuple=True)
            ii.append(i)
            jj.append(j)
            ss.append(sh.expand(len(i), 3))
    i, j, s = torch.cat(ii), torch.cat(jj), torch.cat(ss)
    return i, j, s - wrap[j] + wrap[i]


class _Plain:
    """Padded neighbour table of a set and the potential on it."""

    def __init__(self, pos, cell, off, rc=R2):
        dev = _device()
        self.pos = torch.as_tensor(pos, dtype=torch.float64, device=dev)
        self.off = [int(v) for v in off]
        self.N, self.S = self.off[-1], len(self.off) - 1
        cell = torch.as_tensor(cell, dtype=torch.float64, device=dev)
        ii, jj, vv = [], [], []
        for s in range(self.S):
            a, b = self.off[s], self.off[s + 1]
            i, j, sh = _pairs(self.pos[a:b], cell[s], rc)
            ii.append(i + a)
            jj.append(j + a)
            vv.append(sh @ cell[s])
        i, j, v = torch.cat(ii), torch.cat(jj), torch.cat(vv)
        order = torch.argsort(i, stable=True)
        i, j, v = i[order], j[order], v[order]
        count = torch.bincount(i, minlength=self.N)
        self.M = max(1, int(count.max()) if len(i) else 1)
        slot = torch.arange(len(i), device=dev) - (torch.cumsum(count, 0) - count)[i]
        self.mask = torch.zeros(self.N, self.M, dtype=torch.bool, device=dev)
        self.mask[i, slot] = True
        self.j = torch.zeros(self.N, self.M, dtype=torch.long, device=dev)
        self.j[i, slot] = j
        self.shift = torch.zeros(self.N, self.M, 3, dtype=torch.float64, device=dev)
        self.shift[i, slot] = v
        self.sid = torch.repeat_interleave(torch.arange(self.S, device=dev),
                                           torch.as_tensor(np.diff(self.off), device=dev))
        self.size = torch.as_tensor(np.diff(self.off), dtype=torch.float64, device=dev)

    def vectors(self, pos=None):
        p = self.pos if pos is None else pos
        d = p[self.j] + self.shift - p[:, None, :]
        far = torch.tensor([2.0 * R2, 0.0, 0.0], dtype=torch.float64, device=p.device)
        return torch.where(self.mask[..., None], d, far)

    def site_energy(self, d, x):
        """U_i for bond vectors d [N, M, 3] and a parameter vector x (tensor)."""
        r = torch.sqrt((d * d).sum(-1))
        u = d / r[..., None]
        fc = torch.where(r <= R1, torch.ones_like(r),
                         torch.where(r >= R2, torch.zeros_like(r),
                                     0.5 * (1.0 + torch.cos(math.pi * (r - R1) / (R2 - R1)))))
        fc = torch.where(self.mask, fc, torch.zeros_like(fc))
        if len(x) == 6:
            D0, al, r0, beta, n, h = x
            t = u @ u.transpose(1, 2).contiguous() - h
            g = beta * t * t
            fR, fA = D0 * torch.exp(-2.0 * al * (r - r0)), 2.0 * D0 * torch.exp(-al * (r - r0))
        else:
            D0, al, r0, S, gam, n, c, dd, h = x
            t = u @ u.transpose(1, 2).contiguous() - h
            g = gam * (1.0 + (c * c / (dd * dd)) * (t * t / (dd * dd + t * t)))
            fR = D0 / (S - 1.0) * torch.exp(-al * torch.sqrt(2.0 * S) * (r - r0))
            fA = S * D0 / (S - 1.0) * torch.exp(-al * torch.sqrt(2.0 / S) * (r - r0))
        eye = torch.eye(self.M, dtype=torch.bool, device=d.device)
        zeta = (torch.where(eye, torch.zeros_like(g), g) * fc[:, None, :]).sum(-1)
        pos = zeta > 0
        z = torch.where(pos, zeta, torch.ones_like(zeta))
        b = torch.where(pos, (1.0 + z ** n) ** (-0.5 / n), torch.ones_like(z))
        return 0.5 * (fc * (fR - b * fA)).sum(-1)

    def evaluate(self, x, pos=None, graph=False, per_atom=False):
        """E [S], F [N, 3], W [S, 6] (and W_i [N, 3, 3]) of one parameter set."""
        d = self.vectors(pos).detach().requires_grad_(True)
        U = self.site_energy(d, x)
        (G,) = torch.autograd.grad(U.sum(), d, create_graph=graph)
        Gm = torch.where(self.mask[..., None], G, torch.zeros_like(G))
        E = torch.zeros(self.S, dtype=U.dtype, device=U.device).index_add(0, self.sid, U)
        F = Gm.sum(1).index_add(0, self.j.reshape(-1), -Gm.reshape(-1, 3))
        w = -(d[..., :, None] * Gm[..., None, :])
        ws = w.sum(1).reshape(self.N, 9)
        W9 = torch.zeros(self.S, 9, dtype=U.dtype, device=U.device).index_add(0, self.sid, ws)
        out = [E, F, W9[:, [0, 4, 8, 5, 6, 1]]]
        if per_atom:
            out.append(torch.zeros(self.N, 9, dtype=U.dtype, device=U.device)
                       .index_add(0, self.j.reshape(-1), w.reshape(-1, 9)).reshape(self.N, 3, 3))
        return out

    def fitness(self, x, ref, graph=False):
        """Z, Z_e, Z_v, Z_f of one parameter set."""
        E, F, W = self.evaluate(x, graph=graph)
        e, w, f = ref
        z = [torch.sqrt(((E / self.size - e) ** 2).sum() / (e * e).sum()),
             torch.sqrt(((W / self.size[:, None] - w) ** 2).sum() / (w * w).sum()),
             torch.sqrt(((F - f) ** 2).sum() / (f * f).sum())]
        return torch.stack([z[0] + z[1] + z[2]] + z)


def _reference(inp, plain=None):
    """Reference energies, virials per atom and forces: the potential at the
    hidden parameter set."""
    plain = plain or _Plain(inp["pos"], inp["cell"], inp["off"])
    E, F, W = plain.evaluate(torch.as_tensor(inp["hidden"], device=plain.pos.device))
    return (E / plain.size).detach(), (W / plain.size[:, None]).detach(), F.detach()


def exact(case, seed):
    inp = _inputs(case, seed)
    dev = _device()
    if case["kind"] == "md":
        return _exact_md(case, inp)
    plain = _Plain(inp["pos"], inp["cell"], inp["off"])
    xs = torch.as_tensor(inp["x"], dtype=torch.float64, device=dev)
    if case["kind"] == "fit":
        ref = _reference(inp, plain)
        return torch.stack([plain.fitness(x, ref).detach() for x in xs])
    if case["kind"] == "grad":
        ref = _reference(inp, plain)
        Z, G = [], []
        for x in xs:
            x = x.clone().requires_grad_(True)
            z = plain.fitness(x, ref, graph=True)
            (g,) = torch.autograd.grad(z[0], x)
            Z.append(z.detach())
            G.append(g)
        return torch.stack(Z), torch.stack(G)
    virial = case["kind"] == "force" or case["atom_virial"]
    res = [[t.detach() for t in plain.evaluate(x, per_atom=virial)] for x in xs]
    out = {k: torch.stack([r[q] for r in res]) for q, k in enumerate(["E", "F", "W"] + ["Wi"] * virial)}
    if case["kind"] == "force":
        vel = torch.as_tensor(inp["vel"], device=dev)
        out["J"] = (out["Wi"] @ vel[None, :, :, None]).squeeze(-1).sum(1)
    return out


def _exact_md(case, inp):
    """Velocity Verlet with the driving force F_ext,i = W_i^T F_e minus its mean."""
    dev = _device()
    plain = _Plain(inp["pos"], inp["cell"], inp["off"], rc=R2 + 0.5)
    x = torch.as_tensor(inp["x"][0], dtype=torch.float64, device=dev)
    pos, vel = plain.pos.clone(), torch.as_tensor(inp["vel"], device=dev).clone()
    mass = torch.as_tensor(inp["mass"], device=dev)[:, None]
    fe = torch.tensor(inp["fe"], dtype=torch.float64, device=dev)
    origin = pos.clone()
    etot, heat = [], []

    def forces():
        E, F, _, Wi = plain.evaluate(x, pos=pos, per_atom=True)
        ext = (Wi * fe[None, :, None]).sum(1)
        return E.detach(), (F + ext - ext.mean(0)).detach(), Wi.detach()

    E, F, Wi = forces()
    for _ in range(case["steps"]):
        vel = vel + 0.5 * F / (mass * MV2)
        pos = pos + vel
        if float(((pos - origin) ** 2).sum(1).max()) >= 0.0625:
            plain = _Plain(pos.cpu().numpy(), inp["cell"], inp["off"], rc=R2 + 0.5)
            origin = pos.clone()
        E, F, Wi = forces()
        heat.append((Wi @ vel[:, :, None]).squeeze(-1).sum(0))
        vel = vel + 0.5 * F / (mass * MV2)
        etot.append(E[0] + 0.5 * MV2 * (mass * vel * vel).sum())
    return {"pos": pos.cpu().numpy(), "vel": vel.cpu().numpy(),
            "etot": torch.stack(etot).cpu().numpy(), "J": torch.stack(heat).cpu().numpy()}
