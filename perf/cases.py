"""The work a user of the solver has it do, as cases that can be timed and compared.

Every case goes through the public entry points (`Plan`, `Batch`, `solve` under
autograd, the particle-mesh calls) at the sizes of the repository's own
workloads: unigrids, nested and mass-refined AMR, batches of uneven hierarchies,
adaptive time steps, periodic boxes, the gradient of a loss, and a particle grid
that is planned anew.  Orders run from the paper's own p = 3 to 8, in the FP64
form and in the mixed FP32 form.  A program that asks for the mixed form asks
for single-precision results, and keeps them in single precision: those cases
end with that conversion.
"""
import math
import random
from functools import lru_cache

import numpy as np
import torch

import paper_2607_19489_amd as A
from paper_2607_19489_amd.pm import ParticleHierarchy, cic_deposit, cic_interpolate

DEV = "cuda"
# pairs up to which exact() sums directly (some seconds of FP64 arithmetic)
DIRECT_PAIRS = 1.0e11


def listed():
    return [
        # the smallest call: a coarse box at the paper's own setting (p = 3, multipoles to the quadrupole); launches
        {"name": "unigrid16_p3_cap", "kind": "solve", "base": 4, "extra": 0, "p": 3, "precision": "fp64", "quad_cap": True},
        # a small uniform box at full precision, as in a test problem or an inner solve
        {"name": "unigrid32_p4", "kind": "solve", "base": 5, "extra": 0, "p": 4, "precision": "fp64"},
        # the ordinary AMR solve: a base grid with one refined region, in both forms
        {"name": "amr2_p6_fp32", "kind": "solve", "base": 6, "extra": 1, "p": 6, "precision": "fp32", "radius": 0.15},
        {"name": "amr2_p6", "kind": "solve", "base": 6, "extra": 1, "p": 6, "precision": "fp64", "radius": 0.15},
        # a periodic (cosmological) box with two nested refinements
        {"name": "periodic_p5", "kind": "solve", "base": 6, "extra": 2, "p": 5, "precision": "fp64", "radius": 0.15,
         "periodic": True, "self_potential": True},
        # the production solve: about 8M leaves on five levels, refined by mass
        {"name": "deep_p6_fp32", "kind": "solve", "base": 7, "extra": 4, "p": 6, "precision": "fp32", "clumps": 32,
         "threshold": 1.25},
        # the sub-cycle of the two finest levels in an adaptive time step
        {"name": "ats_p6_fp32", "kind": "ats", "base": 6, "extra": 3, "p": 6, "precision": "fp32", "clumps": 16,
         "threshold": 2.0},
        # many uneven boxes in one call (parameter scans, training sets), low and high order
        {"name": "batch24_p4_fp32", "kind": "batch", "members": 24, "p": 4, "precision": "fp32"},
        {"name": "batch8_p8_fp32", "kind": "batch", "members": 8, "p": 8, "precision": "fp32"},
        # forward and backward: energy and acceleration losses with respect to the masses, large and small
        {"name": "grad_p6_fp32", "kind": "grad", "base": 7, "extra": 2, "p": 6, "precision": "fp32", "radius": 0.2},
        {"name": "grad_p4", "kind": "grad", "base": 5, "extra": 1, "p": 4, "precision": "fp64", "radius": 0.2},
        # a time step whose particles have moved to other cells: new hierarchy, new plan, deposit, solve, interpolate
        {"name": "follow_p6", "kind": "follow", "base": 6, "extra": 2, "p": 6, "precision": "fp64", "particles": 2},
    ]


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "ats", "batch", "grad", "follow"])
    precision = rng.choice(["fp32", "fp64"])
    p = rng.choice([3, 4, 5, 6, 6, 7, 8])
    c = {"kind": kind, "p": p, "precision": precision}
    if kind == "batch":
        c["members"] = int(round(2.0 ** rng.uniform(0.0, 3.3 if p >= 7 and precision == "fp64" else 4.5)))
        c["geometry"] = rng.randrange(1 << 20)
        return c
    if kind == "follow":
        c.update(base=rng.choice([4, 5, 6]), extra=rng.choice([0, 1, 2]), particles=int(round(2.0 ** rng.uniform(1.0, 6.0))))
        return c
    # base grids of 8^3 to 128^3 cells; the large ones not at the highest orders, nor in FP64 with a gradient
    if kind == "grad" and precision == "fp64":
        p = c["p"] = min(p, 6)
    c["base"] = rng.choice([3, 4, 5, 6, 6] + ([7] if p <= 6 and (kind, precision) != ("grad", "fp64") else []))
    c["extra"] = rng.choice([1, 2, 3] if kind == "ats" else [0, 1, 2] if c["base"] == 7 else [0, 1, 2, 3])
    if rng.random() < 0.5:
        c["radius"] = round(rng.uniform(0.06, 0.2), 4)
    else:
        c["clumps"] = rng.randrange(1, 33)
        c["threshold"] = round(2.0 ** rng.uniform(1.0, 4.0), 3)
        c["geometry"] = rng.randrange(1 << 20)
    if kind == "solve":
        if rng.random() < 0.25:
            c["periodic"] = True
        if rng.random() < 0.25:
            c["quad_cap"] = True
        if rng.random() < 0.25:
            c["self_potential"] = True
    return c


# -- densities and hierarchies ------------------------------------------------

def _density(case):
    """(weight, centre, scale, kind) of the mass components: a Plummer sphere,
    and Gaussian clumps where the case asks for them."""
    parts = [(1.0, (0.5, 0.5, 0.5), 0.05 if case.get("base", 6) >= 6 else 0.1, "plummer")]
    r = random.Random(case.get("geometry", 3))
    for _ in range(case.get("clumps", 0)):
        parts.append((10.0 ** r.uniform(-3.0, -2.0), tuple(r.uniform(0.1, 0.9) for _ in range(3)), r.uniform(0.005, 0.02),
                      "gauss"))
    return parts


def _rho(parts, ijk, level):
    """Density at the centres of cells ijk[n, 3] (float64, on the device)."""
    x = (ijk.double() + 0.5) / float(1 << level)
    out = torch.zeros(x.shape[0], dtype=torch.float64, device=x.device)
    for w, c, s, kind in parts:
        r2 = (x[:, 0] - c[0]).square_().add_((x[:, 1] - c[1]).square()).add_((x[:, 2] - c[2]).square())
        if kind == "plummer":
            out += 3.0 * w / (4.0 * math.pi * s ** 3) * (1.0 + r2 / (s * s)).pow_(-2.5)
        else:
            out += w / ((2.0 * math.pi) ** 1.5 * s ** 3) * torch.exp(-0.5 * r2 / (s * s))
    return out


def _raster(level):
    n = 1 << level
    i = torch.arange(n ** 3, device=DEV)
    return torch.stack([i // (n * n), i // n % n, i % n], 1).int()


def _children(cells):
    o = torch.tensor([[o & 1, o >> 1 & 1, o >> 2] for o in range(8)], device=DEV, dtype=torch.int32)
    return (2 * cells[:, None, :] + o[None]).reshape(-1, 3)


def _dilate(g, periodic):
    for d in range(3):
        up, down = torch.roll(g, 1, d), torch.roll(g, -1, d)
        if not periodic:
            up.select(d, 0).zero_()
            down.select(d, g.shape[d] - 1).zero_()
        g = g | up | down
    return g


def _mask(cells, level):
    n = 1 << level
    g = torch.zeros(n, n, n, dtype=torch.bool, device=DEV)
    c = cells.long()
    g[c[:, 0], c[:, 1], c[:, 2]] = True
    return g


class Grid:
    """A graded hierarchy with the arrays `Plan` takes: the base level in raster
    order, finer levels oct by oct in the order of their fathers."""

    def __init__(self, case):
        base, extra, periodic = case["base"], case["extra"], bool(case.get("periodic"))
        parts = _density(case)
        self.boxlen, self.levelmin = 1.0, base
        wanted, cells = [], _raster(base)
        for lev in range(base, base + extra):
            if "radius" in case:
                x = (cells.double() + 0.5) / float(1 << lev) - 0.5
                w = x.square().sum(1) <= (case["radius"] * 0.5 ** (lev - base)) ** 2
            else:
                w = _rho(parts, cells, lev) * 8.0 ** -lev > case.get("threshold", 8.0) * sum(q[0] for q in parts) * 8.0 ** -base
            wanted.append(cells[w])
            cells = _children(wanted[-1])
        # a refined cell needs the 27 neighbours of its father refined
        for i in range(extra - 1, 0, -1):
            if wanted[i].shape[0]:
                g = _dilate(_mask(wanted[i].div(2, rounding_mode="floor"), base + i - 1), periodic) | _mask(wanted[i - 1], base + i - 1)
                wanted[i - 1] = g.nonzero().int()
        self.ijk, self.ref = [_raster(base)], []
        for i in range(extra):
            c = self.ijk[-1].long()
            self.ref.append(_mask(wanted[i], base + i)[c[:, 0], c[:, 1], c[:, 2]])
            if not bool(self.ref[-1].any()):
                break
            self.ijk.append(_children(self.ijk[-1][self.ref[-1]]))
        if len(self.ref) < len(self.ijk):
            self.ref.append(torch.zeros(self.ijk[-1].shape[0], dtype=torch.bool, device=DEV))
        self.levelmax = base + len(self.ijk) - 1
        self.ncell = np.array([c.shape[0] for c in self.ijk], dtype=np.int64)
        self.total = int(self.ncell.sum())
        self._rho = torch.cat([_rho(parts, c, base + i) * 8.0 ** -(base + i) for i, c in enumerate(self.ijk)])
        self.leaf = ~torch.cat(self.ref)
        self.level = torch.cat([torch.full((c.shape[0],), base + i, dtype=torch.int32, device=DEV) for i, c in enumerate(self.ijk)])
        self._flat_ijk = torch.cat(self.ijk).cpu().numpy()
        self._flat_ref = torch.cat(self.ref).to(torch.uint8).cpu().numpy()

    def flat_ijk(self):
        return self._flat_ijk

    def flat_refined(self):
        return self._flat_ref

    def masses(self, seed):
        """Cell masses with one percent of noise (refined cells have theirs too; the solver passes over them)."""
        g = torch.Generator(device=DEV).manual_seed(seed)
        return self._rho * (1.0 + 0.01 * (2.0 * torch.rand(self.total, dtype=torch.float64, device=DEV, generator=g) - 1.0))

    def centres(self):
        return torch.cat([(c.double() + 0.5) / float(1 << (self.levelmin + i)) for i, c in enumerate(self.ijk)])


def _member_cases(case):
    """Base grids of 16^3 to 64^3 cells with none to three levels above eight times the mean mass."""
    r = random.Random(case.get("geometry", 4000))
    out = []
    for _ in range(case["members"]):
        out.append({"base": r.choice([4, 5, 6]), "extra": r.randrange(4), "clumps": r.choice([0, 8]), "threshold": 8.0,
                    "geometry": r.randrange(1 << 20)})
    return out


def _particles(case, seed):
    """Particles on circular orbits about the centre, anywhere along them."""
    r = random.Random(seed)
    pos = []
    for k in range(case["particles"]):
        rad, a = 0.075 + 0.15 * (k // 2) / max(1, case["particles"]), r.uniform(0.0, 2.0 * math.pi)
        pos.append([0.5 + rad * math.cos(a), 0.5 + rad * math.sin(a), 0.5 + r.uniform(-0.02, 0.02)])
    return np.array(pos), np.full(case["particles"], 0.02 / case["particles"])


def _options(case):
    o = {"p": case["p"], "precision": case["precision"]}
    o.update({k: True for k in ("quad_cap", "self_potential", "periodic") if case.get(k)})
    return o


def _outputs(case, *tensors):
    """The results as the program keeps them: single precision from the mixed form."""
    return [t.float() for t in tensors] if case["precision"] == "fp32" else list(tensors)


# -- one pass -----------------------------------------------------------------

def _buffers(n):
    return (torch.zeros(n, dtype=torch.float64, device=DEV), torch.zeros(n, 3, dtype=torch.float64, device=DEV))


def prepare(case, seed):
    s = {"case": case}
    if case["kind"] == "follow":
        pos, mass = _particles(case, seed)
        s.update(host_pos=pos, pos=torch.from_numpy(pos).to(DEV), pmass=torch.from_numpy(mass).to(DEV))
        return s
    if case["kind"] == "batch":
        grids = [Grid(c) for c in _member_cases(case)]
        plans = [A.Plan(g, **_options(case)) for g in grids]
        s["batch"] = A.Batch(plans)
        for q in plans:
            q.close()
        s["mass"] = [g.masses(seed + 1000 * i) for i, g in enumerate(grids)]
        bufs = [_buffers(g.total) for g in grids]
        s["phi"], s["acc"] = [b[0] for b in bufs], [b[1] for b in bufs]
        return s
    g = Grid(case)
    s["plan"] = A.Plan(g, **_options(case))
    s["phi"], s["acc"] = _buffers(g.total)
    s["mass"] = g.masses(seed)
    if case["kind"] == "ats":
        # the masses of the two finest levels change between the substeps
        s["lmax"] = g.levelmax
        s["steps"] = _ats_steps(g)
        m, s["masses"] = s["mass"], []
        for k, (lev, _) in enumerate(s["steps"]):
            m = torch.where(g.level >= lev, g.masses(seed + 101 + k), m)
            s["masses"].append(m)
        s["plan"].solve(s["mass"], phi=s["phi"], acc=s["acc"])
    elif case["kind"] == "grad":
        s["leaf"] = g.leaf
        s["target"] = torch.zeros(g.total, 3, dtype=torch.float64, device=DEV)
    return s


def _ats_steps(g):
    """The calls of one step of the second finest level: itself, then two steps of the finest."""
    if g.levelmax == g.levelmin:
        return [(g.levelmax, 1)]
    return [(g.levelmax - 1, 2), (g.levelmax, 1), (g.levelmax, 2)]


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "solve":
        return _outputs(case, *state["plan"].solve(state["mass"], phi=state["phi"], acc=state["acc"]))
    if kind == "ats":
        for (lev, icount), m in zip(state["steps"], state["masses"]):
            state["plan"].solve(m, level=lev, icount=icount, phi=state["phi"], acc=state["acc"])
        return _outputs(case, state["phi"], state["acc"])
    if kind == "batch":
        phi, acc = state["batch"].solve(state["mass"], phis=state["phi"], accs=state["acc"])
        return _outputs(case, *phi, *acc)
    if kind == "grad":
        m = state["mass"].detach().requires_grad_(True)
        phi, acc = A.solve(m, state["plan"])
        loss = 0.5 * (m * phi * state["leaf"]).sum() + 0.5 * (acc - state["target"]).square().mean()
        loss.backward()
        return _outputs(case, phi.detach(), acc.detach(), m.grad)
    # follow: what a step of the particle loop does when its grid has to change
    base, top = case["base"], case["base"] + case["extra"]
    h = ParticleHierarchy(state["host_pos"], base, top)
    plan = A.Plan(h, **_options(case))
    mass = torch.zeros(h.total, dtype=torch.float64, device=DEV)
    phi, acc = _buffers(h.total)
    cic_deposit(plan, h.levelmax, state["pos"], state["pmass"], mass)
    plan.solve(mass, phi=phi, acc=acc)
    pacc, pphi = cic_interpolate(plan, h.levelmax, state["pos"], acc, phi)
    plan.close()
    return _outputs(case, pacc, pphi, phi, acc)


# -- work and exact results -----------------------------------------------------

@lru_cache(maxsize=64)
def _counts(items):
    """(bytes, flops, leaves, leaves of the two finest levels) of one solve.  A
    translation of order n meets the (2 n + 1) independent harmonics of that
    order; a pair of cells takes 23 operations."""
    case = dict(items)
    if case["kind"] == "follow":
        h = ParticleHierarchy(_particles(case, 1)[0], case["base"], case["base"] + case["extra"])
    else:
        h = Grid(case)
    opts = {k: v for k, v in _options(case).items() if k not in ("p", "precision")}
    i = A.hierarchy_check(h, p=case["p"], precision=case["precision"], **opts)
    p = case["p"]
    m2l = 2 * sum((2 * n + 1) * (p - n + 1) ** 2 for n in range(p + 1))
    m2p = 2 * ((p + 1) ** 2 + 3 * p ** 2)
    flops = i["m2l_pairs"] * m2l + (i["m2p_pairs"] + i["near_m2p_pairs"]) * m2p + 23.0 * i["p2p_pairs"]
    lv = [int(x) for x in i["leaves_per_level"]]
    fine = (lv[h.levelmax - 1] if h.levelmax > h.levelmin else 0, lv[h.levelmax])
    return 8.0 * i["nleaves"] + 32.0 * i["nleaves"], flops, i["nleaves"], fine


def work(case):
    case = {k: v for k, v in case.items() if k != "name"}
    if case["kind"] == "batch":
        parts = [_counts(tuple(sorted({"kind": "solve", "p": case["p"], "precision": case["precision"], **c}.items())))
                 for c in _member_cases(case)]
        return {"bytes": sum(q[0] for q in parts), "flops": sum(q[1] for q in parts)}
    nbytes, flops, leaves, fine = _counts(tuple(sorted(case.items())))
    if case["kind"] == "grad":  # the backward pass is the transposed map
        return {"bytes": 2.0 * nbytes, "flops": 2.0 * flops}
    if case["kind"] == "ats":  # only the leaves of the solved levels
        solved = fine[0] + 2.0 * fine[1]
        return {"bytes": 40.0 * solved, "flops": flops * solved / leaves}
    return {"bytes": nbytes, "flops": flops}


def _cube_potential():
    """Potential at the centre of a uniform cube of unit side and mass: 3 ln(2 + sqrt 3) - pi / 2."""
    return 3.0 * math.log(2.0 + math.sqrt(3.0)) - 0.5 * math.pi


def _direct(x, xs, m, weights=None):
    """Potential and acceleration at x[n, 3] of the masses m at xs, self pairs left
    out; with `weights` = (phi_bar, acc_bar) instead the transposed sum: at each
    x, sum over xs of phi_bar g + acc_bar . a for a unit mass at x."""
    phi = torch.empty(x.shape[0], dtype=torch.float64, device=x.device)
    acc = torch.empty(x.shape[0], 3, dtype=torch.float64, device=x.device)
    step = max(1, int(2.0e8 / max(1, xs.shape[0])))
    for a in range(0, x.shape[0], step):
        d = [x[a:a + step, i, None] - xs[None, :, i] for i in range(3)]
        inv = (d[0] * d[0] + d[1] * d[1] + d[2] * d[2]).rsqrt_()
        inv.masked_fill_(torch.isinf(inv), 0.0)
        inv3 = inv * inv * inv
        if weights is None:
            phi[a:a + step] = -(inv @ m)
            for i in range(3):
                acc[a:a + step, i] = -((inv3 * d[i]) @ m)
        else:
            phi[a:a + step] = -(inv @ weights[0])
            for i in range(3):
                phi[a:a + step] += (inv3 * d[i]) @ weights[1][:, i].contiguous()
    return phi, acc


def _direct_grid(case, g, mass, solved=None):
    """phi and acc over all cells (0 where nothing is written) by direct summation."""
    at = g.leaf if solved is None else g.leaf & solved
    x = g.centres()
    phi, acc = _buffers(g.total)
    p, a = _direct(x[at], x[g.leaf], mass[g.leaf])
    phi[at], acc[at] = p, a
    if case.get("self_potential"):
        phi[at] -= _cube_potential() * mass[at] * torch.exp2(g.level[at].double())
    return phi, acc


def exact(case, seed):
    """Direct summation in FP64 (the method's own truncation stays in the
    difference), where it takes seconds; none for periodic boxes."""
    if case.get("periodic"):
        return None
    if case["kind"] == "follow":
        return _exact_follow(case, seed)
    if case["kind"] == "batch":
        grids = [Grid(c) for c in _member_cases(case)]
        if sum(float(g.leaf.sum()) ** 2 for g in grids) > DIRECT_PAIRS:
            out = [_direct_grid(case, g, g.masses(seed + 1000 * i)) if float(g.leaf.sum()) ** 2 * len(grids) <= DIRECT_PAIRS
                   else (None, None) for i, g in enumerate(grids)]
        else:
            out = [_direct_grid(case, g, g.masses(seed + 1000 * i)) for i, g in enumerate(grids)]
        return [o[0] for o in out] + [o[1] for o in out]
    g = Grid(case)
    n = float(g.leaf.sum())
    if n * n * (2 if case["kind"] == "grad" else 1) > DIRECT_PAIRS:
        return None
    mass = g.masses(seed)
    if case["kind"] == "solve":
        return list(_direct_grid(case, g, mass))
    if case["kind"] == "ats":
        return _exact_ats(case, g, mass, seed)
    phi, acc = _direct_grid(case, g, mass)
    phib, accb = 0.5 * mass * g.leaf, acc / (3.0 * g.total)
    x = g.centres()[g.leaf]
    back, _ = _direct(x, x, None, (phib[g.leaf], accb[g.leaf]))
    grad = 0.5 * phi * g.leaf
    grad[g.leaf] += back
    return [phi, acc, grad]


def _exact_ats(case, g, mass, seed):
    """Stale trees keep the masses of their last rebuild."""
    phi, acc = _direct_grid(case, g, mass)
    m = held = mass
    for k, (lev, icount) in enumerate(_ats_steps(g)):
        m = torch.where(g.level >= lev, g.masses(seed + 101 + k), m)
        if lev == g.levelmin or icount > 1:
            held = torch.where(g.level >= lev, m, held)
        solved = g.level == lev
        p, a = _direct_grid(case, g, held, solved)
        phi[solved & g.leaf], acc[solved & g.leaf] = p[solved & g.leaf], a[solved & g.leaf]
    return [phi, acc]


def _exact_follow(case, seed):
    """Cloud-in-cell deposit, direct sums between the cells that hold mass, and
    the same weights back (the particles' values; none for the grid's)."""
    pos, mass = _particles(case, seed)
    h = 0.5 ** (case["base"] + case["extra"])
    u = pos / h - 0.5
    i0 = np.floor(u).astype(np.int64)
    f = u - i0
    cells, weights = [], []
    for o in range(8):
        bit = np.array([o & 1, o >> 1 & 1, o >> 2])
        cells.append(i0 + bit)
        weights.append(np.prod(np.where(bit, f, 1.0 - f), axis=1))
    cells, weights = np.stack(cells, 1), np.stack(weights, 1)
    keys, where = np.unique(cells.reshape(-1, 3), axis=0, return_inverse=True)
    where = where.reshape(weights.shape)
    m = np.zeros(len(keys))
    np.add.at(m, where, weights * mass[:, None])
    x = torch.from_numpy((keys + 0.5) * h)
    phi, acc = _direct(x, x, torch.from_numpy(m))
    w, idx = torch.from_numpy(weights), torch.from_numpy(where)
    return [(w[:, :, None] * acc[idx]).sum(1), (w * phi[idx]).sum(1), None, None]
