"""Performance cases: the calls that a path-dynamics program makes, over their real range.

A program that samples trajectories builds one system, one plan and one path, and then
calls the path gradient (or steps of path dynamics, which contain it) over and over; the
force, Hessian-vector and energy calls serve analysis and preparation.  Every case goes
through the package's public entry points.  Systems are generic and generated here: the
sizes, densities, cutoffs, time steps and path increments are those of the synthetic
workloads of this repository (`workloads`), the Lennard-Jones sizes of the dense mixtures
are chosen to fit their lattice so that the structures need no relaxation.

A case is a dict:
    call    "grad" (exact gradient), "grad_fd" (finite-difference comparison),
            "energy", "forces", "hvp", "pmd" (Langevin steps with bias), "batch"
    system  "crystal", "water", "mixed", "membrane";  Q atoms, N beads (configurations)
    pme     particle-mesh Ewald instead of reaction field
    graph   the call captured once and replayed
    steps   (pmd) steps per call;  paths, qmin, qmax, nmin, nmax (batch)
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_2501_11962_amd as mop

KT = 0.0083144626 * 300.0        # kJ/mol
F_ELEC = 138.935458              # kJ mol^-1 nm e^-2
FD_H = 1e-4                      # nm
TETHER = 0.1                     # mean reversion of a path's beads to the first one
CHAIN = 50                       # atoms of a chain
PMD = dict(tau=0.0005, gamma=250.0, kT=KT, seed=77)
BIAS = dict(sigma=0.02, height=1.0, bias_factor=5.0, kT=KT, stride=2)


# ---- the cases ----------------------------------------------------------------------

def listed():
    def case(name, call, system, Q, N, pme=False, graph=False, **more):
        return dict(name=name, call=call, system=system, Q=Q, N=N, pme=pme, graph=graph, **more)

    return [
        # the smallest path in use (a 256-atom crystal): launches and latency count; as a
        # program calls it, and captured once in a graph as a tight sampling loop does
        case("grad crystal 256x32", "grad", "crystal", 256, 32),
        case("grad crystal 256x32 graph", "grad", "crystal", 256, 32, graph=True),
        # a solvent box, the ordinary size of a first study
        case("grad water 3000x64", "grad", "water", 3000, 64),
        # long path of a mid-sized mixture, ragged atom count, four atom types
        case("grad mixed 22999x96", "grad", "mixed", 22999, 96),
        # the membrane-sized system: the headline size
        case("grad membrane 150000x16", "grad", "membrane", 150000, 16),
        # the same with particle-mesh Ewald, the long-range method of production runs,
        # and at the solvent-box size
        case("grad membrane 150000x16 pme", "grad", "membrane", 150000, 16, pme=True),
        case("grad water 3000x16 pme", "grad", "water", 3000, 16, pme=True),
        # independent paths of uneven sizes in one call
        case("batch 12 water paths", "batch", "water", 0, 0, paths=12, qmin=1000, qmax=20000,
             nmin=16, nmax=128),
        # thermostatted path dynamics with the metadynamics bias: the sampling loop itself
        case("pmd water 3000x16 bias", "pmd", "water", 3000, 16, steps=4),
        # forces and energies of a handful of configurations (analysis, set-up)
        case("forces mixed 4999x7", "forces", "mixed", 4999, 7),
        # Hessian-vector products of a mid-sized mixture
        case("hvp mixed 23000x12", "hvp", "mixed", 23000, 12),
        # the finite-difference form of the Hessian term, kept as the comparison
        case("grad_fd water 3000x32", "grad_fd", "water", 3000, 32),
    ]


def draw(rng: random.Random):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    call = rng.choice(["grad"] * 6 + ["batch", "pmd", "forces", "hvp", "energy", "grad_fd"])
    if call == "batch":
        return dict(call=call, system="water", Q=0, N=0, pme=False, graph=False,
                    paths=rng.randint(2, 12), qmin=log(300, 2000), qmax=log(2500, 16000),
                    nmin=rng.randint(2, 20), nmax=rng.randint(24, 100))
    system = rng.choice(["crystal", "water", "mixed", "membrane"])
    lo, hi = dict(crystal=(200, 60000), water=(300, 90000), mixed=(600, 90000),
                  membrane=(9000, 140000))[system]
    Q = log(lo, hi)
    pme = system != "crystal" and rng.random() < 0.3
    most = (1.2e6 if pme else 2.0e6) * (0.5 if call in ("pmd", "grad_fd") else 1.0)
    N = max(2, min(log(2, 128), int(most / Q)))
    case = dict(call=call, system=system, Q=Q, N=N, pme=pme,
                graph=call == "grad" and rng.random() < 0.25)
    if call == "pmd":
        case["steps"] = rng.randint(1, 4)
    return case


# ---- systems and paths --------------------------------------------------------------

def _serpentine(nx, ny, nz):
    """Lattice indices ordered so that consecutive sites are neighbours."""
    k, j, i = np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
    j = np.where(k % 2 == 0, j, ny - 1 - j)
    row = k * ny + np.arange(ny)[None, :, None]
    i = np.where(row % 2 == 0, i, nx - 1 - i)
    return np.stack([i, j, k], -1).reshape(-1, 3)


def _waters(rng, o):
    """Three-site waters (H, O, H) with random orientations on oxygen positions o."""
    n = len(o)
    u = rng.standard_normal((n, 3))
    u /= np.linalg.norm(u, axis=1, keepdims=True)
    w = np.cross(u, rng.standard_normal((n, 3)))
    w /= np.linalg.norm(w, axis=1, keepdims=True)
    half, r0 = math.radians(104.52) / 2, 0.1
    x = np.stack([o + r0 * (math.cos(half) * u + math.sin(half) * w), o,
                  o + r0 * (math.cos(half) * u - math.sin(half) * w)], 1).reshape(-1, 3)
    b = 3 * np.arange(n)
    bonds = np.stack([b, b + 1, b + 1, b + 2], 1).reshape(-1, 2)
    return (x, np.tile([1.008, 15.999, 1.008], n), np.tile([0.41, -0.82, 0.41], n),
            np.tile([1, 0, 1], n), bonds)


def _chains(first, sites_nm, period, total):
    """Bonds of CHAIN-atom chains on the first CHAIN of every `period` of `total` atoms."""
    s = np.arange(0, total - CHAIN + 1, period)
    i = (s[:, None] + np.arange(CHAIN - 1)).reshape(-1)
    r0 = np.linalg.norm(sites_nm[i + 1] - sites_nm[i], axis=1)
    mol, pos = np.arange(total) + 10 ** 7, np.zeros(total, np.int64)
    a = (s[:, None] + np.arange(CHAIN)).reshape(-1)
    mol[a], pos[a] = np.repeat(np.arange(len(s)), CHAIN), np.tile(np.arange(CHAIN), len(s))
    return first + np.stack([i, i + 1], 1), r0, mol, pos


def _smooth(n):
    while True:
        m = n
        for f in (2, 3, 5, 7):
            while m % f == 0:
                m //= f
        if m == 1:
            return n
        n += 1


def _system(kind, Q, seed, pme):
    rng = np.random.default_rng(seed)
    dt, nu = 0.001, 250.0
    no = np.zeros((0, 2), np.int64)
    if kind == "crystal":
        m = math.ceil(Q ** (1 / 3) - 1e-9)
        a = 0.31
        sites = _serpentine(m, m, m)
        sites = sites[np.sort(rng.permutation(len(sites))[:Q])]
        box = np.full(3, m * a)
        x = (sites + 0.5) * a + rng.normal(0, 0.01, (Q, 3))
        mass, typ = np.full(Q, 16.0), np.zeros(Q)
        charge = np.where(sites.sum(1) % 2 == 0, 0.4, -0.4)
        charge = charge - charge.mean()
        sigma, eps = [0.28], [0.65]
        bonds, r0, kb = no, np.zeros(0), np.zeros(0)
        mol, pos, rc, dt, nu = np.arange(Q), np.zeros(Q), 0.9, 0.002, 5.0
    elif kind == "water":
        n = max(Q // 3, 1)
        L = (3 * n / 100.0) ** (1 / 3)
        m = math.ceil(n ** (1 / 3) - 1e-9)
        sites = _serpentine(m, m, m)
        sites = sites[np.sort(rng.permutation(len(sites))[:n])]
        x, mass, charge, typ, bonds = _waters(rng, (sites + 0.5) * (L / m) + rng.normal(0, 0.005, (n, 3)))
        box = np.full(3, L)
        sigma, eps = [0.27, 0.0], [0.65, 0.0]
        r0, kb = np.full(len(bonds), 0.1), np.full(len(bonds), 345000.0)
        mol, pos, rc = np.repeat(np.arange(n), 3), np.tile([0, 1, 2], n), 1.0
    elif kind == "mixed":
        L = (Q / 101.3) ** (1 / 3)
        m = math.ceil(Q ** (1 / 3) - 1e-9)
        sites = _serpentine(m, m, m)[:Q]
        s = (sites + 0.5) * (L / m)
        box = np.full(3, L)
        bonds, r0, mol, pos = _chains(0, s, 143, Q)      # 35% of the atoms in chains
        x = s + rng.normal(0, 0.008, (Q, 3))
        mass, typ = np.full(Q, 16.0), rng.integers(0, 4, Q)
        charge = rng.normal(0, 0.3, Q)
        charge = charge - charge.mean()
        sigma, eps = np.linspace(0.15, 0.2, 4), np.linspace(0.2, 0.9, 4)
        kb, rc = np.full(len(bonds), 2.5e5), 1.0
    else:
        # dense chain slab (4/15 of the box height) between layers of water, 1 : 1 : 1.5
        Lx = 10.0 * (Q / 150000.0) ** (1 / 3)
        box = np.array([Lx, Lx, 1.5 * Lx])
        nslab = int(round(0.321 * Q))
        nslab += (Q - nslab) % 3
        nx = int(round(Lx / 0.2))
        nz = -(-nslab // (nx * nx))
        h = box[2] * 4 / 15
        s = (_serpentine(nx, nx, nz)[:nslab] + 0.5) * np.array([Lx / nx, Lx / nx, h / nz])
        s = s + np.array([0, 0, 0.5 * (box[2] - h)])
        bonds, r0, mol, pos = _chains(0, s, CHAIN, nslab)
        n = (Q - nslab) // 3
        g = 0.313
        wx = max(1, int(Lx / g))
        wz = -(-n // (wx * wx))
        w = _serpentine(wx, wx, wz)
        w = w[np.sort(rng.permutation(len(w))[:n])]
        o = (w + 0.5) * np.array([Lx / wx, Lx / wx, (box[2] - h) / wz])
        o[:, 2] = np.where(o[:, 2] < 0.5 * (box[2] - h), o[:, 2], o[:, 2] + h)
        wxyz, wm, wq, wt, wb = _waters(rng, o + rng.normal(0, 0.005, o.shape))
        x = np.concatenate([s + rng.normal(0, 0.005, s.shape), wxyz])
        mass = np.concatenate([np.full(nslab, 16.0), wm])
        core = np.hypot(s[:, 0] - 0.5 * Lx, s[:, 1] - 0.5 * Lx) < 0.13 * Lx
        typ = np.concatenate([rng.integers(0, 4, nslab) + np.where(core, 6, 2), wt])
        sq = rng.normal(0, 0.3, nslab)
        charge = np.concatenate([sq - sq.mean(), wq])
        sigma = np.concatenate([[0.27, 0.0], np.linspace(0.14, 0.19, 4), np.linspace(0.14, 0.19, 4)])
        eps = np.concatenate([[0.65, 0.0], np.linspace(0.2, 0.9, 4), np.linspace(0.2, 0.9, 4)])
        bonds = np.concatenate([bonds, wb + nslab])
        r0 = np.concatenate([r0, np.full(len(wb), 0.1)])
        kb = np.concatenate([np.full(len(bonds) - len(wb), 2.5e5), np.full(len(wb), 345000.0)])
        mol = np.concatenate([mol, 10 ** 8 + np.repeat(np.arange(n), 3)])
        pos = np.concatenate([pos, np.tile([0, 1, 2], n)])
        rc = 1.2
    x = np.mod(x, box)
    rc = min(rc, 0.45 * float(box.min()))
    s = dict(Q=len(x), box=box, x=x, mass=mass, charge=charge, type=typ, sigma=np.asarray(sigma),
             epsilon=np.asarray(eps), bonds=bonds, bond_r0=r0, bond_k=kb, mol=mol, molpos=pos,
             rc=rc, eps_rf=78.0, eps_r=1.0, dt=dt, nu=nu)
    if pme:
        s.update(elec="pme", pme_order=4, ewald_rtol=1e-5,
                 pme_grid=[max(_smooth(math.ceil(v / 0.12)), 8) for v in box])
    return s


def _path(s, N, seed):
    """N tethered Brownian beads (N, Q, 3) from the system's structure."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    x0 = torch.from_numpy(s["x"]).cuda()
    step = torch.sqrt(2 * KT * s["dt"] / (torch.from_numpy(s["mass"]).cuda() * s["nu"]))
    if s["nu"] < 10.0:
        step = torch.full_like(step, 0.005)
    R = torch.empty((N, s["Q"], 3), dtype=torch.float64, device="cuda")
    R[0] = x0
    for n in range(N - 1):
        z = torch.randn((s["Q"], 3), dtype=torch.float64, device="cuda", generator=g)
        R[n + 1] = R[n] + TETHER * (x0 - R[n]) + step[:, None] * z
    return R


def _gauss(shape, scale, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return scale * torch.randn(shape, dtype=torch.float64, device="cuda", generator=g)


def _batch_specs(case):
    """(Q, N) of each path: drawn by the case, the same for every seed."""
    rng = random.Random("%(paths)d %(qmin)d %(qmax)d %(nmin)d %(nmax)d" % case)
    out = []
    for _ in range(case["paths"]):
        q = math.exp(rng.uniform(math.log(case["qmin"]), math.log(case["qmax"])))
        out.append((3 * max(int(q / 3), 1), rng.randint(case["nmin"], case["nmax"])))
    return out


def _groups(s):
    """Two groups of atoms, each near one place: a ligand and its pocket."""
    d = s["x"] - 0.5 * s["box"]
    order = np.argsort((d ** 2).sum(1), kind="stable")
    return order[:8].astype(np.int32), order[8:8 + max(1, min(800, s["Q"] // 16))].astype(np.int32)


def _inputs(case, seed):
    """Systems, paths and what else the call takes; no library object."""
    if case["call"] == "batch":
        ss = [_system("water", q, seed * 101 + k, False) for k, (q, _) in enumerate(_batch_specs(case))]
        Rs = [_path(s, n, seed * 101 + 50 + k) for k, (s, (_, n)) in enumerate(zip(ss, _batch_specs(case)))]
        return dict(systems=ss, paths=Rs)
    s = _system(case["system"], case["Q"], seed, case["pme"])
    R = _path(s, case["N"], seed + 1)
    more = dict(system=s, R=R)
    if case["call"] == "hvp":
        more["V"] = _gauss(tuple(R.shape), 1e-3, seed + 2)
    if case["call"] == "pmd":
        more["V"] = _gauss(tuple(R.shape), 1.0, seed + 2) * torch.sqrt(KT / torch.from_numpy(s["mass"]).cuda())[:, None]
    return more


# ---- a pass -------------------------------------------------------------------------

def prepare(case, seed):
    given = _inputs(case, seed)
    ctx = mop.Context()
    state = dict(call=case["call"], ctx=ctx, graph=None)
    if case["call"] == "batch":
        plans = [mop.Plan(mop.System(ctx, s), R.shape[0]) for s, R in zip(given["systems"], given["paths"])]
        batch = mop.Batch(plans, [R.shape[0] for R in given["paths"]])
        state.update(batch=batch, R=batch.pack(given["paths"]))
        return state
    s, R = given["system"], given["R"]
    plan = mop.Plan(mop.System(ctx, s), R.shape[0])
    state.update(plan=plan, R=R, V=given.get("V"))
    if case["call"] == "pmd":
        a, b = _groups(s)
        state["bias"] = mop.Bias(plan, a, b, max_gaussians=100000, **BIAS)
        state["steps"], state["step0"] = case["steps"], 0
        state["G"], _ = mop.veff_grad(plan, R)
        state["bias"].apply(R, state["G"])
    if case["graph"]:
        G, v = mop.veff_grad(plan, R)
        torch.cuda.synchronize()
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        state["graph"], state["out"] = torch.cuda.CUDAGraph(), (G, v)
        with torch.cuda.graph(state["graph"], stream=side):
            ctx.set_stream()
            mop.veff_grad(plan, R, G=G, veff=v)
        ctx.set_stream()
    return state


def run(state):
    call = state["call"]
    if state["graph"] is not None:
        state["graph"].replay()
        return state["out"]
    if call == "grad":
        return mop.veff_grad(state["plan"], state["R"])
    if call == "grad_fd":
        return mop.veff_grad(state["plan"], state["R"], mode=1, fd_h=FD_H)
    if call == "energy":
        return mop.veff_energy(state["plan"], state["R"])
    if call == "forces":
        return mop.bead_forces(state["plan"], state["R"])
    if call == "hvp":
        return mop.bead_hvp(state["plan"], state["R"], state["V"])
    if call == "batch":
        return state["batch"].veff_grad(state["R"])
    E = mop.pmd_step(state["plan"], state["R"], state["V"], state["G"], PMD["tau"], state["steps"],
                     PMD["gamma"], PMD["kT"], PMD["seed"], state["step0"], bias=state["bias"])
    state["step0"] += state["steps"]
    return state["R"], state["V"], state["G"], E


# ---- the work that a pass cannot do without -----------------------------------------

# operations of one pair within the cutoff, each pair once: force, Hessian-vector product
# (with Ewald real space), counted from the pair formulas
PAIR_FLOPS = {False: (33, 58), True: (61, 92)}


def _pairs(kind, Q):
    rho, rc = dict(crystal=(33.6, 0.9), water=(100.0, 1.0), mixed=(101.3, 1.0), membrane=(100.0, 1.2))[kind]
    L = (Q / rho / (1.5 if kind == "membrane" else 1.0)) ** (1 / 3)
    return 0.5 * Q * rho * 4 / 3 * math.pi * min(rc, 0.45 * L) ** 3


def _one_work(call, kind, Q, N, pme, steps=1):
    force, hvp = PAIR_FLOPS[pme]
    beads = dict(forces=N, hvp=N).get(call, max(N - 1, 1))
    passes = dict(grad=force + hvp, pmd=force + hvp, batch=force + hvp, grad_fd=3 * force,
                  energy=force, forces=force, hvp=hvp)[call]
    flops = beads * _pairs(kind, Q) * passes
    if pme:
        K = 580.0 * Q / 100.0
        ffts = dict(grad=4, pmd=4, hvp=4, grad_fd=6, energy=2, forces=2)[call]
        flops += beads * ffts * (2.5 * K * math.log2(K) + Q * 64 * 8)
    per_atom = dict(grad=48, batch=48, grad_fd=48, energy=24, forces=36, hvp=60, pmd=144)[call]
    return steps * Q * N * per_atom, steps * flops


def work(case):
    if case["call"] == "batch":
        each = [_one_work("batch", "water", q, n, False) for q, n in _batch_specs(case)]
        return {"bytes": sum(b for b, _ in each), "flops": sum(f for _, f in each)}
    b, f = _one_work(case["call"], case["system"], case["Q"], case["N"], case["pme"], case.get("steps", 1))
    return {"bytes": b, "flops": f}


# ---- the same in 64 bits, from the definitions --------------------------------------

class _Exact:
    """U(x) of a system in float64 torch; forces and Hessian-vector products by autograd."""

    def __init__(self, s):
        self.s = s
        t = lambda v, dt=torch.float64: torch.as_tensor(np.asarray(v), dtype=dt).cuda()  # noqa: E731
        self.box, self.q, self.typ = t(s["box"]), t(s["charge"]), t(s["type"], torch.int64)
        self.mol, self.pos = t(s["mol"], torch.int64), t(s["molpos"], torch.int64)
        self.sig, self.eps, self.mass = t(s["sigma"]), t(s["epsilon"]), t(s["mass"])
        self.bi, self.bj = t(s["bonds"][:, 0], torch.int64), t(s["bonds"][:, 1], torch.int64)
        self.r0, self.kb = t(s["bond_r0"]), t(s["bond_k"])
        self.K = self.mass * s["nu"] / (2 * s["dt"])
        self.c = s["dt"] / (self.mass * s["nu"])
        self.pme = s.get("elec") == "pme"
        rc, er, erf = s["rc"], s["eps_r"], s["eps_rf"]
        self.f = F_ELEC / er
        self.krf = (erf - er) / ((2 * erf + er) * rc ** 3)
        if self.pme:
            lo, hi = 0.0, 100.0
            for _ in range(200):
                mid = 0.5 * (lo + hi)
                lo, hi = (mid, hi) if math.erfc(mid * rc) > s["ewald_rtol"] else (lo, mid)
            self.beta = 0.5 * (lo + hi)
            self._mesh()

    def mi(self, d):
        return d - self.box * torch.round(d / self.box)

    def pairs(self, x):
        """Indices (i < j) of the atoms closer than the cutoff."""
        Q, rc = x.shape[0], self.s["rc"]
        n = [int(L // rc) for L in self.s["box"]]
        if min(n) < 4:
            n, M = [1, 1, 1], Q
            table = torch.arange(Q, device="cuda")[None]
            near = torch.zeros((1, 1), dtype=torch.int64, device="cuda")
        else:
            nt = torch.tensor(n, device="cuda")
            w = torch.remainder(x, self.box) / self.box
            c = torch.minimum((w * nt).long(), nt - 1)
            cell = (c[:, 0] * n[1] + c[:, 1]) * n[2] + c[:, 2]
            order = torch.argsort(cell, stable=True)
            count = torch.bincount(cell, minlength=n[0] * n[1] * n[2])
            start = torch.cumsum(count, 0) - count
            M = int(count.max())
            k = torch.arange(M, device="cuda")
            table = torch.where(k < count[:, None], order[torch.clamp(start[:, None] + k, max=Q - 1)], -1)
            ids = torch.stack(torch.meshgrid(*[torch.arange(v, device="cuda") for v in n], indexing="ij"), -1).reshape(-1, 3)
            o = torch.tensor([[a, b, e] for a in (-1, 0, 1) for b in (-1, 0, 1) for e in (-1, 0, 1)], device="cuda")
            nb = torch.remainder(ids[:, None] + o, nt)
            near = (nb[..., 0] * n[1] + nb[..., 1]) * n[2] + nb[..., 2]
        out = []
        rows = max(1, int(4e7 / (M * near.shape[1])))   # atoms i at a time
        flat = table.reshape(-1)
        owner = torch.arange(table.shape[0], device="cuda").repeat_interleave(table.shape[1])
        owner, flat = owner[flat >= 0], flat[flat >= 0]
        for k in range(0, len(flat), rows):
            i = flat[k:k + rows]
            j = table[near[owner[k:k + rows]]].reshape(len(i), -1)
            d2 = 0.0
            for a in range(3):
                d = x[:, a][j] - x[i, a][:, None]
                L = float(self.box[a])
                d2 = d2 + (d - L * torch.round(d / L)) ** 2
            keep = (d2 < rc * rc) & (j > i[:, None])
            r, e = torch.nonzero(keep, as_tuple=True)
            out.append((i[r], j[r, e]))
        return torch.cat([p[0] for p in out]), torch.cat([p[1] for p in out])

    def _mesh(self):
        s, p = self.s, 4
        K, V, b = s["pme_grid"], float(self.box.prod()), self.beta

        def M(n, v):
            if n == 2:
                return max(0.0, 1 - abs(v - 1))
            return (v * M(n - 1, v) + (n - v) * M(n - 1, v - 1)) / (n - 1)

        mod, fr = [], []
        for a in range(3):
            m = np.arange(K[a])
            z = sum(M(p, k + 1) * np.exp(2j * np.pi * m * k / K[a]) for k in range(p - 1))
            f = np.where(2 * m < K[a], m, m - K[a]) / s["box"][a]
            n = K[a] // 2 + 1 if a == 2 else K[a]
            mod.append((1 / np.abs(z) ** 2)[:n])
            fr.append((m / s["box"][a])[:n] if a == 2 else f)
        m2 = fr[0][:, None, None] ** 2 + fr[1][None, :, None] ** 2 + fr[2][None, None] ** 2
        B = mod[0][:, None, None] * mod[1][None, :, None] * mod[2][None, None]
        with np.errstate(divide="ignore", invalid="ignore"):
            C = np.where(m2 > 0, np.exp(-np.pi ** 2 * m2 / b ** 2) / (np.pi * V * m2), 0.0)
        w = np.full(K[2] // 2 + 1, 2.0)
        w[0] = 1.0
        if K[2] % 2 == 0:
            w[-1] = 1.0
        self.green = torch.from_numpy(0.5 * self.f * B * C * w).cuda()
        q = self.s["charge"]
        self.e0 = -self.f * b / math.sqrt(math.pi) * float((q ** 2).sum()) \
            - self.f * math.pi * float(q.sum()) ** 2 / (2 * V * b * b)

    def mesh_energy(self, x):
        K = self.s["pme_grid"]
        w, base = [], []
        for a in range(3):
            u = x[:, a] / self.box[a]
            u = K[a] * (u - torch.floor(u).detach())
            b = torch.floor(u.detach())
            f = u - b
            th = [f, 1 - f]
            for n in (3, 4):
                th = [((f + j) * th[j] if j < n - 1 else 0) + ((n - f - j) * th[j - 1] if j else 0) for j in range(n)]
                th = [v / (n - 1) for v in th]
            w.append(torch.stack(th, 1))
            base.append(torch.remainder(b.long()[:, None] - torch.arange(4, device="cuda"), K[a]))
        idx = (base[0][:, :, None, None] * K[1] + base[1][:, None, :, None]) * K[2] + base[2][:, None, None, :]
        val = self.q[:, None, None, None] * w[0][:, :, None, None] * w[1][:, None, :, None] * w[2][:, None, None, :]
        grid = torch.zeros(K[0] * K[1] * K[2], dtype=torch.float64, device="cuda").index_add(0, idx.reshape(-1), val.reshape(-1))
        F = torch.view_as_real(torch.fft.rfftn(grid.reshape(K)))
        return (self.green * (F ** 2).sum(-1)).sum()

    def energy(self, x, i, j):
        s, rc = self.s, self.s["rc"]
        d = self.mi(x[j] - x[i])
        r = torch.sqrt((d ** 2).sum(1))
        ex = (self.mol[i] == self.mol[j]) & ((self.pos[i] - self.pos[j]).abs() <= 2)
        qq = self.f * self.q[i] * self.q[j]
        sg = 0.5 * (self.sig[self.typ[i]] + self.sig[self.typ[j]])
        ep = torch.sqrt(self.eps[self.typ[i]] * self.eps[self.typ[j]])
        c6 = 4 * ep * sg ** 6
        c12 = c6 * sg ** 6
        lj = c12 * r ** -12 - c6 * r ** -6
        lj_c = c12 * rc ** -12 - c6 * rc ** -6
        lj_d = (-12 * c12 * rc ** -12 + 6 * c6 * rc ** -6) / rc
        if self.pme:
            b = self.beta
            psi, psi_c = torch.erfc(b * r) / r, math.erfc(b * rc) / rc
            psi_d = -psi_c / rc - 2 * b / math.sqrt(math.pi) * math.exp(-(b * rc) ** 2) / rc
            out = -qq * torch.erf(b * r) / r
        else:
            psi = 1 / r + self.krf * r ** 2
            psi_c = 1 / rc + self.krf * rc ** 2
            psi_d = -1 / rc ** 2 + 2 * self.krf * rc
            out = torch.zeros_like(r)
        e = lj - lj_c + qq * (psi - psi_c) - (r - rc) * (lj_d + qq * psi_d)
        U = torch.where(ex, out, e).sum()
        rb = torch.sqrt((self.mi(x[self.bj] - x[self.bi]) ** 2).sum(1))
        U = U + (0.5 * self.kb * (rb - self.r0) ** 2).sum()
        if self.pme:
            U = U + self.mesh_energy(x) + self.e0
        return U

    def at(self, x, v=None):
        """U, F and, for v (a tensor or a function of F), H v."""
        i, j = self.pairs(x)
        y = x.detach().clone().requires_grad_(True)
        U = self.energy(y, i, j)
        (g,) = torch.autograd.grad(U, y, create_graph=v is not None)
        F = -g.detach()
        if v is None:
            return U.detach(), F, None
        v = v(F) if callable(v) else v
        (h,) = torch.autograd.grad((g * v).sum(), y)
        return U.detach(), F, h

    def veff(self, R, fd=0.0, grad=True):
        """G (N, Q, 3), V_eff, U(R^1), spring energy (exact or finite-difference form)."""
        N = R.shape[0]
        G = torch.zeros_like(R)
        u1, es = None, torch.zeros((), dtype=torch.float64, device="cuda")
        K, c = self.K[:, None], self.c[:, None]
        for n in range(max(N - 1, 1)):
            keep = []

            def v(F):
                keep.append(self.mi(R[n + 1] - R[n]) - c * F)
                return keep[0]

            U, F, h = self.at(R[n], v if N > 1 and grad and not fd else None)
            if n == 0:
                u1 = U
                G[0] -= F
            if N == 1:
                break
            d = keep[0] if keep else v(F)
            es = es + 0.5 * (K * d ** 2).sum()
            if not grad:
                continue
            if fd:
                e = fd / torch.sqrt((d ** 2).sum(1).max())
                _, fp, _ = self.at(R[n] + e * d)
                _, fm, _ = self.at(R[n] - e * d)
                half = -(fp - fm) / (4 * e)
            else:
                half = 0.5 * h
            G[n] += half - K * d
            G[n + 1] += K * d
        return G, u1 + es, u1, es


def _normals(count, step, seed):
    """The thermostat's deviates (count, 3) of one step: Philox4x64-10 on (index, step)."""
    gen = np.random.Philox(counter=((int(step) << 64) - 1) % (1 << 256), key=int(seed))
    u = (np.floor_divide(gen.random_raw(4 * count), np.uint64(1 << 12)).astype(np.float64) + 0.5) * 2.0 ** -52
    u = u.reshape(count, 4)
    r0, r1 = np.sqrt(-2 * np.log(u[:, 0])), np.sqrt(-2 * np.log(u[:, 2]))
    a0, a1 = 2 * np.pi * u[:, 1], 2 * np.pi * u[:, 3]
    return torch.from_numpy(np.stack([r0 * np.cos(a0), r0 * np.sin(a0), r1 * np.cos(a1)], 1)).cuda()


class _ExactBias:
    def __init__(self, X):
        self.X = X
        a, b = _groups(X.s)
        self.groups = [torch.from_numpy(v.astype(np.int64)).cuda() for v in (a, b)]
        self.hist = []

    def s(self, x):
        m = []
        for g in self.groups:
            w = self.X.mass[g][:, None]
            m.append(x[g[0]] + (w * self.X.mi(x[g] - x[g[0]])).sum(0) / w.sum())
        return torch.sqrt((self.X.mi(m[1] - m[0]) ** 2).sum())

    def apply(self, R, G, deposit):
        ends = [R[0].clone().requires_grad_(True), R[-1].clone().requires_grad_(True)]
        S = self.s(ends[1]) - self.s(ends[0])
        V = sum((w * torch.exp(-(S - c) ** 2 / (2 * BIAS["sigma"] ** 2)) for c, w in self.hist), 0.0 * S)
        g = torch.autograd.grad(V, ends)
        G[0] += g[0]
        G[-1] += g[1]
        V, S = V.detach(), S.detach()
        if deposit:
            self.hist.append((S, BIAS["height"] * torch.exp(-V / (BIAS["kT"] * (BIAS["bias_factor"] - 1)))))
        return V, S


def _exact_pmd(X, R, V, steps):
    tau, c1 = PMD["tau"], math.exp(-PMD["gamma"] * PMD["tau"])
    c2 = math.sqrt((1 - c1 * c1) * PMD["kT"])
    R, V, m = R.clone(), V.clone(), X.mass[:, None]
    bias = _ExactBias(X)
    G, _, _, _ = X.veff(R)
    bias.apply(R, G, False)
    E = []
    for k in range(steps):
        V -= 0.5 * tau * G / m
        R += 0.5 * tau * V
        V = c1 * V + c2 * _normals(R.shape[0] * R.shape[1], k, PMD["seed"]).reshape(R.shape) / torch.sqrt(m)
        R += 0.5 * tau * V
        G, v, _, _ = X.veff(R)
        vb, S = bias.apply(R, G, k % BIAS["stride"] == 0)
        V -= 0.5 * tau * G / m
        E.append(torch.stack([v, 0.5 * (m * V ** 2).sum(), vb, S]))
    return R, V, G, torch.stack(E)


def exact(case, seed):
    given = _inputs(case, seed)
    if case["call"] == "batch":
        each = [_Exact(s).veff(R)[:2] for s, R in zip(given["systems"], given["paths"])]
        return torch.cat([g.reshape(-1) for g, _ in each]), torch.stack([v for _, v in each])
    X, R = _Exact(given["system"]), given["R"]
    call = case["call"]
    if call in ("grad", "grad_fd"):
        G, v, _, _ = X.veff(R, FD_H if call == "grad_fd" else 0.0)
        return G, v.reshape(1)
    if call == "energy":
        _, v, u1, es = X.veff(R, grad=False)
        return torch.stack([v, u1, es])
    if call == "forces":
        each = [X.at(x)[:2] for x in R]
        return torch.stack([f for _, f in each]), torch.stack([u for u, _ in each])
    if call == "hvp":
        return torch.stack([X.at(x, v)[2] for x, v in zip(R, given["V"])])
    return _exact_pmd(X, R, given["V"], case["steps"])
