"""Finite-difference gradients where the displacement carries an atom over a face of its
column: V_eff belongs to R whatever the binning of R - eps d looks like (mode 1), and the
search on the binning of R finds every pair of the displaced atoms (mode 2).

The systems are charged Lennard-Jones lattices without bonds, with one or a few atoms set
0.4e-4 nm from a column face and moving across it (a path of two beads whose increment is
0.05 nm for those atoms, so that the largest displacement is fd_h = 1e-4 nm, and zero for the
others).
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

FD_H = 1e-4
STEP = 0.05      # nm, of the moving atoms
NEAR = 0.4e-4    # nm, their distance from the face


@pytest.fixture(scope="module")
def mop():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2501_11962_amd as m
    m.lib()
    return m


@pytest.fixture(scope="module")
def ctx(mop):
    return mop.Context()


def cuda(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x, np.float64)).cuda()


def rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def lattice(Q, seed, rc, box=1.97, m=7):
    """Q atoms on a random choice of m^3 sites; forces move nothing by much (small dt / nu)."""
    rng = np.random.default_rng(seed)
    s = dict(W.cfg1(), rc=rc, dt=1e-3, nu=250.0, Q=Q)
    sites = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 3)
    sites = sites[np.sort(rng.permutation(m ** 3)[:Q])]
    s["x"] = (sites + 0.5) * (box / m) + rng.normal(0.0, 0.01, (Q, 3))
    s["box"] = np.full(3, box)
    q = np.where(sites.sum(1) % 2 == 0, 0.4, -0.4)
    s["charge"] = q - q.mean()
    for k in ("mass", "type"):
        s[k] = np.asarray(s[k])[:Q].copy()
    s["sigma"] = np.full_like(np.asarray(s["sigma"], np.float64), 0.24)
    s["mol"], s["molpos"] = np.arange(Q), np.zeros(Q, np.int64)
    return s


def bins(x, L, n):
    u = np.floor((x / L - np.floor(x / L)) * 2.0 ** 32).astype(np.uint64)
    return ((u * np.uint64(n)) >> np.uint64(32)).astype(np.int64)


def columns(s, info, x):
    return bins(x[:, 0], s["box"][0], info["ncx"]) * info["ncy"] + bins(x[:, 1], s["box"][1], info["ncy"])


def slot_total(s, info, x):
    n = np.bincount(columns(s, info, x), minlength=info["ncx"] * info["ncy"])
    return int(((n + 7) // 8 * 8).sum())


def clear_of(x, i, box, dmin=0.2):
    d = x - x[i]
    d -= box * np.rint(d / box)
    r2 = (d ** 2).sum(1)
    r2[i] = 1.0
    return r2.min() > dmin ** 2


def path_with_changed_slots(info, grow):
    """(system, path) whose R^1 - eps d has 8 slots more (grow) or fewer than R^1."""
    for seed in range(200):
        s = lattice(200 + seed % 7, seed, 0.9)
        cw = s["box"][0] / info["ncx"]
        for i in range(s["Q"]):
            x = s["x"].copy()
            face = cw * round(x[i, 0] / cw)
            if not 0.0 < face < s["box"][0]:
                continue
            x[i, 0] = face + NEAR
            y = x.copy()
            y[i, 0] = face + NEAR - FD_H
            change = slot_total(s, info, y) - slot_total(s, info, x)
            if change == (8 if grow else -8) and clear_of(x, i, s["box"]):
                R = np.stack([x, x])
                R[1, i, 0] += STEP
                return s, R
    raise AssertionError("no such path")


@pytest.mark.parametrize("pme", [False, True])
@pytest.mark.parametrize("grow", [False, True])
def test_veff_of_rebinned_finite_differences_is_that_of_the_path(grow, pme, mop, ctx):
    s0 = lattice(200, 0, 0.9)
    s, R = path_with_changed_slots(mop.Plan(mop.System(ctx, s0), 2).info(), grow)
    if pme:
        s = W.with_pme(s)
    plan = mop.Plan(mop.System(ctx, s), 2)
    v0 = float(mop.veff_energy(plan, cuda(R))[0])
    plan.ws[256:].fill_(0x40)        # what an earlier call left is not part of any result
    G, v = mop.veff_grad(plan, cuda(R), mode=1, fd_h=FD_H)
    _, v2 = mop.veff_grad(plan, cuda(R), mode=2, fd_h=FD_H)
    assert plan.status() == 0
    assert float(v2[0]) == v0
    assert float(v[0]) == v0
    if not pme:
        bt = mop.Batch([plan, plan], [2, 1])
        bt.ws[256:].fill_(0x40)
        _, vb = bt.veff_grad(bt.pack([cuda(R), cuda(R[:1])]), mode=1, fd_h=FD_H)
        assert bt.status() == 0
        assert float(vb[0]) == v0


def path_with_straying_references(info, s, seed):
    """A path of two beads in which the fourth atom of as many clusters as possible lies just
    inside an x or y face of its column and is moved across it by +eps d or by -eps d.  (The
    search takes a cluster's fourth slot as its reference.)"""
    rng = np.random.default_rng(seed)
    x = s["x"].copy()
    n = [info["ncx"], info["ncy"]]
    col = columns(s, info, x)
    zb = bins(x[:, 2], s["box"][2], info["nzb"])
    out = np.zeros(x.shape)
    moved = 0
    for c in np.unique(col):
        atoms = np.nonzero(col == c)[0]
        atoms = atoms[np.lexsort((atoms, zb[atoms]))]     # slot order
        for i in atoms[3::8]:
            a, up = int(rng.integers(2)), bool(rng.integers(2))
            w = s["box"][a] / n[a]
            k = (c // n[1]) if a == 0 else (c % n[1])
            y = x.copy()
            y[i, a] = (k + 1) * w - NEAR if up else k * w + NEAR
            if clear_of(y, i, s["box"]):
                x, moved = y, moved + 1
                out[i, a] = STEP * rng.choice([-1.0, 1.0])
    assert np.array_equal(columns(s, info, x), col) and moved >= 10
    return np.stack([x, x + out])


# columns of about rc / 1.9: the outermost column of the stencil starts at half the cut-off
@pytest.mark.parametrize("pme", [False, True])
@pytest.mark.parametrize("how", [dict(newton3=True), dict(list_cap=-1), dict(list_cap=1), dict()])
def test_kept_binning_finds_every_pair_of_displaced_atoms(how, pme, mop, ctx):
    """Finite differences on the binning of R against re-binned ones: searched (Newton-3
    kernels, no lists, lists that overflow) and replayed.  eps is 2e-3, so the FP32 forces (1e3,
    to 1e-7) leave 1e-2 per component beside a gradient of 1e5: 1e-7, held to 1e-5.  A missed
    pair is wrong by its whole force / (4 eps)."""
    if pme and how.get("newton3"):
        pytest.skip("Newton-3 kernels are for reaction field")
    s = lattice(256, 3, 0.6)
    if pme:
        s = W.with_pme(s)
    sysm = mop.System(ctx, s)
    plan = mop.Plan(sysm, 2, col_width=0.6 / 1.9, **how)
    info = plan.info()
    assert info["ncx"] == 6 and info["ncy"] == 6
    R = path_with_straying_references(info, s, 4)
    G2, v2 = mop.veff_grad(plan, cuda(R), mode=2, fd_h=FD_H)
    ref = mop.Plan(sysm, 2)
    G1, v1 = mop.veff_grad(ref, cuda(R), mode=1, fd_h=FD_H)
    assert plan.status() == 0 and ref.status() == 0
    e = rel(G2.cpu().numpy(), G1.cpu().numpy())
    print(f"[fd kept bins] {how} pme={pme}: G {e:.2e}", flush=True)
    assert e < 1e-5
    assert abs(float(v2[0]) - float(v1[0])) < 1e-6 * abs(float(v1[0]))
