"""Sizes at which the library changes its way of working: binning of a bead in one
workgroup (atoms in registers up to 4096, from memory above, separate launches for few large
beads), the listed stencil of the pair search, excluded-partner maps of Ewald systems, the
one-workgroup tile order of mesh atoms, LDS tiles of the mesh gather, and bias groups and
histories larger than a workgroup.  Every result is compared with the FP64 oracle.

Tolerances are those of the other parity tests (relative L2 per bead: forces 1e-5,
Hessian-vector products 1e-4; energies of beads 1e-5): the FP32 pair terms set the error on
every path.  The bias is FP64 on both sides: a height comes from a sum of at most 1100 Gaussians
whose exponents move by less than 1e-12 with the rounding of S, so 1e-9 leaves room for the
recursion over the deposits.
"""
import numpy as np
import pytest

import workloads as W
from oracle import mop_bias as MB
from oracle.potential import Model

pytestmark = pytest.mark.gpu

TOL_F, TOL_HV, TOL_U, TOL_BIAS = 1e-5, 1e-4, 1e-5, 1e-9


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


def rel(a, b):
    a = np.asarray(a, np.float64)
    b = np.asarray(b, np.float64)
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


def cuda(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x, np.float64)).cuda()


def compare(mop, plan, m, R, beads, what, energy=True):
    """Forces, energy and H v of all beads of R; the listed ones against oracle model m."""
    F, U = mop.bead_forces(plan, cuda(R))
    V = np.random.default_rng(5).normal(0.0, 1.0, R.shape)
    HV = mop.bead_hvp(plan, cuda(R), cuda(V))
    assert plan.status() == 0
    F, U, HV = F.cpu().numpy(), U.cpu().numpy(), HV.cpu().numpy()
    for b in beads:
        ef, eh = rel(F[b], m.forces(R[b])), rel(HV[b], m.hvp(R[b], V[b]))
        print(f"[edges] {what} bead {b}: F {ef:.2e} HV {eh:.2e}", flush=True)
        assert ef < TOL_F and eh < TOL_HV
        if energy:
            u = m.energy(R[b])
            assert abs(U[b] - u) < TOL_U * max(abs(u), 1.0)


# 1023 / 1026: one and two atoms per thread; 4095 / 4098: registers, memory; 5100: few beads
# of a size that goes to separate launches, and with many beads back to one workgroup each
@pytest.mark.parametrize("Q,B", [(1023, 3), (1026, 3), (4095, 2), (4098, 2), (5100, 2), (5100, 24),
                                 (9000, 22)])
def test_bead_binning_at_its_size_limits(Q, B, mop, ctx, cl_oracle):
    s = W.water_box(Q, 600 + Q % 97, rc=0.6)
    R, _, _ = W.random_walk_path(s, B, 61)
    R[B - 1, ::7] += s["box"] * np.array([1.0, -2.0, 3.0])   # unwrapped copies
    compare(mop, mop.Plan(mop.System(ctx, s), B), cl_oracle.CellModel(s), R, [0, B - 1], f"bins {Q}x{B}")


@pytest.mark.parametrize("Q", [258, 4098, 6000])
def test_overlaps_across_faces_of_the_box(Q, mop, ctx):
    """A pair of different molecules 0.006 nm apart (0.0087 in the corner) on both sides of a
    face of the box, which is a face of bins and columns too, sets the status; the same pair
    0.05 nm apart does not."""
    s = W.water_box(Q, 77, rc=0.6)
    R, _, _ = W.random_walk_path(s, 3, 5, 0.0)
    plan = mop.Plan(mop.System(ctx, s), 3)
    L = s["box"]
    for axes in ((0,), (1,), (2,), (0, 1, 2)):
        for d, want in ((0.005, mop.MOP_DEV_OVERLAP), (0.05, 0)):
            R2 = R.copy()
            at = np.array([0.41, 0.37, 0.53]) * L
            p, q = at.copy(), at.copy()
            for a in axes:
                p[a], q[a] = 0.0005, L[a] + 0.0005 - d
            R2[1, 1], R2[1, 4] = p, q
            plan.clear_status()
            mop.bead_forces(plan, cuda(R2))
            assert plan.status() == want, (axes, d)
    plan.clear_status()


# columns far below and above the cut-off; columns that are their own neighbours through
# the box; bins so tall that a column holds more than 256 candidates of one cluster
@pytest.mark.parametrize("cw,zb,waves", [(0.2, 0.05, 4), (0.45, 0.1, 1), (1.0, 0.3, 8), (1.6, 1.0, 2)])
def test_pair_search_over_column_widths(cw, zb, waves, mop, ctx):
    s = W.water_box(1500, 19, rc=1.0)
    R, _, _ = W.random_walk_path(s, 2, 62)
    plan = mop.Plan(mop.System(ctx, s), 2, col_width=cw, zbin=zb, waves=waves)
    compare(mop, plan, Model(s), R, [1], f"search {cw}/{zb}")


@pytest.mark.parametrize("pos", [(0, 1, 2), (0, 1, 0)])
def test_ewald_excluded_partners_with_repeated_positions(pos, mop, ctx):
    """Waters given as molecules: with all three sites at positions of their own, and with both
    hydrogens at one position, where the map from keys to atoms can't be used.  Both exclude
    the three pairs of a water.  (Two atoms at one position count as one atom in the
    erf(beta r) term of excluded pairs, so one of the hydrogens has no charge.)"""
    s = W.with_pme(W.water_box(300, seed=5, rc=0.6))
    s["charge"] = np.tile([0.82, -0.82, 0.0], 100)
    t = dict(s, molpos=np.tile(pos, 100))
    R, _, _ = W.random_walk_path(s, 2, 63)
    plan = mop.Plan(mop.System(ctx, t, use_molecules=True), 2)
    compare(mop, plan, Model(s), R, [1], f"keys {pos}", energy=False)


@pytest.mark.parametrize("Q,grid,order", [(4095, (20, 20, 20), 4), (4098, (20, 20, 20), 4),
                                          (300, (15, 16, 23), 4), (300, (15, 16, 23), 6),
                                          (300, (15, 15, 15), 8), (300, (16, 24, 18), 8)])
def test_mesh_order_and_tiles_at_their_limits(Q, grid, order, mop, ctx, cl_oracle):
    """4096 atoms are the most that one workgroup orders; 15 points are the longest tile (one
    on its axis), 23 the grid whose two tiles differ most."""
    s = W.with_pme(W.water_box(Q, seed=5, rc=0.6), grid=grid, order=order)
    R, _, _ = W.random_walk_path(s, 2, 64)
    R[1, ::5] -= s["box"] * np.array([2.0, 1.0, -1.0])
    compare(mop, mop.Plan(mop.System(ctx, s), 2), cl_oracle.CellModel(s), R, [1], f"mesh {Q} {grid} {order}",
            energy=False)


@pytest.mark.parametrize("na,nb,deposits", [(1, 1, 3), (1500, 1100, 8), (5, 1025, 1100)])
def test_bias_groups_and_histories_beyond_a_workgroup(na, nb, deposits, mop, ctx):
    s = W.water_box(3000, 23, rc=0.6)
    N = 3
    order = np.argsort(s["x"][:, 0], kind="stable").astype(np.int32)
    A, B = order[:na], order[-nb:]
    plan = mop.Plan(mop.System(ctx, s), N)
    args = (0.02, 1.5, 5.0, 2.494)
    bias = mop.Bias(plan, A, B, *args, stride=1, max_gaussians=2048)
    ob = MB.Bias(A, B, s["mass"], s["box"], *args, stride=1)
    paths = [W.random_walk_path(s, N, 40 + k, 0.01)[0] for k in range(8)]
    dev = [cuda(R) for R in paths]
    for k in range(deposits):
        out = bias.apply(dev[k % 8], deposit=True).cpu().numpy()
        S, V, _ = ob.apply(paths[k % 8], step=0)
        assert out[1] == pytest.approx(S, rel=1e-12, abs=1e-14)
        assert out[0] == pytest.approx(V, rel=TOL_BIAS, abs=1e-14)
    c, w = bias.history()
    assert len(c) == deposits
    assert np.allclose(w, ob.heights, rtol=TOL_BIAS, atol=0.0)
    G = cuda(np.zeros_like(paths[0]))
    bias.apply(dev[0], G)
    _, _, Gb = MB.bias_gradient(paths[0], A, B, s["mass"], s["box"], ob.centers, ob.heights, 0.02)
    assert rel(G.cpu().numpy(), Gb) < TOL_BIAS
