"""The forms of binning (a workgroup per bead with its atoms in registers, one without, the
kernels over all beads) inside one call, with displaced configurations, for the Newton-3
kernels' sums, and where the overlap check lists more tasks than it holds."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


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


# 300: registers; 4200 with 74 pair beads: a workgroup each; 30000: few large beads; 1002 in
# 34 x 34 columns: more columns than one workgroup takes.  Paths of two beads have one pair bead,
# which has energies in a launch of its own and in a batch alike.
@pytest.mark.parametrize("mode", [0, 1])
def test_batch_of_all_forms_equals_single_calls(mode, mop, ctx):
    specs = [(300, 2, {}), (4200, 75, {}), (30000, 2, {}), (1002, 2, dict(col_width=0.063))]
    plans, paths = [], []
    for k, (q, n, opts) in enumerate(specs):
        s = W.water_box(q, 70 + k, rc=0.6)
        plans.append(mop.Plan(mop.System(ctx, s), n, **opts))
        paths.append(cuda(W.random_walk_path(s, n, 80 + k)[0]))
    assert plans[3].info()["ncx"] * plans[3].info()["ncy"] > 1024
    bt = mop.Batch(plans, [n for _, n, _ in specs])
    G, v = bt.veff_grad(bt.pack(paths), mode=mode)
    assert bt.status() == 0
    for k, g in enumerate(bt.unpack(G)):
        G1, v1 = mop.veff_grad(plans[k], paths[k], mode=mode)
        assert plans[k].status() == 0
        assert np.array_equal(g.cpu().numpy(), G1.cpu().numpy()), specs[k]
        assert float(v[k]) == float(v1[0]), specs[k]


# 4098: a workgroup per bead without registers for any number of beads; 5100 x 25 too, but by
# the number of its beads.  G of a bead is that of a path of the bead and its neighbours.
@pytest.mark.parametrize("Q,N", [(4098, 3), (5100, 25)])
def test_rebinned_finite_differences_of_large_beads(Q, N, mop, ctx, cl_oracle):
    from oracle import path as OP
    s = W.water_box(Q, 41, rc=0.6)
    R, _, _ = W.random_walk_path(s, N, 42)
    plan = mop.Plan(mop.System(ctx, s), N)
    h = 1e-4
    G, v = mop.veff_grad(plan, cuda(R), mode=1, fd_h=h)
    assert plan.status() == 0
    G = G.cpu().numpy()
    m = cl_oracle.CellModel(s)
    for n in (0, N - 2):
        a, b = max(n - 1, 0), min(n + 2, N)
        want = OP.veff_grad_fd(m, np.ascontiguousarray(R[a:b]), h)[n - a]
        e = float(np.linalg.norm(G[n] - want) / np.linalg.norm(want))
        print(f"[bins fd] {Q}x{N} bead {n}: {e:.2e}", flush=True)
        assert e < 1e-4          # tolerance of the other finite-difference tests
    assert float(v[0]) == float(mop.veff_energy(plan, cuda(R))[0])


@pytest.mark.parametrize("Q,B", [(300, 3), (4098, 2), (5100, 24), (5100, 2)])
def test_newton3_sums_are_clear_on_every_call(Q, B, mop, ctx):
    """The Newton-3 kernels add to sums that the binning clears: two different inputs one after
    the other in a workspace full of large values, against the full-shell kernels (to the
    tolerances of forces and of Hessian-vector products; the two kinds round coordinates
    about different clusters)."""
    s = W.water_box(Q, 43, rc=0.6)
    sysm = mop.System(ctx, s)
    full, plan = mop.Plan(sysm, B), mop.Plan(sysm, B, newton3=True)
    plan.ws[256:].fill_(0x50)
    V = cuda(np.random.default_rng(3).normal(0.0, 1.0, (B, Q, 3)))
    for seed in (44, 45):
        R = cuda(W.random_walk_path(s, B, seed)[0])
        for f, tol in ((lambda p: mop.bead_forces(p, R)[0], 1e-5), (lambda p: mop.bead_hvp(p, R, V), 1e-4)):
            a, b = f(plan).double(), f(full).double()
            assert float((a - b).norm() / b.norm()) < tol
    assert plan.status() == full.status() == 0


def test_overlaps_beyond_the_task_list(mop, ctx):
    """Bins of 0.003 nm make every atom look at three or four bins above its own: 12,000 tasks
    or more for a list of 2048, the rest looked at in place.  Each of these pairs of molecules
    0.006 nm apart along z has to be found, wherever its atom's tasks went; none at 0.05."""
    Q = 4095
    s = W.water_box(Q, 46, rc=0.6)
    R, _, _ = W.random_walk_path(s, 2, 47, 0.0)
    plan = mop.Plan(mop.System(ctx, s), 2, col_width=1.0, zbin=0.003)
    info = plan.info()
    assert info["ncx"] * info["ncy"] * info["nzb"] * 4 < 60000 and info["nzb"] > 1000
    plan.clear_status()
    mop.bead_forces(plan, cuda(R))
    assert plan.status() == 0
    for i in (1, 700, 1402, 2101, 2800, 3499, 4090):
        for d, want in ((0.006, mop.MOP_DEV_OVERLAP), (0.05, 0)):
            R2 = R.copy()
            at = np.array([0.41, 0.37, 0.53]) * s["box"]
            j = i - 3 if i > 3 else i + 3
            R2[1, i], R2[1, j] = at, at + [0.0, 0.0, d]
            plan.clear_status()
            mop.bead_forces(plan, cuda(R2))
            assert plan.status() == want, (i, d)
    plan.clear_status()


@pytest.mark.parametrize("Q", [3000, 6000])
def test_overlaps_in_crowded_bins(Q, mop, ctx):
    """Bins of 1 nm hold a hundred atoms; a pair 0.006 nm apart whose slots lie far from each
    other in one bin is found, and none at 0.05 nm (registers and the separate check)."""
    s = W.water_box(Q, 48, rc=0.6)
    R, _, _ = W.random_walk_path(s, 2, 49, 0.0)
    plan = mop.Plan(mop.System(ctx, s), 2, col_width=1.0, zbin=1.0)
    info = plan.info()
    assert Q / (info["ncx"] * info["ncy"] * info["nzb"]) > 80
    at = (0.5 / np.array([info["ncx"], info["ncy"], info["nzb"]])) * s["box"]   # centre of a bin
    for i, j in ((1, 4), (1, Q - 2), (Q // 2, Q - 5), (Q - 8, 7)):
        for d, want in ((0.006, mop.MOP_DEV_OVERLAP), (0.05, 0)):
            R2 = R.copy()
            # nothing else near: the other sites of the bin's centre move half a box away
            c = R2[1] - at
            c -= s["box"] * np.rint(c / s["box"])
            R2[1][(c ** 2).sum(1) < 0.09 ** 2] += 0.5 * s["box"]
            R2[1, i], R2[1, j] = at, at + [0.0, d, 0.0]
            plan.clear_status()
            mop.bead_forces(plan, cuda(R2))
            assert plan.status() == want, (i, j, d)
    plan.clear_status()
