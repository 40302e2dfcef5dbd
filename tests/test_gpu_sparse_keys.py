"""Exclusion keys of explicit chain positions with wide gaps: a system takes device memory in
proportion to its atoms, and its results are those of the same positions without gaps."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

GAP = 10 ** 8     # positions left out inside one molecule; keys stay below 2^27


@pytest.fixture(scope="module")
def mop():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2501_11962_amd as m
    m.lib()
    return m


@pytest.mark.parametrize("pme", [False, True])
def test_wide_gaps_take_no_memory_and_change_no_result(pme, mop):
    import torch
    s = W.water_box(300, seed=5, rc=0.6)
    if pme:
        s = W.with_pme(s)
    # the last two waters as one molecule, its second water 5 or GAP positions up the chain
    mol = np.repeat(np.arange(100), 3)
    mol[297:] = 98
    pos = np.tile([0, 1, 2], 100)
    R = torch.from_numpy(W.random_walk_path(s, 3, 63)[0]).cuda()
    ctx = mop.Context()
    mop.System(ctx, s)
    out = []
    for gap in (5, GAP):
        pos[297:] = gap + np.arange(3)
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        sysm = mop.System(ctx, dict(s, mol=mol, molpos=pos), use_molecules=True)
        taken = free - torch.cuda.mem_get_info()[0]
        print(f"[sparse keys] pme={pme} gap {gap}: {taken / 2**20:.0f} MiB", flush=True)
        # 17 small arrays, each in at most one allocation unit of 2 MiB
        assert taken < 64 * 2 ** 20
        plan = mop.Plan(sysm, 3)
        G, v = mop.veff_grad(plan, R)
        F, U = mop.bead_forces(plan, R)
        assert plan.status() == 0
        out.append([t.cpu().numpy() for t in (G, v, F, U)])
    for a, b in zip(*out):
        assert np.array_equal(a, b)
