"""Mesh tiles with many atoms, whose potentials several workgroups gather: one tile (a grid of
15 points per axis) at the edges of a part, and eight tiles of 9 points per axis with two
parts each; forces and Hessian-vector products against the FP64 oracle, at the
tolerances of the other parity tests."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Q,grid,order", [(255, 15, 4), (258, 15, 4), (513, 15, 4), (3000, 15, 4),
                                          (3000, 15, 8), (4098, 18, 6)])
def test_crowded_tiles(Q, grid, order, cl_oracle):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2501_11962_amd as mop
    s = W.with_pme(W.water_box(Q, seed=6, rc=0.6), grid=(grid,) * 3, order=order)
    R, _, _ = W.random_walk_path(s, 2, 65)
    # the second bead wrapped into the box, the first as it walked
    R[1] = np.mod(R[1], s["box"])
    V = np.random.default_rng(7).normal(0.0, 1.0, R.shape)
    plan = mop.Plan(mop.System(mop.Context(), s), 2)
    cuda = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    F, _ = mop.bead_forces(plan, cuda(R))
    H = mop.bead_hvp(plan, cuda(R), cuda(V))
    assert plan.status() == 0
    m = cl_oracle.CellModel(s)
    for b in range(2):
        f, h = m.forces(R[b]), m.hvp(R[b], V[b])
        ef = float(np.linalg.norm(F[b].cpu().numpy() - f) / np.linalg.norm(f))
        eh = float(np.linalg.norm(H[b].cpu().numpy() - h) / np.linalg.norm(h))
        print(f"[tiles] {Q} {grid} {order} bead {b}: F {ef:.2e} HV {eh:.2e}", flush=True)
        assert ef < 1e-5 and eh < 1e-4
