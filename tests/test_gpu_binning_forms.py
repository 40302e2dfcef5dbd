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
