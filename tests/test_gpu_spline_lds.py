"""GPU: the one-launch B-spline step where its LDS is largest: shapes whose
counted bytes, by which they are accepted, fill 64 KB while the launch takes
68 KB of the 160 KB that a workgroup may have.  Its control-point gradient and
per-sample outputs against the two-launch form, and the first shape past the
edge refused."""
import numpy as np
import pytest
import torch

from paper_2603_05493_amd import synth
from tests import parity as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("links,spheres,K", [(35, 12, 35), (37, 12, 30)])
def test_one_launch_at_the_lds_edge(links, spheres, K):
    from paper_2603_05493_amd import wb
    from paper_2603_05493_amd.iteration import BsplineIteration
    rb = synth.random_tree(links - 1, spheres, seed=1)
    d, T = rb.n_dof, 5
    rng = np.random.default_rng(51)
    U = torch.from_numpy(synth._f32(rng.uniform(-1.2, 1.2, (d, T, K))).astype(np.float32)).cuda()
    th0 = torch.from_numpy(synth._f32(rng.uniform(-1.2, 1.2, (d, T))).astype(np.float32)).cuda()
    r = wb.Robot(rb).to_device("cuda:0")
    a, b = (BsplineIteration(r, U.clone(), th0, dt=0.05, torque_weight=1e-3, margin=0.01, hinge_weight=1.0, form=f)
            for f in ("two_launch", "one_launch"))
    a.run(step=False)
    b.run(step=False)
    torch.cuda.synchronize()
    by_traj = lambda t: t.permute(1, 0, 2).reshape(T, -1).double().cpu().numpy()
    assert P.normwise(by_traj(b.g_U), by_traj(a.g_U), floor=1e-6).max() < P.TOL
    for k in ("tau", "g_qd", "g_qdd"):
        assert P.normwise(P.host(getattr(b.fused, k)), P.host(getattr(a.fused, k)), floor=1e-6).max() < P.TOL, k
    wide = U.repeat(1, 1, 2)
    past = BsplineIteration(r, wide, th0, dt=0.05, torque_weight=1e-3, margin=0.01, hinge_weight=1.0, form="one_launch")
    with pytest.raises(Exception, match="LDS"):
        past.run(step=False)
