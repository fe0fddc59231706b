"""GPU: torques and joint-angle gradients of the forms that sum wrenches about
the world origin over a scan (RNEA and its VJP without a cache, the fused
iteration) stay within twice the error, over all joints and states, of the
recursion in link coordinates in float32 on the CPU: the scans' differences
of accumulated forces must leave no rounding of their own."""
import numpy as np
import pytest
import torch

from paper_2603_05493_amd import synth
from tests import parity as P
from tests import recursion

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("label,factory", [("tree12", lambda: synth.random_tree(12, 2, seed=0)),
                                           ("tree37", lambda: synth.random_tree(37, 2, seed=945)),
                                           ("tree48", lambda: synth.random_tree(48, 2, seed=3)),
                                           ("humanoid", lambda: synth.humanoid48(seed=0))])
def test_torque_and_angle_gradient(oracle, label, factory):
    from paper_2603_05493_amd import wb
    from paper_2603_05493_amd.iteration import FusedIteration
    rb, B = factory(), 1003
    r = wb.Robot(rb).to_device("cuda:0")
    st = synth.states(rb, B, seed=41, q_range=np.pi)
    w = synth.weights((B, rb.n_dof), seed=42)
    x = [P.dev(a) for a in (st.q, st.qd, st.qdd)]
    tau, _ = wb.wb_rnea(r, *x, want_cache=False)
    g_q = wb.wb_rnea_backward(r, *x, None, P.dev(w))[0]
    it = FusedIteration(r, B, w=P.dev(w), margin=0.01, hinge_weight=0.0)
    it.run(*x, step=False)
    torch.cuda.synchronize()
    args = (rb, st.q, st.qd, st.qdd)
    ref = dict(tau=oracle.rnea(*args), g_q=oracle.rnea_vjp(*args, w)[0])
    yard = recursion.rnea_and_vjp(rb, st, w, torch.float32)
    for form, got in (("lanes", dict(tau=tau, g_q=g_q)), ("fused", dict(tau=it.tau, g_q=it.g_q))):
        for k, t in got.items():
            err, bound = np.linalg.norm(P.host(t) - ref[k]), 2.0 * np.linalg.norm(yard[k] - ref[k])
            print(label, form, k, f"error {err / np.linalg.norm(ref[k]):.2e}, of the bound {err / bound:.2f}")
            assert err <= bound, (label, form, k)
