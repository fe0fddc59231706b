"""GPU: a robot that took a heavy payload at run time computes as one created
with it, to the bit: the kernels that sum subtrees over lanes in post-order
order siblings by mass, so that little is subtracted from a light branch, and
the order follows an inertia update.  A payload on the first, a middle and the
last tip, taken and put down again; the fused iteration, RNEA and its VJP
without a cache, and a plan created before the update."""
import copy

import numpy as np
import pytest
import torch

from paper_2603_05493_amd import synth
from tests import parity as P

pytestmark = pytest.mark.gpu


def _i6(I):
    return [I[0, 0], I[1, 1], I[2, 2], I[0, 1], I[0, 2], I[1, 2]]


def _all(robots, x, w, plan=None):
    from paper_2603_05493_amd import wb
    from paper_2603_05493_amd.iteration import FusedIteration
    r = robots
    q, qd, qdd = x
    it = FusedIteration(r, q.shape[1], w=w, margin=0.01, hinge_weight=1.0)
    it.run(q, qd, qdd, step=False)
    tau, _ = wb.wb_rnea(r, q, qd, qdd, want_cache=False)
    g = wb.wb_rnea_backward(r, q, qd, qdd, None, w)
    out = [it.tau, it.cost, it.g_q, it.g_qd, it.g_qdd, it.max_pen, it.argmax, it.n_coll, tau, *g]
    pt = torch.empty_like(q)
    (plan or wb.Plan([r], [q.shape[1]])).run([dict(q=q.clone(), qd=qd.clone(), qdd=qdd.clone(), tau=pt)], 1e-3, 0.01, 1.0, 0.0)
    torch.cuda.synchronize()
    return [t.clone() for t in (*out, pt)]


@pytest.mark.parametrize("label,factory", [("humanoid", lambda: synth.humanoid48(seed=0)),
                                           ("tree20", lambda: synth.random_tree(20, 4, seed=17))])
@pytest.mark.parametrize("which", [0, 0.5, 1])
def test_lane_order_follows_the_payload(label, factory, which):
    from paper_2603_05493_amd import wb
    rb, B = factory(), 300
    tips = [k for k in range(rb.n_links) if k not in set(rb.parent.tolist())]
    link = tips[round(which * (len(tips) - 1))]
    heavy = copy.deepcopy(rb)
    heavy.mass = np.array(rb.mass)
    heavy.mass[link] = 30.0
    st = synth.states(rb, B, seed=61, q_range=1.5)
    x = [P.dev(a) for a in (st.q, st.qd, st.qdd)]
    w = P.dev(synth.weights((B, rb.n_dof), seed=62))
    r = wb.Robot(rb).to_device("cuda:0")
    plan = wb.Plan([r], [B])
    empty = _all(r, x, w, plan)
    r.set_link_inertia(link, 30.0, rb.com[link], _i6(rb.inertia[link]))
    for i, (a, b) in enumerate(zip(_all(r, x, w, plan), _all(wb.Robot(heavy).to_device("cuda:0"), x, w))):
        assert torch.equal(a, b), (label, link, i, "with the payload")
    r.set_link_inertia(link, float(rb.mass[link]), rb.com[link], _i6(rb.inertia[link]))
    for i, (a, b) in enumerate(zip(_all(r, x, w, plan), empty)):
        assert torch.equal(a, b), (label, link, i, "put down")
