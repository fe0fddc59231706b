"""GPU: the fused iteration at the edges of its sweep tables, against the FP64
oracle: one block, robots whose four wavefronts and block table are counted
at just under and over 64 KB of LDS (a launch takes a quarter), and one with far links (a wide rounding margin in
the bounding spheres); 64- and 16-lane groups."""
import numpy as np
import pytest
import torch

from paper_2603_05493_amd import synth
from tests import parity as P

pytestmark = pytest.mark.gpu


def _far():
    rb = synth.random_tree(9, 3, seed=12)
    rb.fixed_p = synth._f32(np.asarray(rb.fixed_p) * 20.0)
    return rb


def _balled():
    """Every link within reach of every other: the survivors of the broad phase overflow its list."""
    rb = synth.random_tree(40, 2, seed=13)
    rb.fixed_p = synth._f32(np.asarray(rb.fixed_p) * 0.02)
    return rb


ROBOTS = [("balled41", _balled), ("chain3", lambda: synth.serial_chain(3, 1, seed=1)), ("tree53x12", lambda: synth.random_tree(52, 12, seed=2)),
          ("tree55x12", lambda: synth.random_tree(54, 12, seed=3)), ("far10", _far)]


@pytest.mark.parametrize("label,factory", ROBOTS)
@pytest.mark.parametrize("B", [1, 67])
def test_fused_iteration_at_table_limits(oracle, label, factory, B):
    from paper_2603_05493_amd import wb
    from paper_2603_05493_amd.iteration import FusedIteration
    rb = factory()
    r = wb.Robot(rb).to_device("cuda:0")
    assert r.fused_supported
    st = synth.states(rb, B, seed=4, q_range=1.5)
    w = synth.weights((B, rb.n_dof), seed=5)
    it = FusedIteration(r, B, w=P.dev(w), margin=0.01, hinge_weight=1.0)
    it.run(P.dev(st.q), P.dev(st.qd), P.dev(st.qdd), step=False)
    torch.cuda.synchronize()
    _, _, c = oracle.fk(rb, st.q)
    ext = P.extent(c)
    pens = oracle.self_collision_pens(rb, c)
    mp = it.max_pen.cpu().numpy().astype(np.float64)
    assert P.scaled(mp[:, None], pens.max(1)[:, None], ext).max() < P.TOL
    delta = P.DELTA * np.maximum(ext, 1.0)[:, None]
    nc = it.n_coll.cpu().numpy()
    assert np.all((nc >= (pens > delta).sum(1)) & (nc <= (pens > -delta).sum(1)))
    top = np.sort(pens, 1)
    clear = (top[:, -1] - (top[:, -2] if pens.shape[1] > 1 else -np.inf)) > delta[:, 0]
    assert np.array_equal(it.argmax.cpu().numpy()[clear], pens.argmax(1)[clear])
    assert P.normwise(P.host(it.tau), oracle.rnea(rb, st.q, st.qd, st.qdd), floor=1e-3).max() < P.TOL
    ref = oracle.rnea_vjp(rb, st.q, st.qd, st.qdd, w)
    am = it.argmax.cpu().numpy()
    gc = oracle.self_collision_backward(rb, c, am, mp, 0.01, np.ones(B))
    g_q = ref[0] + oracle.fk_backward(rb, st.q, g_spheres=gc)
    for got, want in ((it.g_q, g_q), (it.g_qd, ref[1]), (it.g_qdd, ref[2])):
        assert P.normwise(P.host(got), want, floor=1e-6).max() < P.TOL
