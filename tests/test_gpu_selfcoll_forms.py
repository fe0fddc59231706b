"""GPU: the self-collision kernels' staging forms at their edges -- the block
table in LDS, or in device memory where it does not fit beside the states,
four states or fewer beside each other -- in both splits, for batches that end inside a
workgroup's chunk, against the FP64 oracle on the same centres."""
import numpy as np
import pytest
import torch

from paper_2603_05493_amd import synth
from tests import parity as P

pytestmark = pytest.mark.gpu

ROBOTS = [("chain3", lambda: synth.serial_chain(3, 1, seed=1)),           # one block
          ("tree60", lambda: synth.random_tree(60, 3, seed=2)),           # 16-bit, table in LDS
          ("tree200", lambda: synth.random_tree(200, 1, seed=3)),         # 16-bit entries would fit, the table not
          ("tree260", lambda: synth.random_tree(260, 1, seed=4)),         # 32-bit entries, four states
          ("tree260x5", lambda: synth.random_tree(260, 5, seed=5))]       # 32-bit entries, one state


@pytest.mark.parametrize("label,factory", ROBOTS)
@pytest.mark.parametrize("B", [1, 6, 131])
@pytest.mark.parametrize("apart", [False, True])
def test_staging_forms(oracle, label, factory, B, apart):
    from paper_2603_05493_amd import wb
    rb = factory()
    if rb.n_spheres > 500 and B > 6:
        B = 13
    r = wb.Robot(rb).to_device("cuda:0")
    rng = np.random.default_rng(B)
    # centres at will: a cloud with collisions, or a wide one with hardly any (the second pass)
    c = synth._f32(rng.normal(size=(B, rb.n_spheres, 3)) * (40.0 if apart else 1.0))
    sph = P.dev(c)
    outs = []
    for split in (False, True):
        r.set_sweep_split(1 << 40 if split else 0)
        outs.append(wb.wb_self_collision(r, sph))
    torch.cuda.synchronize()
    for x, y, nm in zip(*outs, ("max_pen", "argmax", "n_coll")):
        assert torch.equal(x, y), f"{label}: {nm} differs between the two splits"
    mp, am, nc = (t.cpu().numpy() for t in outs[0])
    delta = P.DELTA * (40.0 if apart else 1.0)
    for b in range(B):
        pens = oracle.self_collision_pens(rb, c[b:b + 1])[0]
        ext = np.linalg.norm(c[b], axis=-1).max()
        assert abs(mp[b] - pens.max()) <= P.TOL * ext
        top = np.sort(pens)[-2:] if len(pens) > 1 else np.array([-np.inf, pens[0]])
        if top[1] - top[0] > delta:
            assert am[b] == pens.argmax()
        assert (pens > delta).sum() <= nc[b] <= (pens > -delta).sum()
