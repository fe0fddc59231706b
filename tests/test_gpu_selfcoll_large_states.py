"""GPU: self-collision of robots of which 64 KB hold three, two or one state,
up to the largest that is accepted (61,440 bytes of slots a state), in both
splits and at the default threshold, for batches that end inside a workgroup,
against the FP64 oracle on the same centres."""
import numpy as np
import pytest
import torch

from paper_2603_05493_amd import synth
from tests import parity as P

pytestmark = pytest.mark.gpu

ROBOTS = [("three", lambda: synth.random_tree(84, 12, seed=1), 8),      # 17,888 B a state
          ("two", lambda: synth.random_tree(110, 12, seed=2), 5),       # 23,296 B
          ("one_61440", lambda: synth.random_tree(638, 5, seed=3), 3),  # 61,440 B
          ("one_64_slots", lambda: synth.random_tree(56, 64, seed=4), 3)]   # 60,320 B


@pytest.mark.parametrize("label,factory,B", ROBOTS)
@pytest.mark.parametrize("apart", [False, True])
def test_large_states(oracle, label, factory, B, apart):
    from paper_2603_05493_amd import wb
    rb = factory()
    r = wb.Robot(rb).to_device("cuda:0")
    rng = np.random.default_rng(B)
    c = synth._f32(rng.normal(size=(B, rb.n_spheres, 3)) * (40.0 if apart else 1.0))
    sph = P.dev(c)
    outs = []
    for below in (0, 1 << 40, -1):
        r.set_sweep_split(below)
        outs.append(wb.wb_self_collision(r, sph))
    torch.cuda.synchronize()
    for other in outs[1:]:
        for x, y, nm in zip(outs[0], other, ("max_pen", "argmax", "n_coll")):
            assert torch.equal(x, y), f"{label}: {nm} differs between the forms"
    mp, am, nc = (t.cpu().numpy() for t in outs[0])
    delta = P.DELTA * (40.0 if apart else 1.0)
    for b in range(B):
        pens = oracle.self_collision_pens(rb, c[b:b + 1])[0]
        ext = np.linalg.norm(c[b], axis=-1).max()
        assert abs(mp[b] - pens.max()) <= P.TOL * ext
        top = np.partition(pens, -2)[-2:]
        if top[1] - top[0] > delta:
            assert am[b] == pens.argmax()
        assert (pens > delta).sum() <= nc[b] <= (pens > -delta).sum()
