"""GPU: self-collision of robots with so few rows that the wave form evaluates
all of them without a test, at the edge of that rule (120, 128 and 136 rows)
and well inside it, in both forms, against the FP64 oracle on the same centres:
crowded clouds, and wide ones whose states take the second pass; and exact
ties, of which the lowest pair is reported."""
import numpy as np
import pytest
import torch

from paper_2603_05493_amd import synth
from tests import parity as P
from tests import test_gpu_selfcoll_large_states as large

pytestmark = pytest.mark.gpu


def _blocks(n, spheres):
    """Seven links of which n pairs are checked."""
    rb = synth.serial_chain(6, spheres, seed=7)
    rb.allow = np.zeros((rb.n_links, rb.n_links), np.uint8)
    pairs = [(a, b) for a in range(7) for b in range(a + 1, 7)][:n]
    for a, b in pairs:
        rb.allow[a, b] = rb.allow[b, a] = 1
    return rb


ROBOTS = [("chain3", lambda: synth.serial_chain(3, 5, seed=1), 70), ("chain7", lambda: synth.serial_chain(7, 5, seed=0), 133),
          ("rows120", lambda: _blocks(15, 8), 66), ("rows128", lambda: _blocks(16, 8), 66),
          ("rows136", lambda: _blocks(17, 8), 66), ("slots16", lambda: _blocks(8, 16), 34)]


@pytest.mark.parametrize("label,factory,B", ROBOTS)
@pytest.mark.parametrize("apart", [False, True])
def test_few_rows(oracle, label, factory, B, apart):
    large.test_large_states(oracle, label, factory, B, apart)


def test_exact_tie():
    from paper_2603_05493_amd import wb
    rb = _blocks(16, 8)
    rb.sphere_r = synth._f32(np.full(rb.n_spheres, 0.05))
    r = wb.Robot(rb).to_device("cuda:0")
    for scale in (0.01, 10.0):   # every pair collides, or none
        c = np.zeros((5, rb.n_spheres, 3))
        link = np.asarray(rb.sphere_link)
        c[:, :, 0] = scale * (link % 2)   # spheres of even and of odd links coincide: many equal distances
        outs = []
        for below in (0, 1 << 40):
            r.set_sweep_split(below)
            outs.append(wb.wb_self_collision(r, P.dev(c)))
        torch.cuda.synchronize()
        for x, y in zip(*outs):
            assert torch.equal(x, y)
        s, t = (np.asarray(a) for a in r.pairs())
        d = np.abs(c[0, s, 0] - c[0, t, 0])
        assert (outs[0][1].cpu().numpy() == np.flatnonzero(d == d.min())[0]).all()
