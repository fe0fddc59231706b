"""GPU: batches past the ends of the slices that kernels with several threads a
state are launched on (2^24 states), and past the batch at which one grid
would need 2^32 threads: states on both sides of each edge and the last ones
agree with a small batch of the same states."""
import numpy as np
import pytest
import torch

from paper_2603_05493_amd import synth

pytestmark = pytest.mark.gpu

SLICE = 1 << 24


def _sparse_robot():
    """41 links, of which three turn and two hold a sphere."""
    rb = synth.random_tree(40, 1, seed=6)
    turn = (5, 17, 40)
    rb.joint_index = np.array([turn.index(k) if k in turn else -1 for k in range(rb.n_links)], dtype=np.int32)
    rb.joint_type = np.array([rb.joint_type[k] if k in turn else 0 for k in range(rb.n_links)], dtype=rb.joint_type.dtype)
    keep = [3, 38]
    rb.sphere_link, rb.sphere_pos, rb.sphere_r = rb.sphere_link[keep], rb.sphere_pos[keep], rb.sphere_r[keep]
    return rb


def _picks(B):
    edges = [0] + [e for e in (SLICE, 2 * SLICE, 1 << 26, 1 << 30) if e < B]
    at = [i for e in edges for i in range(e - 6, e + 6)] + list(range(B - 6, B))
    return torch.tensor(sorted({i for i in at if 0 <= i < B}), device="cuda")


def _rows(n, B, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.rand((n, B), generator=g, device="cuda") * 3 - 1.5


def _close(big, small, at):
    assert torch.allclose(big[..., at], small, rtol=1e-5, atol=1e-6)


@pytest.mark.parametrize("B", [SLICE + 5, (1 << 26) + 9])
def test_fk(B):
    from paper_2603_05493_amd import wb
    r = wb.Robot(_sparse_robot()).to_device("cuda:0")
    r.set_dispatch(-1, 0, 0)
    q, at = _rows(3, B, 1), _picks(B)
    _, sph = wb.wb_fk(r, q, want_pose=False)
    torch.cuda.synchronize()
    _close(sph, wb.wb_fk(r, q[:, at].contiguous(), want_pose=False)[1], at)


def test_fk_adjoint():
    from paper_2603_05493_amd import wb
    r = wb.Robot(synth.serial_chain(2, 1, seed=3)).to_device("cuda:0")
    r.set_dispatch(-1, 0, 0)
    B, S = SLICE + 5, r.n_spheres
    q, gs, at = _rows(2, B, 1), _rows(3 * S, B, 2).view(S, 3, B), _picks(B)
    g_q = wb.wb_fk_backward(r, q, g_spheres=gs)
    torch.cuda.synchronize()
    _close(g_q, wb.wb_fk_backward(r, q[:, at].contiguous(), g_spheres=gs[..., at].contiguous()), at)


def test_cached_rnea():
    from paper_2603_05493_amd import wb
    r = wb.Robot(synth.serial_chain(2, 1, seed=3)).to_device("cuda:0")
    B = SLICE + 5
    q, qd, qdd, w, at = _rows(2, B, 1), _rows(2, B, 2), _rows(2, B, 3), _rows(2, B, 4), _picks(B)
    tau, cache = wb.wb_rnea(r, q, qd, qdd)
    g = wb.wb_rnea_backward(r, q, qd, qdd, cache, w)
    torch.cuda.synchronize()
    p = [t[..., at].contiguous() for t in (q, qd, qdd, w)]
    tau_s, cache_s = wb.wb_rnea(r, *p[:3])
    _close(tau, tau_s, at)
    for x, y in zip(g, wb.wb_rnea_backward(r, *p[:3], cache_s, p[3])):
        _close(x, y, at)


@pytest.mark.parametrize("B", [SLICE + 5, (1 << 30) + 9])
def test_cost_head(B):
    from paper_2603_05493_amd import wb
    tau, at = _rows(1, B, 1), _picks(B)
    cost = torch.empty(B, device="cuda")
    wb.wb_cost_head(tau, None, 0.5, None, 0.0, 0.0, cost, None, None)
    torch.cuda.synchronize()
    _close(cost, 0.5 * tau[0, at] ** 2, at)
