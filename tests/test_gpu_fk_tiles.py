"""GPU: the tiled forms of forward kinematics (groups of lanes in tiles of 4
and 16 states, level by level) and its adjoint (groups of lanes in tiles of 4
and 8, level by level in tiles of 8), the hinge
adjoint's runs of spheres and the cost head's quarters, against the FP64
oracle at their edges: lane counts (2, 16, 17, 33 and 64 links), batches that
end inside a tile on both sides of the wide tiles' threshold, rows padded
with NaN."""
import numpy as np
import pytest
import torch

from paper_2603_05493_amd import synth
from tests import parity as P

pytestmark = pytest.mark.gpu

ROBOTS = [("chain1", lambda: synth.serial_chain(1, 3, seed=2)), ("tree16", lambda: synth.random_tree(15, 2, seed=4)),
          ("tree17", lambda: synth.random_tree(16, 3, seed=5, random_fixed_rotation=True, dfs_order=False)),
          ("tree33", lambda: synth.random_tree(32, 1, seed=7)), ("tree64", lambda: synth.random_tree(63, 1, seed=8))]


@pytest.mark.parametrize("label,factory", ROBOTS)
@pytest.mark.parametrize("size", ["one", "small", "wide"])
@pytest.mark.parametrize("form", ["group", "levels"])
def test_tiled_fk_and_adjoint(oracle, label, factory, size, form):
    from paper_2603_05493_amd import wb
    rb = factory()
    r = wb.Robot(rb).to_device("cuda:0")
    below = (1 << 40) if form == "group" else 0
    r.set_dispatch(-1, below, below)
    full = 16 * torch.cuda.get_device_properties(0).multi_processor_count
    B = {"one": 1, "small": 101, "wide": full + 11}[size]
    ld = B + 2
    st = synth.states(rb, B, seed=3, q_range=1.5)
    pad = lambda a: torch.nn.functional.pad(P.dev(a), (0, ld - B), value=float("nan")).contiguous()
    nan = lambda *s: torch.full((*s, ld), float("nan"), device="cuda")
    q = pad(st.q)
    n, L, S = rb.n_dof, rb.n_links, rb.n_spheres
    pose, sph = wb.wb_fk(r, q, nan(L, 12), nan(S, 3), nb=B)
    _, sph2 = wb.wb_fk(r, q, None, nan(S, 3), want_pose=False, nb=B)
    rng = np.random.default_rng(4)
    gc, gR, gp = rng.normal(size=(B, S, 3)), rng.normal(size=(B, L, 3, 3)), rng.normal(size=(B, L, 3))
    g_s = wb.wb_fk_backward(r, q, g_spheres=pad(gc), link_pose=pose, g_q=nan(n), nb=B)
    g_b = wb.wb_fk_backward(r, q, g_spheres=pad(gc), g_link_pose=pad(np.concatenate([gR.reshape(B, -1, 9), gp], 2)),
                            g_q=nan(n), nb=B)
    torch.cuda.synchronize()
    for t in (pose, sph, sph2, g_s, g_b):
        assert torch.isnan(t[..., B:]).all(), f"{label}: padding written"
        assert torch.isfinite(t[..., :B]).all(), f"{label}: not written"
    pick = np.unique(np.concatenate([np.arange(min(B, 20)), np.arange(max(0, B - 20), B)]))
    sub = lambda t: P.host(t[..., :B])[pick]
    R, p, c = oracle.fk(rb, st.q[pick])
    ext = P.extent(c)
    ps = sub(pose)
    assert P.normwise(ps[:, :, :9], R.reshape(len(pick), -1, 9), floor=1.0).max() < P.TOL
    assert P.scaled(ps[:, :, 9:], p, ext).max() < P.TOL
    assert max(P.scaled(sub(sph), c, ext).max(), P.scaled(sub(sph2), c, ext).max()) < P.TOL
    ref = oracle.fk_backward(rb, st.q[pick], g_spheres=gc[pick])
    both = oracle.fk_backward(rb, st.q[pick], g_spheres=gc[pick], g_R=gR[pick], g_p=gp[pick])
    assert P.normwise(sub(g_s), ref, floor=1e-6).max() < P.TOL
    assert P.normwise(sub(g_b), both, floor=1e-6).max() < P.TOL


@pytest.mark.parametrize("B", [1, 65, 9000])
@pytest.mark.parametrize("spheres", [1, 7])
def test_hinge_adjoint_runs(oracle, B, spheres):
    from paper_2603_05493_amd import wb
    rb = synth.random_tree(6, spheres, seed=11)
    r = wb.Robot(rb).to_device("cuda:0")
    st = synth.states(rb, B, seed=5, q_range=1.5)
    _, sph = wb.wb_fk(r, P.dev(st.q))
    mp, am, _ = wb.wb_self_collision(r, sph)
    margin = 0.3   # most states within it
    gc = torch.rand(B, device="cuda") + 0.5
    g = wb.wb_self_collision_backward(r, sph, am, mp, margin, gc)
    torch.cuda.synchronize()
    ref = oracle.self_collision_backward(rb, P.host(sph), am.cpu().numpy(), mp.cpu().numpy().astype(np.float64), margin,
                                         gc.cpu().numpy().astype(np.float64))
    assert P.normwise(P.host(g), ref, floor=1e-6).max() < P.TOL


@pytest.mark.parametrize("n", [1, 3, 4, 5, 48])
@pytest.mark.parametrize("B", [1, 63, 129])
@pytest.mark.parametrize("weighted", [False, True])
def test_cost_head_quarters(n, B, weighted):
    from paper_2603_05493_amd import wb
    g = torch.Generator(device="cuda").manual_seed(n * 100 + B)
    tau = torch.randn(n, B, generator=g, device="cuda")
    w = torch.randn(n, B, generator=g, device="cuda") if weighted else None
    mp = torch.randn(B, generator=g, device="cuda") * 0.02
    cost, gt, gm = torch.empty(B, device="cuda"), torch.empty(n, B, device="cuda"), torch.empty(B, device="cuda")
    wb.wb_cost_head(tau, w, 1e-3, mp, 0.01, 2.0, cost, gt, gm)
    torch.cuda.synchronize()
    t, m = tau.double(), mp.double() + float(np.float32(0.01))
    terms = w.double() * t if weighted else float(np.float32(1e-3)) * t * t
    ref = terms.sum(0) + 2.0 * torch.relu(m)
    scale = terms.abs().sum(0) + 2.0 * torch.relu(m)
    assert ((cost.double() - ref).abs() <= (n + 3) * 2.0 ** -24 * scale).all()   # a rounding per term, three to join
    assert torch.equal(gt, w if weighted else 2.0 * np.float32(1e-3) * tau)
    assert torch.equal(gm, torch.where(mp + np.float32(0.01) > 0, 2.0, 0.0))
