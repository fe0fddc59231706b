"""The Newton-Euler recursion in link coordinates as a torch program on the
CPU, with its gradients by autograd, and the adjoint of forward kinematics link
by link: run in float32, yardsticks for what the recursions themselves lose to
rounding."""
import numpy as np
import torch


def rnea(rb, q, qd, qdd, dtype):
    """Torques [B, n] from q, qd, qdd [B, n] (tensors, differentiable)."""
    B = q.shape[0]
    t = lambda a: torch.as_tensor(np.asarray(a, dtype=np.float64)).to(dtype)
    ex = lambda a: t(a).expand(B, 3)
    mv = lambda M, x: (M * x[..., None, :]).sum(-1)
    cross = lambda a, b: torch.linalg.cross(a, b, dim=-1)
    zero = torch.zeros(B, 3, dtype=dtype)
    w, v, al, a = [zero], [zero], [zero], [-ex(rb.gravity)]
    R, m, f = [None], [zero], [zero]
    for k in range(1, rb.n_links):
        p, j, r, Rk = int(rb.parent[k]), int(rb.joint_index[k]), ex(rb.fixed_p[k]), t(rb.fixed_R[k]).expand(B, 3, 3)
        s = ex(rb.axis[k])
        if j >= 0:
            mult = float(rb.joint_mult[k])
            th = mult * q[:, j] + float(rb.joint_offset[k])
            x, y, z = t(rb.axis[k])
            K = torch.stack([torch.stack([0 * x, -z, y]), torch.stack([z, 0 * x, -x]), torch.stack([-y, x, 0 * x])])
            sn, cs = torch.sin(th)[:, None, None], torch.cos(th)[:, None, None]
            J = cs * torch.eye(3, dtype=dtype) + sn * K + (1 - cs) * torch.outer(t(rb.axis[k]), t(rb.axis[k]))
            Rk = (Rk[..., :, :, None] * J[..., None, :, :]).sum(-2)
        RT = Rk.transpose(1, 2)
        wk, vk = mv(RT, w[p]), mv(RT, v[p] + cross(w[p], r))
        alk, ak = mv(RT, al[p]), mv(RT, a[p] + cross(al[p], r))
        if j >= 0:
            sd = (mult * qd[:, j])[:, None] * s
            wk = wk + sd
            alk, ak = alk + (mult * qdd[:, j])[:, None] * s + cross(wk, sd), ak + cross(vk, sd)
        mass, c, In = float(rb.mass[k]), ex(rb.com[k]), t(rb.inertia[k])

        def inertia(x, y):
            h = mass * (y + cross(x, c))
            return mv(In, x) + cross(c, h), h
        n1, f1 = inertia(alk, ak)
        n2, f2 = inertia(wk, vk)
        w.append(wk), v.append(vk), al.append(alk), a.append(ak), R.append(Rk)
        m.append(n1 + cross(wk, n2) + cross(vk, f2)), f.append(f1 + cross(wk, f2))
    tau = [torch.zeros(B, dtype=dtype)] * rb.n_dof
    for k in range(rb.n_links - 1, 0, -1):
        p, j = int(rb.parent[k]), int(rb.joint_index[k])
        if j >= 0:
            tau[j] = tau[j] + float(rb.joint_mult[k]) * (m[k] * ex(rb.axis[k])).sum(-1)
        if p > 0:
            fp = mv(R[k], f[k])
            m[p], f[p] = m[p] + mv(R[k], m[k]) + cross(ex(rb.fixed_p[k]), fp), f[p] + fp
    return torch.stack(tau, 1)


def rnea_and_vjp(rb, st, w, dtype):
    """dict of tau, g_q, g_qd, g_qdd [B, n], the gradients of sum(w * tau)."""
    x = [torch.as_tensor(np.asarray(a, dtype=np.float64)).to(dtype).requires_grad_() for a in (st.q, st.qd, st.qdd)]
    tau = rnea(rb, *x, dtype)
    g = torch.autograd.grad((torch.as_tensor(np.asarray(w, dtype=np.float64)).to(dtype) * tau).sum(), x)
    return dict(zip(("tau", "g_q", "g_qd", "g_qdd"), [t.detach().double().numpy() for t in (tau, *g)]))


def related(rb, joint):
    """Joints that turn an ancestor or a descendant of a link that `joint` turns, itself included."""
    chain = []
    for k in range(rb.n_links):
        c, p = {k}, k
        while p > 0:
            p = int(rb.parent[p])
            c.add(p)
        chain.append(c)
    mine = [k for k in range(rb.n_links) if int(rb.joint_index[k]) == joint]
    near = {i for i in range(rb.n_links) for k in mine if i in chain[k] or k in chain[i]}
    return sorted({int(rb.joint_index[i]) for i in near if int(rb.joint_index[i]) >= 0})


def fk_adjoint(rb, q, g_sph, dtype):
    """Joint gradients [B, n] of sum(g_sph * centres): forces and moments about the
    links' own origins, children added from the tips on."""
    B, L = q.shape[0], rb.n_links
    t = lambda a: np.asarray(a, dtype=np.float64).astype(dtype)
    mv = lambda M, x: (M * x[..., None, :]).sum(-1, dtype=dtype)
    cross = lambda a, b: np.stack([a[:, 1] * b[:, 2] - a[:, 2] * b[:, 1], a[:, 2] * b[:, 0] - a[:, 0] * b[:, 2],
                                   a[:, 0] * b[:, 1] - a[:, 1] * b[:, 0]], 1)
    mm = lambda X, Y: (X[..., :, :, None] * Y[..., None, :, :]).sum(-2, dtype=dtype)
    q, g_sph = t(q), t(g_sph)
    R, p = [np.broadcast_to(np.eye(3, dtype=dtype), (B, 3, 3))], [np.zeros((B, 3), dtype)]
    for k in range(1, L):
        a, j, Rk = int(rb.parent[k]), int(rb.joint_index[k]), np.broadcast_to(t(rb.fixed_R[k]), (B, 3, 3))
        if j >= 0:
            th = t(rb.joint_mult[k]) * q[:, j] + t(rb.joint_offset[k])
            x, y, z = t(rb.axis[k])
            K = np.array([[0, -z, y], [z, 0, -x], [-y, x, 0]], dtype)
            sn, cs = np.sin(th)[:, None, None], np.cos(th)[:, None, None]
            Rk = mm(Rk, cs * np.eye(3, dtype=dtype) + sn * K + (1 - cs) * np.outer(t(rb.axis[k]), t(rb.axis[k])))
        p.append(mv(R[a], np.broadcast_to(t(rb.fixed_p[k]), (B, 3))) + p[a])
        R.append(mm(R[a], Rk))
    F, M = [np.zeros((B, 3), dtype) for _ in range(L)], [np.zeros((B, 3), dtype) for _ in range(L)]
    for s, l in enumerate(rb.sphere_link):
        g = g_sph[:, s]
        F[l] = F[l] + g
        M[l] = M[l] + cross(mv(R[l], np.broadcast_to(t(rb.sphere_pos[s]), (B, 3))), g)
    out = np.zeros((B, rb.n_dof), dtype)
    for k in range(L - 1, 0, -1):
        a, j = int(rb.parent[k]), int(rb.joint_index[k])
        if j >= 0:
            out[:, j] += t(rb.joint_mult[k]) * (mv(R[k], np.broadcast_to(t(rb.axis[k]), (B, 3))) * M[k]).sum(-1, dtype=dtype)
        F[a] = F[a] + F[k]
        M[a] = M[a] + M[k] + cross(p[k] - p[a], F[k])
    return out.astype(np.float64)
