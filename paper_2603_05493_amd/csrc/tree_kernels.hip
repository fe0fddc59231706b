// RNEA and its vector-Jacobian product without a cache (cuRoboV2 Alg. 4 and
// the role of Alg. 5, with transforms and every forward quantity recomputed
// in the backward), and the adjoint of forward kinematics (Alg. 1) from
// sphere and pose gradients, for robots of at most 64 links.  Two mappings:
//   * one state per group of G lanes, lane i holding link perm[i] in
//     depth-first post-order as in the fused iteration: RNEA (k_rnea_lanes)
//     and the adjoint of small batches (k_fk_backward_tile, whose group
//     stages its states' gradients through LDS);
//   * one thread per (state, link) of a tile of states, the links of a level
//     of the tree at a time: the adjoint of large batches
//     (k_fk_backward_levels), about the links' own origins.
//
// The first carries the recursions in world coordinates (Plucker vectors
// about the world origin), where they become tree sums:
//   v_k = sum over the root path of S qd,  a_k = -g + sum of (S qdd + v x S qd),
//   f_k = I_k a_k + v_k x* I_k v_k - X*_k f_ext_k,
//   F_k = sum over the subtree of f,  tau = S . F.
// Path sums use pointer jumping over the parent lanes, subtree sums the
// difference of two values of a group scan (the force part of F split so that
// its scan is exact); link poses, velocities,
// accelerations and forces never leave registers, so the forward needs no
// traversal storage and the backward needs no cache.  The VJP is the exact
// reverse mode of those sums (the transpose of a path sum is a subtree sum
// and vice versa):
//   fb = pathsum(taub S);  ab = I fb;  vb = -fb x* I v - I (v x fb)
//   A = subsum(ab);  vb += (S qd) x* A;  V = subsum(vb)
//   qdd-bar = S.A,  qd-bar = S.V + (v x S).A
//   q-bar = (fb x S).F + ((a - qd v x S) x S).A + (v x S).V,  f_ext-bar = -X*^T fb
// (derived at rnea_adjoint).  Mimic joints: link l turns by m_l q_j + o_l; lane j of the
// group gathers joint j's torque (and adjoints) from the links it drives,
// and returns m_l tau-bar_j to each of them.
#include "tree.h"

namespace wb {

// A world-frame (about the world origin) motion or force vector in the
// coordinates of the link with pose (R, p), and back for a force.
__device__ __forceinline__ SV motion_to_link(const M3 &R, V3 p, SV u) {
    return sv(mulT(R, u.w), mulT(R, u.l + cross(u.w, p)));
}
__device__ __forceinline__ SV force_to_world(const M3 &R, V3 p, SV f) {
    const V3 Rf = mul(R, f.l);
    return sv(mul(R, f.w) + cross(p, Rf), Rf);
}

// RNEA (or its VJP, BWD), one state per group of G lanes.
// nb: states; B: row length of every [k][B] array (the ABI's ld >= nb).
template <bool BWD, int G>
__global__ void __launch_bounds__(256)
    k_rnea_lanes(DevRobot rb, DevFused fz, int64_t nb, int64_t B, const float *__restrict__ q,
                 const float *__restrict__ qd, const float *__restrict__ qdd, const float *__restrict__ f_ext,
                 float *__restrict__ tau, const float *__restrict__ g_tau, float *__restrict__ g_q,
                 float *__restrict__ g_qd, float *__restrict__ g_qdd, float *__restrict__ g_fext) {
    const int gl = threadIdx.x & (G - 1);
    const int64_t s = ((int64_t)blockIdx.x * 256 + threadIdx.x) / G;
    const bool valid = s < nb;
    const int64_t b = valid ? s : nb - 1;   // groups past the end compute on a valid state, store nothing
    const int *li = fz.li;
    const float *lf = fz.lf;
    const bool act = gl < rb.L;
    const int parent_lane = li[1 * 64 + gl];
    const bool revolute = li[5 * 64 + gl] != 0;
    const int jidx = li[3 * 64 + gl];
    const int link = li[0 * 64 + gl];
    const Subtree sub = subtree_of(li[2 * 64 + gl], gl);
    auto subsum = [&](SV x) { return subtree_sum(x, sub, G); };
    const bool mim = fz.mimic != 0;
    float th = 0.f, thd = 0.f, thdd = 0.f, mult = 1.f;
    if (revolute) {
        const int64_t o = (int64_t)jidx * B + b;
        th = q[o];
        thd = qd[o];
        thdd = qdd[o];
        if (mim) {
            mult = lf[29 * 64 + gl];
            th = mult * th + lf[30 * 64 + gl];
            thd *= mult;
            thdd *= mult;
        }
    }
    M3 R;
    V3 p;
    lane_world_pose(fz, gl, revolute, th, parent_lane, G, R, p);
    SV S = zsv();
    if (revolute) {
        const V3 sw = mul(R, v3(lf[0 * 64 + gl], lf[1 * 64 + gl], lf[2 * 64 + gl]));
        S = sv(sw, cross(p, sw));
    }
    WInertia J;
    J.m = lf[15 * 64 + gl];
    J.cw = mul(R, v3(lf[16 * 64 + gl], lf[17 * 64 + gl], lf[18 * 64 + gl])) + p;
    {
        float Ic[6];
#pragma unroll
        for (int t = 0; t < 6; ++t) Ic[t] = lf[(19 + t) * 64 + gl];
        rotate_inertia(R, Ic, J.I);
    }
    // Lanes past the robot are massless links without a joint on the root:
    // every sum below is zero there without a guard.
    const SV v = path_sum(thd * S, parent_lane, fz.jsteps, G);
    const SV c = crm(v, S);
    SV a = path_sum(thdd * S + thd * c, parent_lane, fz.jsteps, G);
    if (act) a += sv(v3(0.f, 0.f, 0.f), v3(-rb.gx, -rb.gy, -rb.gz));
    const SV Iv = iw_apply(J, v);
    SV F = iw_apply(J, a) + crf(v, Iv);
    if (f_ext && act) {   // external force in world coordinates, X* f_ext
        const float *fx = f_ext + (int64_t)(link * 6) * B + b;
        F = F - force_to_world(R, p, sv(v3(fx[0], fx[B], fx[2 * B]), v3(fx[3 * B], fx[4 * B], fx[5 * B])));
    }
    F = subtree_sum_wrench(F, sub, fz.branched != 0, G);
    const bool jlane = mim ? gl < rb.n : revolute;
    const int64_t jrow = (int64_t)(mim ? gl : jidx) * B + b;
    if (!BWD) {
        float t = revolute ? dot(S, F) : 0.f;
        if (mim) t = gather_joint(mult * t, fz, gl, G);
        if (valid && jlane) tau[jrow] = t;
        return;
    }
    // tau-bar of the lane's link: m_l tau-bar_j with mimic joints
    float taub = jlane ? g_tau[jrow] : 0.f;
    if (mim) {
        const float tj = __shfl(taub, revolute ? jidx : gl, G);
        taub = revolute ? mult * tj : 0.f;
    }
    const SV fb = path_sum(taub * S, parent_lane, fz.jsteps, G);
    if (g_fext && act && valid) {
        // -X*^T fb: moment part -R^T fb_w, force part -R^T (fb_l + fb_w x p)
        const SV gf = motion_to_link(R, p, fb);
        float *gx = g_fext + (int64_t)(link * 6) * B + b;
        gx[0] = -gf.w.x; gx[B] = -gf.w.y; gx[2 * B] = -gf.w.z;
        gx[3 * B] = -gf.l.x; gx[4 * B] = -gf.l.y; gx[5 * B] = -gf.l.z;
    }
    float thd_b, thdd_b;
    float th_b = rnea_adjoint(S, c, v, a, F, J, Iv, fb, thd, subsum, thd_b, thdd_b);
    if (mim) {
        th_b = gather_joint(mult * th_b, fz, gl, G);
        thd_b = gather_joint(mult * thd_b, fz, gl, G);
        thdd_b = gather_joint(mult * thdd_b, fz, gl, G);
    }
    if (valid && jlane) {
        g_q[jrow] = th_b;
        g_qd[jrow] = thd_b;
        g_qdd[jrow] = thdd_b;
    }
}

// The world pose of lane gl's link for one state (th from q, with mimic
// joints' multiplier and offset).
template <int G>
__device__ __forceinline__ void state_pose(const DevFused &fz, int gl, const float *__restrict__ q, int64_t B,
                                           int64_t b, float &mult, M3 &R, V3 &p) {
    const bool revolute = fz.li[5 * 64 + gl] != 0;
    float th = 0.f;
    mult = 1.f;
    if (revolute) {
        th = q[(int64_t)fz.li[3 * 64 + gl] * B + b];
        if (fz.mimic) {
            mult = fz.lf[29 * 64 + gl];
            th = mult * th + fz.lf[30 * 64 + gl];
        }
    }
    lane_world_pose(fz, gl, revolute, th, fz.li[1 * 64 + gl], G, R, p);
}

// Row link * 12 + e of a pose tile of TS states: element e of the link's
// pose (rotation row-major, then translation); rows are padded by one float.
template <int TS>
__device__ __forceinline__ void pose_put(float *tile, int link, int s, const M3 &R, V3 p) {
    float *r = tile + link * 12 * (TS + 1) + s;
#pragma unroll
    for (int t = 0; t < 9; ++t) r[t * (TS + 1)] = R.m[t];
    r[9 * (TS + 1)] = p.x;
    r[10 * (TS + 1)] = p.y;
    r[11 * (TS + 1)] = p.z;
}
template <int TS>
__device__ __forceinline__ void pose_get(const float *tile, int link, int s, M3 &R, V3 &p) {
    const float *r = tile + link * 12 * (TS + 1) + s;
#pragma unroll
    for (int t = 0; t < 9; ++t) R.m[t] = r[t * (TS + 1)];
    p = v3(r[9 * (TS + 1)], r[10 * (TS + 1)], r[11 * (TS + 1)]);
}

// Writes a pose tile: thread (t, r) takes state t of the rows r, r + G, ...
// and of every G-th sphere's centre, formed from its link's pose.
template <int G, int TS>
__device__ __forceinline__ void fk_tile_out(const DevRobot &rb, const float *tile, int64_t s0, int64_t nb, int64_t B,
                                            float *__restrict__ pose, float *__restrict__ sph) {
    const int t = threadIdx.x % TS;
    const int64_t b = s0 + t;
    if (b >= nb) return;
    if (pose)
        for (int r = threadIdx.x / TS; r < 12 * rb.L; r += G) pose[(int64_t)r * B + b] = tile[r * (TS + 1) + t];
    if (sph)
        for (int i = threadIdx.x / TS; i < rb.S; i += G) {
            const float4 c4 = rb.sph[i];
            M3 R;
            V3 p;
            pose_get<TS>(tile, rb.sph_link[i], t, R, p);
            const V3 c = mul(R, v3(c4.x, c4.y, c4.z)) + p;
            float *o = sph + (int64_t)i * 3 * B + b;
            o[0] = c.x;
            o[B] = c.y;
            o[2 * B] = c.z;
        }
}

// Forward kinematics (Sec. 6.1) of TS consecutive states by a workgroup of
// TS * G lanes: each group of G lanes forms one state's link poses by
// pointer jumping and leaves them in an LDS tile, from which rows leave in
// pieces of TS floats.  A group writing its own state touches one float of
// every row: humanoid with poses, 2,048 states, 19.0 us so and 8.3 us here.
template <int G, int TS>
__global__ void __launch_bounds__(TS * G) k_fk_tile(DevRobot rb, DevFused fz, int64_t nb, int64_t B,
                                                    const float *__restrict__ q, float *__restrict__ pose,
                                                    float *__restrict__ sph) {
    extern __shared__ float tile[];
    const int64_t s0 = (int64_t)xcd_chunk() * TS;
    {
        const int gl = threadIdx.x & (G - 1), ts = threadIdx.x / G;
        const int64_t b = min(s0 + ts, nb - 1);   // states past the batch repeat its last
        M3 R;
        V3 p;
        float mult;
        state_pose<G>(fz, gl, q, B, b, mult, R, p);
        const int link = fz.li[0 * 64 + gl];
        if (link >= 0) pose_put<TS>(tile, link, ts, R, p);
    }
    __syncthreads();
    fk_tile_out<G, TS>(rb, tile, s0, nb, B, pose, sph);
}

// Link poses of TS consecutive states level by level: thread (t, l) forms
// link l's local rotation in state t, then the levels of the tree compose
// their parents' poses from the tile one after the other, with the arithmetic
// of the one-lane-per-state walk (so that a batch keeps its results to the
// bit).  Every link is composed once, a fraction of the pointer jumps' work.
// R and p: the thread's link's pose; op: its parent's origin.
template <int TS>
__device__ __forceinline__ void level_poses(const DevRobot &rb, float *tile, int t, int l, const LinkF &f,
                                            const LinkI &i, const float *__restrict__ q, int64_t B, int64_t b, M3 &R,
                                            V3 &p, V3 &op) {
    int depth = 0, parent = 0;
    M3 Rl;
    V3 fp = v3(0.f, 0.f, 0.f);
    if (l == 0) {
#pragma unroll
        for (int e = 0; e < 9; ++e) R.m[e] = e % 4 == 0 ? 1.0f : 0.0f;
        p = fp;
        pose_put<TS>(tile, 0, t, R, p);
    } else if (l < rb.L) {
        depth = i.depth;
        parent = i.parent;
        fp = v3(f.fp[0], f.fp[1], f.fp[2]);
        Rl = local_rotation(f, i, i.revolute ? f.mult * q[(int64_t)i.jidx * B + b] + f.offset : 0.0f);
    }
    for (int d = 1; d <= rb.max_depth; ++d) {
        __syncthreads();
        if (depth == d) {
            pose_get<TS>(tile, parent, t, R, op);
            auto row = [&](int e) {   // the walk's order of roundings, spelled out
                return __builtin_fmaf(fp.z, R.m[e + 2], __builtin_fmaf(fp.y, R.m[e + 1], fp.x * R.m[e]));
            };
            p = v3(row(0), row(3), row(6)) + op;
            R = matmul(R, Rl);
            pose_put<TS>(tile, l, t, R, p);
        }
    }
}

// Forward kinematics level by level, for large batches; the barriers between
// levels are hidden once the chip holds several workgroups a compute unit.
// Bound by the bytes written.
template <int G, int TS>
__global__ void __launch_bounds__(TS * G) k_fk_levels(DevRobot rb, int64_t nb, int64_t B,
                                                      const float *__restrict__ q, float *__restrict__ pose,
                                                      float *__restrict__ sph) {
    extern __shared__ float tile[];
    const int64_t s0 = (int64_t)xcd_chunk() * TS;
    const int t = threadIdx.x % TS, l = threadIdx.x / TS;
    const int64_t b = min(s0 + t, nb - 1);
    LinkF f{};
    LinkI i{};
    if (l > 0 && l < rb.L) {
        f = rb.lf[l];
        i = rb.li[l];
    }
    M3 R;
    V3 p, op;
    level_poses<TS>(rb, tile, t, l, f, i, q, B, b, R, p, op);
    __syncthreads();
    fk_tile_out<G, TS>(rb, tile, s0, nb, B, pose, sph);
}

// Adjoint of forward kinematics (Alg. 1) from gradients on sphere centres
// g_sph[S][3][B] and/or link poses g_pose[L][12][B], TS states per workgroup
// as k_fk_tile: the poses are recomputed into the LDS tile; thread (t, l)
// forms the wrench that the gradients of link l exert about the world origin
// in state t, W_l = sum over its spheres of [c x g; g] plus, for a pose
// gradient (G on R, g_p on p), [sum_c r_c x G_c + p x g_p; g_p], reading
// pieces of TS floats, and leaves it in the link's own pose rows; then the
// group's subtree sum of W, projected on the joint's world axis
// S = [s; p x s], is the joint's gradient (a rotation about s moves every
// point and frame of the subtree).  Mimic joints gather m_l times their
// links' values.  The sum is taken in split form: the wrenches of a
// collision cancel in every joint above both spheres.
template <int G, int TS>
__global__ void __launch_bounds__(TS * G) k_fk_backward_tile(DevRobot rb, DevFused fz, int64_t nb, int64_t B,
                                                             const float *__restrict__ q,
                                                             const float *__restrict__ g_pose,
                                                             const float *__restrict__ g_sph,
                                                             float *__restrict__ g_q) {
    extern __shared__ float tile[];
    const int64_t s0 = (int64_t)xcd_chunk() * TS;
    const int gl = threadIdx.x & (G - 1), ts = threadIdx.x / G;
    const int64_t bg = min(s0 + ts, nb - 1);
    const int link = fz.li[0 * 64 + gl], jidx = fz.li[3 * 64 + gl];
    const bool revolute = fz.li[5 * 64 + gl] != 0;
    M3 R;
    V3 p;
    float mult;
    state_pose<G>(fz, gl, q, B, bg, mult, R, p);
    if (link >= 0) pose_put<TS>(tile, link, ts, R, p);
    SV S = zsv();
    if (revolute) {
        const V3 sw = mul(R, v3(fz.lf[0 * 64 + gl], fz.lf[1 * 64 + gl], fz.lf[2 * 64 + gl]));
        S = sv(sw, cross(p, sw));
    }
    __syncthreads();
    {
        const int t = threadIdx.x % TS, l = threadIdx.x / TS;
        const int64_t b = min(s0 + t, nb - 1);
        if (l < rb.L) {
            SV W = zsv();
            pose_get<TS>(tile, l, t, R, p);
            if (g_sph) {
                const int first = rb.li[l].sph_first, cnt = rb.li[l].sph_count;
#pragma unroll 4
                for (int j = 0; j < cnt; ++j) {
                    const float4 c4 = rb.sph[first + j];
                    const V3 c = mul(R, v3(c4.x, c4.y, c4.z)) + p;
                    const float *gp = g_sph + (int64_t)(first + j) * 3 * B + b;
                    const V3 g = v3(gp[0], gp[B], gp[2 * B]);
                    W += sv(cross(c, g), g);
                }
            }
            if (g_pose) {
                const float *gp = g_pose + (int64_t)l * 12 * B + b;
                M3 Gm;
#pragma unroll
                for (int e = 0; e < 9; ++e) Gm.m[e] = gp[e * B];
                const V3 gt = v3(gp[9 * B], gp[10 * B], gp[11 * B]);
                V3 m = cross(p, gt);
#pragma unroll
                for (int c = 0; c < 3; ++c) m += cross(col(R, c), col(Gm, c));
                W += sv(m, gt);
            }
            float *r = tile + l * 12 * (TS + 1) + t;   // the link's own rows: no other thread reads them
            r[0] = W.w.x; r[TS + 1] = W.w.y; r[2 * (TS + 1)] = W.w.z;
            r[3 * (TS + 1)] = W.l.x; r[4 * (TS + 1)] = W.l.y; r[5 * (TS + 1)] = W.l.z;
        }
    }
    __syncthreads();
    SV W = zsv();
    if (link >= 0) {
        const float *r = tile + link * 12 * (TS + 1) + ts;
        W = sv(v3(r[0], r[TS + 1], r[2 * (TS + 1)]), v3(r[3 * (TS + 1)], r[4 * (TS + 1)], r[5 * (TS + 1)]));
    }
    const Subtree sub = subtree_of(fz.li[2 * 64 + gl], gl);
    float th_b = dot(S, subtree_sum_split(W, sub, fz.branched != 0, G));
    if (fz.mimic) th_b = gather_joint(mult * th_b, fz, gl, G);
    const bool jlane = fz.mimic ? gl < rb.n : revolute;
    if (s0 + ts < nb && jlane) g_q[(int64_t)(fz.mimic ? gl : jidx) * B + bg] = th_b;
}

// The adjoint level by level, for large batches: the poses are recomputed as
// above, thread (t, l) forms the force F and the moment M about the link's own origin that the
// gradients of link l exert in state t, reading pieces of TS floats; then the
// levels of the tree add up their children's, tips first, moved to the parent's
// origin, and the joint's gradient is s . M about its world axis.  Moments about
// the links' own origins, summed along the tree, keep their digits where those
// about the world's do not (hinge gradient of the humanoid, 16,384 states,
// relative RMS error of the worst joint: 1.2e-5 here, 3.1e-5 by the tile form
// above), and a value that is not finite reaches the link's ancestors alone.
// Bound by the chain of levels, as RNEA's (humanoid, 24,576 states: 57 us, the
// tile form 44, one state per lane 121).
template <int TS>
__global__ void __launch_bounds__(TS * 64) k_fk_backward_levels(DevRobot rb, DevFused fz, int64_t nb, int64_t B,
                                                                const float *__restrict__ q,
                                                                const float *__restrict__ g_pose,
                                                                const float *__restrict__ g_sph,
                                                                float *__restrict__ g_q) {
    extern __shared__ float tile[];
    const int64_t s0 = (int64_t)xcd_chunk() * TS;
    const int t = threadIdx.x % TS, l = threadIdx.x / TS;
    const int64_t b = min(s0 + t, nb - 1);
    const bool link = l > 0 && l < rb.L, valid = s0 + t < nb;
    LinkF f{};
    LinkI i{};
    if (link) {
        f = rb.lf[l];
        i = rb.li[l];
    }
    M3 R;
    V3 p, op;
    level_poses<TS>(rb, tile, t, l, f, i, q, B, b, R, p, op);
    SV W = zsv();
    if (link && g_sph) {
#pragma unroll 4
        for (int j = 0; j < i.sph_count; ++j) {
            const float4 c4 = rb.sph[i.sph_first + j];
            const float *gp = g_sph + (int64_t)(i.sph_first + j) * 3 * B + b;
            const V3 g = v3(gp[0], gp[B], gp[2 * B]);
            W += sv(cross(mul(R, v3(c4.x, c4.y, c4.z)), g), g);
        }
    }
    if (link && g_pose) {
        const float *gp = g_pose + (int64_t)l * 12 * B + b;
        M3 Gm;
#pragma unroll
        for (int e = 0; e < 9; ++e) Gm.m[e] = gp[e * B];
        V3 m = v3(0.f, 0.f, 0.f);
#pragma unroll
        for (int c = 0; c < 3; ++c) m += cross(col(R, c), col(Gm, c));
        W += sv(m, v3(gp[9 * B], gp[10 * B], gp[11 * B]));
    }
    const int child = link ? rb.kids[l] : -1;
    for (int d = rb.max_depth; d >= 1; --d) {
        __syncthreads();   // the poses are read; the children's rows are in
        if (link && i.depth == d) {
            for (int c = child; c >= 0; c = rb.kids[64 + c]) {
                const float *r = tile + c * 12 * (TS + 1) + t;
                W += sv(v3(r[0], r[TS + 1], r[2 * (TS + 1)]), v3(r[3 * (TS + 1)], r[4 * (TS + 1)], r[5 * (TS + 1)]));
            }
            if (d > 1) {
                const V3 M = W.w + cross(p - op, W.l);
                float *r = tile + l * 12 * (TS + 1) + t;
                r[0] = M.x; r[TS + 1] = M.y; r[2 * (TS + 1)] = M.z;
                r[3 * (TS + 1)] = W.l.x; r[4 * (TS + 1)] = W.l.y; r[5 * (TS + 1)] = W.l.z;
            }
        }
    }
    float th_b = link && i.revolute ? f.mult * dot(mul(R, v3(f.axis[0], f.axis[1], f.axis[2])), W.w) : 0.f;
    if (rb.simple_joints) {
        if (link && i.revolute && valid) g_q[(int64_t)i.jidx * B + b] = th_b;
        return;
    }
    __syncthreads();
    if (l < rb.L) tile[l * (TS + 1) + t] = th_b;
    __syncthreads();
    if (l < rb.n && valid) {
        float acc = 0.f;
        for (int k = 0; k < fz.mc; ++k) {
            const int lane = fz.conn[k * 64 + l];
            if (lane >= 0) acc += tile[fz.li[lane] * (TS + 1) + t];
        }
        g_q[(int64_t)l * B + b] = acc;
    }
}

static int lanes_for(int L) { return L <= 16 ? 16 : (L <= 32 ? 32 : 64); }

// The pointer-jumping form in tiles of 4 states, of 16 where the batch fills
// the chip with them (humanoid with poses, 4 against 16 states a tile: 4.9 /
// 7.0 us at 32 states, 8.3 / 8.7 at 2,048, 12.4 / 9.8 at 4,096; its
// 588-sphere form 6.2 / 8.4, 11.7 / 11.0, 18.9 / 13.3), the adjoint in tiles
// of 4 and 8.
template <int G, int TS>
static void launch_fk_t(const DevRobot &rb, const DevFused &fz, int64_t B, int64_t ld, const float *q, float *pose,
                        float *sph, hipStream_t s) {
    hipLaunchKernelGGL((k_fk_tile<G, TS>), dim3((unsigned)((B + TS - 1) / TS)), dim3(TS * G),
                       (size_t)rb.L * 12 * (TS + 1) * 4, s, rb, fz, B, ld, q, pose, sph);
}
template <int G>
static void launch_fk_l(const DevRobot &rb, int64_t B, int64_t ld, const float *q, float *pose, float *sph,
                        hipStream_t s) {
    constexpr int TS = 16;
    hipLaunchKernelGGL((k_fk_levels<G, TS>), dim3((unsigned)((B + TS - 1) / TS)), dim3(TS * G),
                       (size_t)rb.L * 12 * (TS + 1) * 4, s, rb, B, ld, q, pose, sph);
}
template <int G, int TS>
static void launch_fkb_t(const DevRobot &rb, const DevFused &fz, int64_t B, int64_t ld, const float *q,
                         const float *g_pose, const float *g_sph, float *g_q, hipStream_t s) {
    hipLaunchKernelGGL((k_fk_backward_tile<G, TS>), dim3((unsigned)((B + TS - 1) / TS)), dim3(TS * G),
                       (size_t)rb.L * 12 * (TS + 1) * 4, s, rb, fz, B, ld, q, g_pose, g_sph, g_q);
}

template <int TS>
static void launch_fkb_l(const DevRobot &rb, const DevFused &fz, int64_t B, int64_t ld, const float *q,
                         const float *g_pose, const float *g_sph, float *g_q, hipStream_t s) {
    hipLaunchKernelGGL((k_fk_backward_levels<TS>), dim3((unsigned)((B + TS - 1) / TS)),
                       dim3((unsigned)((rb.L * TS + 63) / 64 * 64)), (size_t)rb.L * 12 * (TS + 1) * 4, s, rb, fz, B, ld,
                       q, g_pose, g_sph, g_q);
}

hipError_t launch_fk_lanes(const DevRobot &rb, const DevFused &fz, int64_t B, int64_t ld, const float *q, float *pose,
                           float *spheres, bool wide, hipStream_t s) {
    if (B == 0) return hipSuccess;
    switch (lanes_for(rb.L)) {
        case 16: wide ? launch_fk_t<16, 16>(rb, fz, B, ld, q, pose, spheres, s) : launch_fk_t<16, 4>(rb, fz, B, ld, q, pose, spheres, s); break;
        case 32: wide ? launch_fk_t<32, 16>(rb, fz, B, ld, q, pose, spheres, s) : launch_fk_t<32, 4>(rb, fz, B, ld, q, pose, spheres, s); break;
        default: wide ? launch_fk_t<64, 16>(rb, fz, B, ld, q, pose, spheres, s) : launch_fk_t<64, 4>(rb, fz, B, ld, q, pose, spheres, s); break;
    }
    return hipGetLastError();
}

hipError_t launch_fk_levels(const DevRobot &rb, int64_t B, int64_t ld, const float *q, float *pose, float *spheres,
                            hipStream_t s) {
    return in_slices(B, [&](int64_t b0, int64_t n) {
        const auto launch = rb.L <= 16 ? launch_fk_l<16> : (rb.L <= 32 ? launch_fk_l<32> : launch_fk_l<64>);
        launch(rb, n, ld, from(q, b0), from(pose, b0), from(spheres, b0), s);
    });
}

hipError_t launch_fk_backward_lanes(const DevRobot &rb, const DevFused &fz, int64_t B, int64_t ld, const float *q,
                                    const float *g_pose, const float *g_sph, float *g_q, bool wide, hipStream_t s) {
    if (B == 0) return hipSuccess;
    switch (lanes_for(rb.L)) {
        case 16: wide ? launch_fkb_t<16, 8>(rb, fz, B, ld, q, g_pose, g_sph, g_q, s) : launch_fkb_t<16, 4>(rb, fz, B, ld, q, g_pose, g_sph, g_q, s); break;
        case 32: wide ? launch_fkb_t<32, 8>(rb, fz, B, ld, q, g_pose, g_sph, g_q, s) : launch_fkb_t<32, 4>(rb, fz, B, ld, q, g_pose, g_sph, g_q, s); break;
        default: wide ? launch_fkb_t<64, 8>(rb, fz, B, ld, q, g_pose, g_sph, g_q, s) : launch_fkb_t<64, 4>(rb, fz, B, ld, q, g_pose, g_sph, g_q, s); break;
    }
    return hipGetLastError();
}

hipError_t launch_fk_backward_levels(const DevRobot &rb, const DevFused &fz, int64_t B, int64_t ld, const float *q,
                                     const float *g_pose, const float *g_sph, float *g_q, hipStream_t s) {
    return in_slices(B, [&](int64_t b0, int64_t n) {
        launch_fkb_l<8>(rb, fz, n, ld, from(q, b0), from(g_pose, b0), from(g_sph, b0), from(g_q, b0), s);
    });
}

template <bool BWD, int G>
static hipError_t launch_rnea_g(const DevRobot &rb, const DevFused &fz, int64_t B, int64_t ld, const float *q,
                                const float *qd, const float *qdd, const float *f_ext, float *tau, const float *g_tau,
                                float *g_q, float *g_qd, float *g_qdd, float *g_fext, hipStream_t s) {
    hipLaunchKernelGGL((k_rnea_lanes<BWD, G>), dim3((unsigned)((B * G + 255) / 256)), dim3(256), 0, s, rb, fz, B, ld, q,
                       qd, qdd, f_ext, tau, g_tau, g_q, g_qd, g_qdd, g_fext);
    return hipGetLastError();
}

template <bool BWD>
static hipError_t launch_rnea_any(const DevRobot &rb, const DevFused &fz, int64_t B, int64_t ld, const float *q,
                                  const float *qd, const float *qdd, const float *f_ext, float *tau,
                                  const float *g_tau, float *g_q, float *g_qd, float *g_qdd, float *g_fext,
                                  hipStream_t s) {
    if (B == 0) return hipSuccess;
    switch (lanes_for(rb.L)) {
        case 16: return launch_rnea_g<BWD, 16>(rb, fz, B, ld, q, qd, qdd, f_ext, tau, g_tau, g_q, g_qd, g_qdd, g_fext, s);
        case 32: return launch_rnea_g<BWD, 32>(rb, fz, B, ld, q, qd, qdd, f_ext, tau, g_tau, g_q, g_qd, g_qdd, g_fext, s);
        default: return launch_rnea_g<BWD, 64>(rb, fz, B, ld, q, qd, qdd, f_ext, tau, g_tau, g_q, g_qd, g_qdd, g_fext, s);
    }
}

hipError_t launch_rnea_lanes(const DevRobot &rb, const DevFused &fz, int64_t B, int64_t ld, const float *q,
                             const float *qd, const float *qdd, const float *f_ext, float *tau, hipStream_t s) {
    return launch_rnea_any<false>(rb, fz, B, ld, q, qd, qdd, f_ext, tau, nullptr, nullptr, nullptr, nullptr, nullptr, s);
}

hipError_t launch_rnea_backward_lanes(const DevRobot &rb, const DevFused &fz, int64_t B, int64_t ld,
                                      const float *q, const float *qd, const float *qdd, const float *f_ext,
                                      const float *g_tau, float *g_q, float *g_qd, float *g_qdd, float *g_fext,
                                      hipStream_t s) {
    return launch_rnea_any<true>(rb, fz, B, ld, q, qd, qdd, f_ext, nullptr, g_tau, g_q, g_qd, g_qdd, g_fext, s);
}

}  // namespace wb
