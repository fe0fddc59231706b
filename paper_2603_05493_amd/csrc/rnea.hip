// Recursive Newton-Euler inverse dynamics and its vector-Jacobian product
// through the forward cache (cuRoboV2 Sec. 6.3, Alg. 4 and the role of
// Alg. 5).
//
// The per-link sweeps follow Alg. 4 in link coordinates with the compact
// transform (R, p) and compact inertia (m, c, Ic), in two forms:
//   * robots of at most 64 links: one thread per (state, link), the links of
//     a level of the tree at a time (k_rnea_levels, k_rnea_backward_levels);
//   * larger ones: one state per lane, links in index order (parents first),
//     which keeps the parent's values in registers whenever the parent is
//     the previous link (a "carry"), touching the cache only at branches.
// Both sum in link coordinates, so the torque of a light link far from the
// base keeps its digits, and a value that is not finite stays with the
// link's ancestors and descendants.  Sums over subtrees taken as differences
// of a scan in world coordinates (tree_kernels.hip, the form without a
// cache) lose a factor of ten at a humanoid's fingers (relative RMS error of
// their torques 1.3e-5 against 1.2e-6) and carry a NaN into every lane
// behind it.
//
// Cache layout [L][18][B]: v (6), a (6), accumulated force F (6) per link;
// link 0 (the fixed base, v = 0, a = -g) is not stored.  External link
// forces f_ext [L][6][B] (link coordinates, moment then force about the link
// origin) enter Alg. 4 as f_k = I a + v x* I v - f_ext_k, so the cached F
// includes them and the backward needs only their adjoint, -F-bar_k.
//
// The backward is the exact reverse mode of the forward sweep (with
// dX/dtheta = -crm(S) X):
//   sweep A, base -> tips:  Fb_k = S m taub + X Fb_p,  thb += (X Fb_p).crf(S) F_k
//   sweep B, tips -> base:  ab_k = I Fb_k + sum_children X_c^T ab_c,
//                           vb_k = -crf(Fb) I v - I crm(v) Fb + crf(S thd) ab_k
//                                  + sum_children X_c^T vb_c,
//                           qdd-bar = S.ab, qd-bar = S.vb - S.(crf(v) ab),
//                           thb -= ab.crm(S) X a_p + vb.crm(S) X v_p.
// The crf(S thd) ab term is the velocity dependence of the Coriolis term of
// the acceleration recursion; it belongs to the exact VJP.
#include "lanes.h"
#include "spatial.h"

namespace wb {

__device__ __forceinline__ SV ld_sv(const float *__restrict__ base, int64_t B) {
    return sv(v3(base[0], base[B], base[2 * B]), v3(base[3 * B], base[4 * B], base[5 * B]));
}
__device__ __forceinline__ void st_sv(float *__restrict__ base, int64_t B, SV x) {
    base[0] = x.w.x; base[B] = x.w.y; base[2 * B] = x.w.z;
    base[3 * B] = x.l.x; base[4 * B] = x.l.y; base[5 * B] = x.l.z;
}
__device__ __forceinline__ void add_sv(float *__restrict__ base, int64_t B, SV x) {
    base[0] += x.w.x; base[B] += x.w.y; base[2 * B] += x.w.z;
    base[3 * B] += x.l.x; base[4 * B] += x.l.y; base[5 * B] += x.l.z;
}

struct JointIn {
    float th, thd, thdd;
};

__device__ __forceinline__ JointIn joint_in(const LinkF &f, const LinkI &i, const float *__restrict__ q,
                                            const float *__restrict__ qd, const float *__restrict__ qdd,
                                            int64_t B, int64_t b) {
    JointIn r{0.f, 0.f, 0.f};
    if (i.revolute) {
        const int64_t o = (int64_t)i.jidx * B + b;
        r.th = f.mult * q[o] + f.offset;
        r.thd = f.mult * qd[o];
        r.thdd = f.mult * qdd[o];
    }
    return r;
}

// nb: states; B: row length of every [k][B] array (the ABI's ld >= nb).
__global__ void __launch_bounds__(256) k_rnea(DevRobot rb, int64_t nb, int64_t B, const float *__restrict__ q,
                                              const float *__restrict__ qd, const float *__restrict__ qdd,
                                              const float *__restrict__ f_ext, float *__restrict__ tau,
                                              float *__restrict__ cache) {
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= nb) return;
    const int L = rb.L;
    const SV a0 = sv(v3(0.f, 0.f, 0.f), v3(-rb.gx, -rb.gy, -rb.gz));
    const SV zero = sv(v3(0.f, 0.f, 0.f), v3(0.f, 0.f, 0.f));
    float *cb = cache + b;
    if (!rb.simple_joints)
        for (int j = 0; j < rb.n; ++j) tau[(int64_t)j * B + b] = 0.0f;
    // Pass 1 (base -> tips): velocities, accelerations, link forces.
    SV v = zero, a = a0;
    for (int k = 1; k < L; ++k) {
        const LinkI li = ldu(rb.li + k);
        const LinkF lf = ldu(rb.lf + k);
        const int p = li.parent;
        SV vp = v, ap = a;
        if (p == 0) {
            vp = zero;
            ap = a0;
        } else if (p != k - 1) {
            vp = ld_sv(cb + (int64_t)(p * 18) * B, B);
            ap = ld_sv(cb + (int64_t)(p * 18 + 6) * B, B);
        }
        const JointIn J = joint_in(lf, li, q, qd, qdd, B, b);
        const M3 R = local_rotation(lf, li, J.th);
        const V3 r = v3(lf.fp[0], lf.fp[1], lf.fp[2]);
        const V3 s = v3(lf.axis[0], lf.axis[1], lf.axis[2]);
        const SV Sqd = sv(J.thd * s, v3(0.f, 0.f, 0.f));
        v = X_apply(R, r, vp) + Sqd;
        a = X_apply(R, r, ap) + sv(J.thdd * s, v3(0.f, 0.f, 0.f)) + crm(v, Sqd);
        SV f = I_apply(lf, a) + crf(v, I_apply(lf, v));
        if (f_ext) f = f - ld_sv(f_ext + (int64_t)(k * 6) * B + b, B);
        float *ck = cb + (int64_t)(k * 18) * B;
        st_sv(ck, B, v);
        st_sv(ck + 6 * B, B, a);
        st_sv(ck + 12 * B, B, f);
    }
    // Pass 3 (tips -> base): accumulate forces into parents, project on joints.
    SV carry = zero;
    bool have_carry = false;
    for (int k = L - 1; k >= 1; --k) {
        const LinkI li = ldu(rb.li + k);
        const LinkF lf = ldu(rb.lf + k);
        float *cF = cb + (int64_t)(k * 18 + 12) * B;
        SV F = ld_sv(cF, B);
        if (have_carry) {
            F += carry;
            st_sv(cF, B, F);
        }
        const JointIn J = joint_in(lf, li, q, qd, qdd, B, b);
        if (li.revolute) {
            const float t = lf.mult * (lf.axis[0] * F.w.x + lf.axis[1] * F.w.y + lf.axis[2] * F.w.z);
            float *tj = tau + (int64_t)li.jidx * B + b;
            if (rb.simple_joints) *tj = t;
            else *tj += t;
        }
        const int p = li.parent;
        have_carry = false;
        if (p >= 1) {
            const M3 R = local_rotation(lf, li, J.th);
            const SV fp = XT_apply(R, v3(lf.fp[0], lf.fp[1], lf.fp[2]), F);
            if (p == k - 1) {
                carry = fp;
                have_carry = true;
            } else {
                add_sv(cb + (int64_t)(p * 18 + 12) * B, B, fp);
            }
        }
    }
}

// ws layout per state: [L][18]: Fb (6), ab (6), vb (6).
__global__ void __launch_bounds__(256) k_rnea_backward(DevRobot rb, int64_t nb, int64_t B, const float *__restrict__ q,
                                                       const float *__restrict__ qd,
                                                       const float *__restrict__ qdd,
                                                       const float *__restrict__ cache,
                                                       const float *__restrict__ g_tau,
                                                       float *__restrict__ g_q, float *__restrict__ g_qd,
                                                       float *__restrict__ g_qdd, float *__restrict__ g_fext,
                                                       float *__restrict__ ws) {
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= nb) return;
    const int L = rb.L;
    const SV a0 = sv(v3(0.f, 0.f, 0.f), v3(-rb.gx, -rb.gy, -rb.gz));
    const SV zero = sv(v3(0.f, 0.f, 0.f), v3(0.f, 0.f, 0.f));
    const float *cb = cache + b;
    float *wb_ = ws + b;
    if (!rb.simple_joints)
        for (int j = 0; j < rb.n; ++j) {
            g_q[(int64_t)j * B + b] = 0.0f;
            g_qd[(int64_t)j * B + b] = 0.0f;
            g_qdd[(int64_t)j * B + b] = 0.0f;
        }
    // Sweep A (base -> tips): adjoint of the force accumulation.
    SV Fb = zero;
    if (g_fext) st_sv(g_fext + b, B, zero);   // the base's force reaches no joint
    for (int k = 1; k < L; ++k) {
        const LinkI li = ldu(rb.li + k);
        const LinkF lf = ldu(rb.lf + k);
        const int p = li.parent;
        SV Fbp = Fb;
        if (p == 0) Fbp = zero;
        else if (p != k - 1) Fbp = ld_sv(wb_ + (int64_t)(p * 18) * B, B);
        const JointIn J = joint_in(lf, li, q, qd, qdd, B, b);
        const M3 R = local_rotation(lf, li, J.th);
        const V3 s = v3(lf.axis[0], lf.axis[1], lf.axis[2]);
        const SV XFp = X_apply(R, v3(lf.fp[0], lf.fp[1], lf.fp[2]), Fbp);
        const float tb = li.revolute ? lf.mult * g_tau[(int64_t)li.jidx * B + b] : 0.0f;
        Fb = sv(tb * s, v3(0.f, 0.f, 0.f)) + XFp;
        float *wk = wb_ + (int64_t)(k * 18) * B;
        st_sv(wk, B, Fb);
        if (g_fext) st_sv(g_fext + (int64_t)(k * 6) * B + b, B, zero - Fb);
        if (li.far_child) {
            st_sv(wk + 6 * B, B, zero);
            st_sv(wk + 12 * B, B, zero);
        }
        if (li.revolute) {
            const SV F = ld_sv(cb + (int64_t)(k * 18 + 12) * B, B);
            const float thb = lf.mult * (dot(XFp.w, cross(s, F.w)) + dot(XFp.l, cross(s, F.l)));
            float *gq = g_q + (int64_t)li.jidx * B + b;
            if (rb.simple_joints) *gq = thb;
            else *gq += thb;
        }
    }
    // Sweep B (tips -> base): adjoint of the velocity/acceleration recursion.
    SV ca = zero, cv = zero;
    bool have_carry = false;
    for (int k = L - 1; k >= 1; --k) {
        const LinkI li = ldu(rb.li + k);
        const LinkF lf = ldu(rb.lf + k);
        const int p = li.parent;
        const float *wk = wb_ + (int64_t)(k * 18) * B;
        const float *ck = cb + (int64_t)(k * 18) * B;
        const SV Fbk = ld_sv(wk, B);
        const SV vk = ld_sv(ck, B);
        SV ab = I_apply(lf, Fbk);
        SV vb = zero - (crf(Fbk, I_apply(lf, vk)) + I_apply(lf, crm(vk, Fbk)));
        if (have_carry) {
            ab += ca;
            vb += cv;
        }
        if (li.far_child) {
            ab += ld_sv(wk + 6 * B, B);
            vb += ld_sv(wk + 12 * B, B);
        }
        const JointIn J = joint_in(lf, li, q, qd, qdd, B, b);
        const V3 s = v3(lf.axis[0], lf.axis[1], lf.axis[2]);
        const SV Sqd = sv(J.thd * s, v3(0.f, 0.f, 0.f));
        vb += crf(Sqd, ab);
        const M3 R = local_rotation(lf, li, J.th);
        const V3 r = v3(lf.fp[0], lf.fp[1], lf.fp[2]);
        if (li.revolute) {
            SV vp = zero, ap = a0;
            if (p != 0) {
                vp = ld_sv(cb + (int64_t)(p * 18) * B, B);
                ap = ld_sv(cb + (int64_t)(p * 18 + 6) * B, B);
            }
            const SV Xa = X_apply(R, r, ap), Xv = X_apply(R, r, vp);
            const float thdd_b = dot(s, ab.w);
            const float thd_b = dot(s, vb.w) - dot(s, crf(vk, ab).w);
            const float th_b = -(dot(ab.w, cross(s, Xa.w)) + dot(ab.l, cross(s, Xa.l)) +
                                 dot(vb.w, cross(s, Xv.w)) + dot(vb.l, cross(s, Xv.l)));
            const int64_t o = (int64_t)li.jidx * B + b;
            if (rb.simple_joints) {
                g_qdd[o] = thdd_b;
                g_qd[o] = thd_b;
            } else {
                g_qdd[o] += lf.mult * thdd_b;
                g_qd[o] += lf.mult * thd_b;
            }
            g_q[o] += lf.mult * th_b;
        }
        have_carry = false;
        if (p >= 1) {
            const SV pa = XT_apply(R, r, ab), pv = XT_apply(R, r, vb);
            if (p == k - 1) {
                ca = pa;
                cv = pv;
                have_carry = true;
            } else {
                float *wp = wb_ + (int64_t)(p * 18) * B;
                add_sv(wp + 6 * B, B, pa);
                add_sv(wp + 12 * B, B, pv);
            }
        }
    }
}

// ---- one thread per (state, link), level by level.  A workgroup takes TS
// consecutive states: thread (t, l) owns link l in state t, so that a wavefront
// touches pieces of TS floats of 64 / TS links' rows.  What passes between
// links goes through an LDS tile, row link * 12 + c holding component c,
// padded by one float.
template <int TS>
__device__ __forceinline__ void row_put(float *tile, int link, int c, int t, SV x) {
    float *r = tile + (link * 12 + c) * (TS + 1) + t;
    r[0] = x.w.x; r[TS + 1] = x.w.y; r[2 * (TS + 1)] = x.w.z;
    r[3 * (TS + 1)] = x.l.x; r[4 * (TS + 1)] = x.l.y; r[5 * (TS + 1)] = x.l.z;
}
template <int TS>
__device__ __forceinline__ SV row_get(const float *tile, int link, int c, int t) {
    const float *r = tile + (link * 12 + c) * (TS + 1) + t;
    return sv(v3(r[0], r[TS + 1], r[2 * (TS + 1)]), v3(r[3 * (TS + 1)], r[4 * (TS + 1)], r[5 * (TS + 1)]));
}

// Joint rows of robots where a joint drives several links: every thread
// leaves its link's (already scaled) value x in the tile, then thread (t, j)
// adds up those of joint j's links.  Every thread of the workgroup calls this.
template <int TS>
__device__ __forceinline__ float joint_sum(float *tile, const DevRobot &rb, const DevFused &fz, int l, int t, float x) {
    __syncthreads();
    if (l < rb.L) tile[l * (TS + 1) + t] = x;
    __syncthreads();
    float acc = 0.f;
    if (l < rb.n)
        for (int k = 0; k < fz.mc; ++k) {
            const int lane = fz.conn[k * 64 + l];
            if (lane >= 0) acc += tile[fz.li[lane] * (TS + 1) + t];
        }
    return acc;
}

// What bounds it is the chain of levels, a barrier, an LDS read and a
// transform each, down the tree and up again: a batch has to fill the chip
// with workgroups to hide it (humanoid, 12 levels: 11 us at 32 to 1,024
// states, 54 us at 24,576, where the bytes take 22; one state per lane 82 and
// 119 us; a 12-joint tree at 256 states 4.5 against 21.5).
// nb: states; B: row length of every [k][B] array (the ABI's ld >= nb).
template <int TS>
__global__ void __launch_bounds__(64 * TS) k_rnea_levels(DevRobot rb, DevFused fz, int64_t nb, int64_t B,
                                                         const float *__restrict__ q, const float *__restrict__ qd,
                                                         const float *__restrict__ qdd,
                                                         const float *__restrict__ f_ext, float *__restrict__ tau,
                                                         float *__restrict__ cache) {
    extern __shared__ float tile[];
    const int t = threadIdx.x % TS, l = threadIdx.x / TS;
    const int64_t s0 = (int64_t)xcd_chunk() * TS, b = min(s0 + t, nb - 1);   // states past the batch repeat its last
    const bool link = l > 0 && l < rb.L, valid = s0 + t < nb;
    const SV zero = sv(v3(0.f, 0.f, 0.f), v3(0.f, 0.f, 0.f));
    LinkI li{};
    LinkF lf{};
    JointIn J{0.f, 0.f, 0.f};
    M3 R;
    if (link) {
        li = rb.li[l];
        lf = rb.lf[l];
        J = joint_in(lf, li, q, qd, qdd, B, b);
        R = local_rotation(lf, li, J.th);
    } else if (l == 0) {
        row_put<TS>(tile, 0, 0, t, zero);
        row_put<TS>(tile, 0, 6, t, sv(v3(0.f, 0.f, 0.f), v3(-rb.gx, -rb.gy, -rb.gz)));
    }
    const V3 r = v3(lf.fp[0], lf.fp[1], lf.fp[2]), s = v3(lf.axis[0], lf.axis[1], lf.axis[2]);
    // base -> tips: velocities and accelerations
    SV v = zero, a = zero;
    for (int d = 1; d <= rb.max_depth; ++d) {
        __syncthreads();
        if (link && li.depth == d) {
            const SV Sqd = sv(J.thd * s, v3(0.f, 0.f, 0.f));
            v = X_apply(R, r, row_get<TS>(tile, li.parent, 0, t)) + Sqd;
            a = X_apply(R, r, row_get<TS>(tile, li.parent, 6, t)) + sv(J.thdd * s, v3(0.f, 0.f, 0.f)) + crm(v, Sqd);
            row_put<TS>(tile, l, 0, t, v);
            row_put<TS>(tile, l, 6, t, a);
        }
    }
    // link forces
    SV F = zero;
    float *ck = cache + (int64_t)(l * 18) * B + b;
    if (link) {
        F = I_apply(lf, a) + crf(v, I_apply(lf, v));
        if (f_ext) F = F - ld_sv(f_ext + (int64_t)(l * 6) * B + b, B);
        if (valid) {
            st_sv(ck, B, v);
            st_sv(ck + 6 * B, B, a);
        }
    }
    // tips -> base: each link adds its children's forces, in its coordinates
    const int child = link ? rb.kids[l] : -1;
    for (int d = rb.max_depth; d >= 1; --d) {
        __syncthreads();
        if (link && li.depth == d) {
            for (int c = child; c >= 0; c = rb.kids[64 + c]) F += row_get<TS>(tile, c, 0, t);
            if (d > 1) row_put<TS>(tile, l, 0, t, XT_apply(R, r, F));
        }
    }
    if (link && valid) st_sv(ck + 12 * B, B, F);
    const float x = link && li.revolute ? lf.mult * dot(s, F.w) : 0.f;
    if (rb.simple_joints) {
        if (link && li.revolute && valid) tau[(int64_t)li.jidx * B + b] = x;
    } else {
        const float sum = joint_sum<TS>(tile, rb, fz, l, t, x);
        if (l < rb.n && valid) tau[(int64_t)l * B + b] = sum;
    }
}

// The exact reverse mode of it (sweeps A and B above), v, a and F read from
// the cache (humanoid: 11.5 us at 1,024 states, 64 us at 24,576, where the
// bytes take 26; one state per lane 127 and 189).
template <int TS>
__global__ void __launch_bounds__(64 * TS) k_rnea_backward_levels(DevRobot rb, DevFused fz, int64_t nb, int64_t B,
                                                                  const float *__restrict__ q,
                                                                  const float *__restrict__ qd,
                                                                  const float *__restrict__ qdd,
                                                                  const float *__restrict__ cache,
                                                                  const float *__restrict__ g_tau,
                                                                  float *__restrict__ g_q, float *__restrict__ g_qd,
                                                                  float *__restrict__ g_qdd,
                                                                  float *__restrict__ g_fext) {
    extern __shared__ float tile[];
    const int t = threadIdx.x % TS, l = threadIdx.x / TS;
    const int64_t s0 = (int64_t)xcd_chunk() * TS, b = min(s0 + t, nb - 1);
    const bool link = l > 0 && l < rb.L, valid = s0 + t < nb;
    const SV zero = sv(v3(0.f, 0.f, 0.f), v3(0.f, 0.f, 0.f));
    LinkI li{};
    LinkF lf{};
    JointIn J{0.f, 0.f, 0.f};
    M3 R;
    SV v = zero;
    if (link) {
        li = rb.li[l];
        lf = rb.lf[l];
        const float *ck = cache + (int64_t)(l * 18) * B + b;
        v = ld_sv(ck, B);
        row_put<TS>(tile, l, 0, t, v);
        row_put<TS>(tile, l, 6, t, ld_sv(ck + 6 * B, B));
        J = joint_in(lf, li, q, qd, qdd, B, b);
        R = local_rotation(lf, li, J.th);
    } else if (l == 0) {
        row_put<TS>(tile, 0, 0, t, zero);
        row_put<TS>(tile, 0, 6, t, sv(v3(0.f, 0.f, 0.f), v3(-rb.gx, -rb.gy, -rb.gz)));
    }
    const V3 r = v3(lf.fp[0], lf.fp[1], lf.fp[2]), s = v3(lf.axis[0], lf.axis[1], lf.axis[2]);
    const bool revolute = link && li.revolute;
    // s x the parent's acceleration and velocity in this link's coordinates
    __syncthreads();
    SV sXa = zero, sXv = zero;
    if (revolute) {
        const SV Xv = X_apply(R, r, row_get<TS>(tile, li.parent, 0, t)), Xa = X_apply(R, r, row_get<TS>(tile, li.parent, 6, t));
        sXa = sv(cross(s, Xa.w), cross(s, Xa.l));
        sXv = sv(cross(s, Xv.w), cross(s, Xv.l));
    }
    // sweep A, base -> tips: adjoint of the force accumulation
    __syncthreads();
    if (l == 0) row_put<TS>(tile, 0, 0, t, zero);
    const float tb = revolute ? lf.mult * g_tau[(int64_t)li.jidx * B + b] : 0.0f;
    SV Fb = zero, XFp = zero;
    for (int d = 1; d <= rb.max_depth; ++d) {
        __syncthreads();
        if (link && li.depth == d) {
            XFp = X_apply(R, r, row_get<TS>(tile, li.parent, 0, t));
            Fb = sv(tb * s, v3(0.f, 0.f, 0.f)) + XFp;
            row_put<TS>(tile, l, 0, t, Fb);
        }
    }
    if (g_fext && l < rb.L && valid) st_sv(g_fext + (int64_t)(l * 6) * B + b, B, zero - Fb);   // the base's reaches no joint
    float th_b = 0.f;
    if (revolute) {
        const SV F = ld_sv(cache + (int64_t)(l * 18 + 12) * B + b, B);
        th_b = dot(XFp.w, cross(s, F.w)) + dot(XFp.l, cross(s, F.l));
    }
    // sweep B, tips -> base: adjoint of the velocity/acceleration recursion
    SV ab = I_apply(lf, Fb);
    SV vb = zero - (crf(Fb, I_apply(lf, v)) + I_apply(lf, crm(v, Fb)));
    const SV Sqd = sv(J.thd * s, v3(0.f, 0.f, 0.f));
    const int child = link ? rb.kids[l] : -1;
    for (int d = rb.max_depth; d >= 1; --d) {
        __syncthreads();
        if (link && li.depth == d) {
            for (int c = child; c >= 0; c = rb.kids[64 + c]) {
                ab += row_get<TS>(tile, c, 0, t);
                vb += row_get<TS>(tile, c, 6, t);
            }
            vb += crf(Sqd, ab);
            if (d > 1) {
                row_put<TS>(tile, l, 0, t, XT_apply(R, r, ab));
                row_put<TS>(tile, l, 6, t, XT_apply(R, r, vb));
            }
        }
    }
    float thd_b = 0.f, thdd_b = 0.f;
    if (revolute) {
        thdd_b = lf.mult * dot(s, ab.w);
        thd_b = lf.mult * (dot(s, vb.w) - dot(s, crf(v, ab).w));
        th_b = lf.mult * (th_b - (dot(ab, sXa) + dot(vb, sXv)));
    }
    if (rb.simple_joints) {
        if (revolute && valid) {
            const int64_t o = (int64_t)li.jidx * B + b;
            g_q[o] = th_b;
            g_qd[o] = thd_b;
            g_qdd[o] = thdd_b;
        }
        return;
    }
    th_b = joint_sum<TS>(tile, rb, fz, l, t, th_b);
    thd_b = joint_sum<TS>(tile, rb, fz, l, t, thd_b);
    thdd_b = joint_sum<TS>(tile, rb, fz, l, t, thdd_b);
    if (l < rb.n && valid) {
        const int64_t o = (int64_t)l * B + b;
        g_q[o] = th_b;
        g_qd[o] = thd_b;
        g_qdd[o] = thdd_b;
    }
}

hipError_t launch_rnea(const DevRobot &rb, int64_t B, int64_t ld, const float *q, const float *qd,
                       const float *qdd, const float *f_ext, float *tau, float *cache, hipStream_t s) {
    if (B == 0) return hipSuccess;
    dim3 grid((unsigned)((B + 255) / 256));
    hipLaunchKernelGGL(k_rnea, grid, dim3(256), 0, s, rb, B, ld, q, qd, qdd, f_ext, tau, cache);
    return hipGetLastError();
}

hipError_t launch_rnea_backward(const DevRobot &rb, int64_t B, int64_t ld, const float *q, const float *qd,
                                const float *qdd, const float *cache, const float *g_tau,
                                float *g_q, float *g_qd, float *g_qdd, float *g_fext, float *ws, hipStream_t s) {
    if (B == 0) return hipSuccess;
    dim3 grid((unsigned)((B + 255) / 256));
    hipLaunchKernelGGL(k_rnea_backward, grid, dim3(256), 0, s, rb, B, ld, q, qd, qdd, cache, g_tau, g_q,
                       g_qd, g_qdd, g_fext, ws);
    return hipGetLastError();
}

// States a tile (wide: 8): 4 where a batch has to be spread over the chip, 8, whose
// pieces of a row are whole 32-byte sectors, from 8 states per compute unit on
// (forward / backward, 4 against 8 states: humanoid 10.8 / 11.2 against 11.0 /
// 11.5 us at 1,024 states, 15.5 / 15.8 against 13.9 / 13.6 at 4,096, 52 / 63
// against 54 / 64 at 24,576; 7-joint chain 7.3 / 7.5 against 6.8 / 7.1 at
// 4,096, 14.2 / 14.3 against 10.5 / 9.7 at 24,576).  16 states gain the chain
// another microsecond there and cost the humanoid 11.
// Threads of a tile's workgroup: one per (state, link), whole wavefronts.
static dim3 level_block(int L, int ts) { return dim3((unsigned)((L * ts + 63) / 64 * 64)); }

template <int TS>
static void launch_levels(const DevRobot &rb, const DevFused &fz, int64_t B, int64_t ld, const float *q,
                          const float *qd, const float *qdd, const float *f_ext, float *tau, float *cache,
                          hipStream_t s) {
    hipLaunchKernelGGL((k_rnea_levels<TS>), dim3((unsigned)((B + TS - 1) / TS)), level_block(rb.L, TS),
                       (size_t)rb.L * 12 * (TS + 1) * 4, s, rb, fz, B, ld, q, qd, qdd, f_ext, tau, cache);
}
template <int TS>
static void launch_backward_levels(const DevRobot &rb, const DevFused &fz, int64_t B, int64_t ld, const float *q,
                                   const float *qd, const float *qdd, const float *cache, const float *g_tau,
                                   float *g_q, float *g_qd, float *g_qdd, float *g_fext, hipStream_t s) {
    hipLaunchKernelGGL((k_rnea_backward_levels<TS>), dim3((unsigned)((B + TS - 1) / TS)), level_block(rb.L, TS),
                       (size_t)rb.L * 12 * (TS + 1) * 4, s, rb, fz, B, ld, q, qd, qdd, cache, g_tau, g_q, g_qd, g_qdd,
                       g_fext);
}

hipError_t launch_rnea_levels(const DevRobot &rb, const DevFused &fz, int64_t B, int64_t ld, const float *q,
                              const float *qd, const float *qdd, const float *f_ext, float *tau, float *cache,
                              bool wide, hipStream_t s) {
    return in_slices(B, [&](int64_t b0, int64_t n) {
        const auto launch = wide ? launch_levels<8> : launch_levels<4>;
        launch(rb, fz, n, ld, from(q, b0), from(qd, b0), from(qdd, b0), from(f_ext, b0), from(tau, b0), cache + b0, s);
    });
}

hipError_t launch_rnea_backward_levels(const DevRobot &rb, const DevFused &fz, int64_t B, int64_t ld, const float *q,
                                       const float *qd, const float *qdd, const float *cache, const float *g_tau,
                                       float *g_q, float *g_qd, float *g_qdd, float *g_fext, bool wide, hipStream_t s) {
    return in_slices(B, [&](int64_t b0, int64_t n) {
        const auto launch = wide ? launch_backward_levels<8> : launch_backward_levels<4>;
        launch(rb, fz, n, ld, from(q, b0), from(qd, b0), from(qdd, b0), cache + b0, from(g_tau, b0), from(g_q, b0),
               from(g_qd, b0), from(g_qdd, b0), from(g_fext, b0), s);
    });
}

}  // namespace wb
