// Group-of-lanes tree operations shared by the kernels that give each state
// a group of G lanes (G = 16, 32 or 64) with lane i holding link perm[i] in
// depth-first post-order (the subtree of lane i is a lane range that ends at
// i): path sums by pointer jumping over the parent lanes,
// subtree sums as differences of a group scan, world-frame inertia
// products, and the per-lane forward kinematics.
#pragma once

#include "lanes.h"
#include "spatial.h"

namespace wb {

// ------------------------------------------------------------ group shuffles
__device__ __forceinline__ SV shfl_sv(SV x, int src, int G) {
    return sv(v3(__shfl(x.w.x, src, G), __shfl(x.w.y, src, G), __shfl(x.w.z, src, G)),
              v3(__shfl(x.l.x, src, G), __shfl(x.l.y, src, G), __shfl(x.l.z, src, G)));
}
__device__ __forceinline__ SV zsv() { return sv(v3(0.f, 0.f, 0.f), v3(0.f, 0.f, 0.f)); }

// Sum of x over the path from the root to this lane's link.  The root (a
// fixed link) and the lanes past the robot must hold zero: they are their
// own parents, so a chain that has reached the root keeps adding that zero,
// exactly, and no lane needs a guard (or a masked copy of x) per step.
__device__ __forceinline__ SV path_sum(SV x, int parent_lane, int steps, int G) {
    int anc = parent_lane;
    for (int s = 0; s < steps; ++s) {
        const SV y = shfl_sv(x, anc, G);
        anc = __shfl(anc, anc, G);
        x += y;
    }
    return x;
}

// The subtree of a lane: the group lanes (before, lane], or [0, lane] where
// there is none before it (then before is the lane itself and some is 0).
struct Subtree {
    int before;
    float some;
};
__device__ __forceinline__ Subtree subtree_of(int before, int glane) {
    return Subtree{before, before != glane ? 1.f : 0.f};
}
__device__ __forceinline__ bool in_subtree(Subtree t, int lane, int glane) {
    return lane <= glane && (t.some == 0.f || lane > t.before);
}

// Sum of x over this lane's subtree: the group's inclusive scan at the
// subtree's last lane (this one) less the scan before its first.  Lanes
// outside the robot must hold zero.
__device__ __forceinline__ SV subtree_sum(SV x, Subtree t, int G) {
    SV s = x;
    group_scan6(s.w.x, s.w.y, s.w.z, s.l.x, s.l.y, s.l.z, G);
    const SV y = shfl_sv(s, t.before, G);
    return sv(v3(__builtin_fmaf(-t.some, y.w.x, s.w.x), __builtin_fmaf(-t.some, y.w.y, s.w.y),
                 __builtin_fmaf(-t.some, y.w.z, s.w.z)),
              v3(__builtin_fmaf(-t.some, y.l.x, s.l.x), __builtin_fmaf(-t.some, y.l.y, s.l.y),
                 __builtin_fmaf(-t.some, y.l.z, s.l.z)));
}

// Half of a value of magnitude up to m, hi = (x + c) - c and lo = x - hi, c
// this constant: hi is on a grid so coarse (2^-17 of the power of two above m)
// that every partial sum of up to 64 of them is exact, so the scan difference
// of hi has no rounding at all and that of lo next to none beside m.
__device__ __forceinline__ float split_constant(float m) {
    // 1.5 * 2^(e + 6) with m < 2^e: adding it rounds to multiples of 2^(e - 17)
    return __builtin_amdgcn_ldexpf(1.5f, min(__builtin_amdgcn_frexp_expf(m) + 6, 127));
}
__device__ __forceinline__ V3 split_hi(V3 x, float c) {
    return v3((x.x + c) - c, (x.y + c) - c, (x.z + c) - c);
}

// The subtree sum with every component split so, for wrenches that cancel: a
// rounding or two of the result remain, and those of the scan of lo, at most
// 2^-36 of the group's largest value each.
// A serial chain subtracts nothing and takes the plain scan.
__device__ __forceinline__ SV subtree_sum_split(SV x, Subtree t, bool branched, int G) {
    if (!branched) return subtree_sum(x, t, G);
    float m = fmaxf(fmaxf(fabsf(x.w.x), fabsf(x.w.y)), fabsf(x.w.z));
    m = fmaxf(fmaxf(m, fabsf(x.l.x)), fmaxf(fabsf(x.l.y), fabsf(x.l.z)));
    const float c = split_constant(group_reduce_max(m, G));
    const SV hi = sv(split_hi(x.w, c), split_hi(x.l, c));
    return subtree_sum(hi, t, G) + subtree_sum(x - hi, t, G);
}

// The subtree sum of the links' wrenches with the force part split so, nine
// values scanned instead of six.  The torque and the VJP's angle adjoint
// multiply the accumulated force by arms about the world origin, and the
// rounding of its plain scan difference was most of their error (relative,
// 48-joint tree, fused: torque 4.8e-7 -> 2.9e-7, angle gradient 6.4e-7 ->
// 4.2e-7; a fused launch of the humanoid 1.7 % longer).
__device__ __forceinline__ SV subtree_sum_wrench(SV x, Subtree t, bool branched, int G) {
    if (!branched) return subtree_sum(x, t, G);
    const float c = split_constant(group_reduce_max(fmaxf(fmaxf(fabsf(x.l.x), fabsf(x.l.y)), fabsf(x.l.z)), G));
    const V3 hi = split_hi(x.l, c);
    V3 lo = x.l - hi;
    group_scan3(lo.x, lo.y, lo.z, G);
    SV s = subtree_sum(sv(x.w, hi), t, G);
    s.l += v3(__builtin_fmaf(-t.some, __shfl(lo.x, t.before, G), lo.x), __builtin_fmaf(-t.some, __shfl(lo.y, t.before, G), lo.y),
              __builtin_fmaf(-t.some, __shfl(lo.z, t.before, G), lo.z));
    return s;
}

// World-frame spatial inertia of a link: mass m, CoM cw and the rotational
// inertia about the CoM in world axes, Iw = R Ic R^T (xx yy zz xy xz yz).
struct WInertia {
    float m;
    V3 cw;
    float I[6];
};
__device__ __forceinline__ SV iw_apply(const WInertia &J, SV u) {
    const V3 h = J.m * (u.l + cross(u.w, J.cw));
    const V3 Iw = v3(J.I[0] * u.w.x + J.I[3] * u.w.y + J.I[4] * u.w.z,
                     J.I[3] * u.w.x + J.I[1] * u.w.y + J.I[5] * u.w.z,
                     J.I[4] * u.w.x + J.I[5] * u.w.y + J.I[2] * u.w.z);
    return sv(Iw + cross(J.cw, h), h);
}
// R Ic R^T for a symmetric Ic given as xx yy zz xy xz yz.
__device__ __forceinline__ void rotate_inertia(const M3 &R, const float *Ic, float *Iw) {
    float T[9];   // R Ic
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const float r0 = R.m[3 * i], r1 = R.m[3 * i + 1], r2 = R.m[3 * i + 2];
        T[3 * i + 0] = r0 * Ic[0] + r1 * Ic[3] + r2 * Ic[4];
        T[3 * i + 1] = r0 * Ic[3] + r1 * Ic[1] + r2 * Ic[5];
        T[3 * i + 2] = r0 * Ic[4] + r1 * Ic[5] + r2 * Ic[2];
    }
    const int ii[6] = {0, 1, 2, 0, 0, 1}, jj[6] = {0, 1, 2, 1, 2, 2};
#pragma unroll
    for (int e = 0; e < 6; ++e)
        Iw[e] = T[3 * ii[e]] * R.m[3 * jj[e]] + T[3 * ii[e] + 1] * R.m[3 * jj[e] + 1] +
                T[3 * ii[e] + 2] * R.m[3 * jj[e] + 2];
}

// Adjoints of a link's joint angle (returned), rate and acceleration, from
// the adjoint fb of its accumulated force (the path sum of taub S), all in
// world coordinates:
//   A = subsum(I fb),  V = subsum((S qd) x* A - fb x* I v - I (v x fb))
//   qdd-bar = S.A,  qd-bar = S.V + (v x S).A
//   q-bar = (fb x S).F + ((a - qd v x S) x S).A + (v x S).V
// A and V are the total adjoints of the link's acceleration and velocity;
// the angle enters the recursions through this link's transform alone
// (dX = -crm(S) X), once each for the parent's velocity v - S qd, the
// parent's acceleration a - S qdd - qd v x S and the force passed to the
// parent, whose adjoint is fb - taub S (every S x S vanishes).  Against
// summing the turned axes and inertias of the whole subtree this takes one
// of three subtree sums and four force products out of the VJP (fused
// iteration of the humanoid, 24,576 states: 108 -> 103 us a launch).
// c = v x S, Iv = I v; subsum the subtree sum to use.  Lanes outside the
// robot must hold zeros.
template <typename Sum>
__device__ __forceinline__ float rnea_adjoint(SV S, SV c, SV v, SV a, SV F, const WInertia &J, SV Iv, SV fb,
                                              float thd, Sum subsum, float &thd_b, float &thdd_b) {
    const SV Acc = subsum(iw_apply(J, fb));
    const SV V = subsum(thd * crf(S, Acc) - (crf(fb, Iv) + iw_apply(J, crm(v, fb))));
    thdd_b = dot(S, Acc);
    thd_b = dot(S, V) + dot(c, Acc);
    return dot(crm(fb, S), F) + dot(crm(a - thd * c, S), Acc) + dot(c, V);
}

// Lane, within the group whose first lane is `first`, for which `mine`
// holds (it holds for exactly one lane of every group).
__device__ __forceinline__ int group_lane_of(bool mine, int first) { return __ffsll(__ballot(mine) >> first) - 1; }

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Sum over the links joint `glane` drives (connectedLinks, lanes of the
// group) of their x; 0 in lanes past the last joint.
__device__ __forceinline__ float gather_joint(float x, const DevFused &fz, int glane, int G) {
    float acc = 0.f;
    for (int kk = 0; kk < fz.mc; ++kk) {
        const int l = fz.conn[kk * 64 + glane];
        const float y = __shfl(x, l >= 0 ? l : glane, G);
        if (l >= 0) acc += y;
    }
    return acc;
}

// World pose (R, p) of the lane's link: the lane's local transform (fixed
// rotation and translation, then the joint rotation by angle th), composed
// with its ancestors' by pointer jumping, T <- T_anc o T, anc <- anc(anc),
// `steps` times.  The root (a fixed link) and the lanes past the robot hold
// the identity and are their own ancestors, so a chain that has reached
// the root keeps composing with the identity, exactly.
__device__ __forceinline__ void lane_world_pose(const DevFused &fz, int gl, bool revolute, float th, int parent_lane,
                                                int G, M3 &R, V3 &p) {
    const float *lf = fz.lf;
    const int *li = fz.li;
#pragma unroll
    for (int t = 0; t < 9; ++t) R.m[t] = lf[(3 + t) * 64 + gl];
    p = v3(lf[12 * 64 + gl], lf[13 * 64 + gl], lf[14 * 64 + gl]);
    if (revolute) {
        float s, c;
        sincosf(th, &s, &c);
        const M3 Jr = axis_angle(v3(lf[0 * 64 + gl], lf[1 * 64 + gl], lf[2 * 64 + gl]), s, c);
        R = li[6 * 64 + gl] ? Jr : matmul(R, Jr);
    }
    int anc = parent_lane;
    for (int st = 0; st < fz.jsteps; ++st) {
        M3 Ra;
#pragma unroll
        for (int t = 0; t < 9; ++t) Ra.m[t] = __shfl(R.m[t], anc, G);
        const V3 pa = v3(__shfl(p.x, anc, G), __shfl(p.y, anc, G), __shfl(p.z, anc, G));
        anc = __shfl(anc, anc, G);
        p = mul(Ra, p) + pa;
        R = matmul(Ra, R);
    }
}

}  // namespace wb
