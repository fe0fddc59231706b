// Small per-state kernels of the optimizer iteration: the hinge adjoint of
// self-collision (a state's spheres in runs over threads), the cost head (a
// state's joints in quarters over four threads) and the gradient step.  All
// keep the states along the lanes of [k][B] arrays (coalesced in B); nb is
// the number of states and B the row length of the arrays (the ABI's
// ld >= nb).
#include <algorithm>
#include "spatial.h"

namespace wb {

// Hinge h = max(0, max_pen + margin) at the most penetrating pair: its
// subgradient moves the two spheres of that pair apart along their centre
// line (cuRoboV2 Sec. 6.2 reduces to one most-penetrating pair per state).
// One thread per (state, run of `per` spheres), the state fastest: the
// [3S][B] output -- zero but for the pair's six entries -- is written in
// coalesced rows, and a state's pair and force are read and formed once per
// run.  Bound by the bytes written; one thread per row and state spent its
// time on launching 69 thousand workgroups (humanoid, 24,576 states).
__global__ void __launch_bounds__(256) k_sc_backward(DevRobot rb, int64_t nb, int64_t B, int per,
                                                     const float *__restrict__ sph,
                                                     const int32_t *__restrict__ argmax,
                                                     const float *__restrict__ max_pen, float margin,
                                                     const float *__restrict__ g_cost,
                                                     float *__restrict__ g_sph) {
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= nb) return;
    const int first = blockIdx.y * per, end = min(first + per, rb.S);
    const int p = argmax[b];
    const bool on = p >= 0 && p < rb.n_pairs && max_pen[b] + margin > 0.0f;
    const int s = on ? rb.pair_s[p] : -1, t = on ? rb.pair_t[p] : -1;
    V3 f = v3(0.f, 0.f, 0.f);   // the gradient on sphere t, its negative on s
    if ((s >= first && s < end) || (t >= first && t < end)) {
        const float *cs = sph + (int64_t)s * 3 * B + b;
        const float *ct = sph + (int64_t)t * 3 * B + b;
        const V3 d = v3(cs[0] - ct[0], cs[B] - ct[B], cs[2 * B] - ct[2 * B]);
        const float n = sqrtf(dot(d, d));
        if (n > 0.0f) f = (g_cost[b] / n) * d;
    }
    for (int i = first; i < end; ++i) {
        const V3 g = i == t ? f : (i == s ? -f : v3(0.f, 0.f, 0.f));
        float *o = g_sph + (int64_t)i * 3 * B + b;
        o[0] = g.x;
        o[B] = g.y;
        o[2 * B] = g.z;
    }
}

// Four threads per state, each a quarter of the joints in index order; their
// partial costs meet in LDS.  One thread per state read its joints one after
// the other on a few hundred wavefronts (humanoid, 24,576 states: 19 us).
constexpr int COST_SPLIT = 4;
__global__ void __launch_bounds__(256) k_cost_head(int64_t nb, int64_t B, int n, const float *__restrict__ tau,
                                                   const float *__restrict__ w, float tw,
                                                   const float *__restrict__ max_pen, float margin,
                                                   float hw, float *__restrict__ cost,
                                                   float *__restrict__ g_tau, float *__restrict__ g_mp) {
    __shared__ float part[COST_SPLIT][64];
    const int t = threadIdx.x & 63, quarter = threadIdx.x >> 6;
    const int64_t b = (int64_t)blockIdx.x * 64 + t;
    const int per = (n + COST_SPLIT - 1) / COST_SPLIT, j1 = min((quarter + 1) * per, n);
    float c = 0.0f;
    if (b < nb) {
#pragma unroll 4
        for (int j = quarter * per; j < j1; ++j) {
            const int64_t o = (int64_t)j * B + b;
            const float tj = tau[o];
            if (w) {
                const float wj = w[o];
                c = __builtin_fmaf(wj, tj, c);
                if (g_tau) g_tau[o] = wj;
            } else {
                c = __builtin_fmaf(tw * tj, tj, c);
                if (g_tau) g_tau[o] = 2.0f * tw * tj;
            }
        }
    }
    part[quarter][t] = c;
    __syncthreads();
    if (quarter != 0 || b >= nb) return;
    c = (part[0][t] + part[1][t]) + (part[2][t] + part[3][t]);
    if (max_pen) {
        const float h = max_pen[b] + margin;
        c += hw * fmaxf(h, 0.0f);
        if (g_mp) g_mp[b] = h > 0.0f ? hw : 0.0f;
    }
    if (cost) cost[b] = c;
}

// One thread per (joint, state): i = j * nb + b, at element j * B + b.
__global__ void __launch_bounds__(256) k_sgd_step(int64_t nb, int64_t B, int64_t total, float lr,
                                                  float *__restrict__ q, float *__restrict__ qd,
                                                  float *__restrict__ qdd, const float *__restrict__ g_q,
                                                  const float *__restrict__ g_q2, const float *__restrict__ g_qd,
                                                  const float *__restrict__ g_qdd) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= total) return;
    const int64_t j = t / nb, i = j * B + (t - j * nb);
    const float gq = g_q[i] + (g_q2 ? g_q2[i] : 0.0f);
    q[i] -= lr * gq;
    qd[i] -= lr * g_qd[i];
    qdd[i] -= lr * g_qdd[i];
}

hipError_t launch_self_collision_backward(const DevRobot &rb, int64_t B, int64_t ld, const float *spheres,
                                          const int32_t *argmax, const float *max_pen,
                                          float margin, const float *g_cost, float *g_sph,
                                          hipStream_t s) {
    if (B == 0 || rb.S == 0) return hipSuccess;
    // runs as long as they leave 2,048 workgroups, up to 16 spheres
    const int64_t blocks = (B + 255) / 256;
    const int per = (int)std::max<int64_t>(std::min<int64_t>(16, blocks * rb.S / 2048), 1);
    hipLaunchKernelGGL(k_sc_backward, dim3((unsigned)blocks, (unsigned)((rb.S + per - 1) / per)), dim3(256), 0, s, rb,
                       B, ld, per, spheres, argmax, max_pen, margin, g_cost, g_sph);
    return hipGetLastError();
}

hipError_t launch_cost_head(int64_t B, int64_t ld, int32_t n, const float *tau, const float *w, float tw,
                            const float *max_pen, float margin, float hw, float *cost,
                            float *g_tau, float *g_maxpen, hipStream_t s) {
    return in_slices(B, [&](int64_t b0, int64_t nb) {
        hipLaunchKernelGGL(k_cost_head, dim3((unsigned)((nb + 63) / 64)), dim3(256), 0, s, nb, ld, n, from(tau, b0),
                           from(w, b0), tw, from(max_pen, b0), margin, hw, from(cost, b0), from(g_tau, b0),
                           from(g_maxpen, b0));
    });
}

hipError_t launch_sgd_step(int64_t B, int64_t ld, int32_t n, float lr, float *q, float *qd, float *qdd,
                           const float *g_q, const float *g_q2, const float *g_qd,
                           const float *g_qdd, hipStream_t s) {
    const int64_t total = B * (int64_t)n;
    if (total == 0) return hipSuccess;
    hipLaunchKernelGGL(k_sgd_step, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, B, ld, total, lr, q,
                       qd, qdd, g_q, g_q2, g_qd, g_qdd);
    return hipGetLastError();
}

}  // namespace wb
