// Internal structures shared by the host code and the HIP kernels of libwb.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>
#include "wb.h"

namespace wb {

// Per-link float record, 32 floats (128 bytes) so a uniform link index turns
// into one scalar-cache fetch in lane-per-state kernels.
struct LinkF {
    float axis[3];     // 0
    float fR[9];       // 3   row-major fixed rotation
    float fp[3];       // 12  fixed translation (child joint origin in parent frame)
    float mult;        // 15
    float offset;      // 16
    float mass;        // 17
    float com[3];      // 18
    float I[6];        // 21  xx yy zz xy xz yz about the CoM, link axes
    float pad[5];      // 27
};
static_assert(sizeof(LinkF) == 128, "LinkF layout");

// Per-link integer record.
struct LinkI {
    int32_t parent;
    int32_t revolute;  // 1 if the link has a revolute joint
    int32_t jidx;      // actuated joint, -1 if fixed
    int32_t sph_first;
    int32_t sph_count;
    int32_t depth;
    int32_t fR_identity;  // fixed rotation is exactly the identity
    int32_t far_child;    // has a child other than link k+1
};
static_assert(sizeof(LinkI) == 32, "LinkI layout");

// Device view of a robot, passed by value to kernels.
struct DevRobot {
    int32_t L, n, S, nmax;        // nmax: sphere slots per link (max spheres on a link)
    int32_t n_blocks, n_blocks_pad, max_depth, simple_joints;  // simple: one link per actuated joint, mult 1, offset 0
    int64_t n_pairs;
    float gx, gy, gz;
    float broad_tol;              // rounding allowance of the matrix-core broad phase (sweep.h)
    const LinkF *__restrict__ lf;         // [L]
    const LinkI *__restrict__ li;         // [L]
    const float4 *__restrict__ sph;       // [S] local centre + radius
    const int32_t *__restrict__ sph_link; // [S]
    const int32_t *__restrict__ sph_slot; // [S] padded slot a*nmax + (s - first sphere of a)
    const float *__restrict__ slot_r;     // [(L+1)*nmax] radius of slot (a,i), -1e30 for empty slots
    const uint32_t *__restrict__ blocks;  // [n_blocks_pad] (16 a) << 16 | 16 b, padded to a multiple of 128 with the pair (L, L)
    const uint32_t *__restrict__ allow;   // [2][64] checked link pairs by matrix-core result (sweep.h); robots of at most 64 links
    const int32_t *__restrict__ kids;     // [2][64] highest child of a link, next lower sibling (-1: none); at most 64 links
    const int32_t *__restrict__ pair_off; // [S] index of sphere s's first pair
    const int32_t *__restrict__ pair_cnt; // [L*L] pairs of a sphere on link a with links a<b'<b
    const int32_t *__restrict__ pair_s;   // [P]
    const int32_t *__restrict__ pair_t;   // [P]
};

// Per-lane tables of the fused kernel: lane i holds link perm[i] in
// depth-first post-order, so the subtree of lane i is a lane range that ends
// at i.  Structure of arrays, 64 entries per field.
//   li[f*64 + i]: f = 0 link, 1 parent lane (own lane: the root), 2 the lane
//                 before the subtree's first (own lane: the subtree starts
//                 at lane 0), 3 joint index (-1 fixed), 4 sphere count,
//                 5 revolute, 6 fixed rotation is the identity
//   lf[f*64 + i]: f = 0..2 axis, 3..11 fixed R, 12..14 fixed p, 15 mass,
//                 16..18 CoM, 19..24 inertia (xx yy zz xy xz yz),
//                 25..27 centre and 28 radius of the link's bounding sphere in
//                 link coordinates, the sweep's rounding margin for any state
//                 of the robot included (-1e30 without spheres), 29 joint
//                 multiplier, 30 joint offset
//   lsph[j*64 + i]: local centre and radius of the link's j-th sphere
//   conn[k*64 + j]: lane of the k-th link that joint j drives, -1 past the
//                 end of the list (read only when mimic is set)
// Lanes past the last link hold an empty link: link -1, their own parent, no
// joint, no spheres, identity fixed rotation, zero mass.
struct DevFused {
    int32_t supported;   // L <= 64 and the sweep tables fit the LDS budget
    int32_t jsteps;      // pointer-jumping steps, ceil(log2(max_depth + 1))
    int32_t mimic;       // some joint drives several links, or a multiplier != 1 or offset != 0
    int32_t mc;          // longest connectedLinks list
    int32_t branched;    // some subtree does not start at lane 0 (not a serial chain)
    const int32_t *__restrict__ li;
    const float *__restrict__ lf;
    const float4 *__restrict__ lsph;
    const int32_t *__restrict__ conn;
};

// Device pointers of one robot's batch in a fused iteration.
struct TreeIO {
    float *q, *qd, *qdd;          // [n][B], updated in place when lr != 0
    const float *w;               // [n][B] or null
    float *tau, *cost, *max_pen;  // optional outputs
    int32_t *argmax, *n_coll;
    float *g_q, *g_qd, *g_qdd;
    const float *f_ext;           // [L][6][B] external link forces (link coordinates) or null
    float *g_fext;                // [L][6][B] their gradient or null
    int64_t ld;                   // row length B of the [k][B] arrays (>= the states)
};

// Scalars of the cost head and the step.
struct StepScalars {
    float torque_weight, margin, hinge_weight, lr;
};

// The spline-sampling form of the fused iteration: its states are the
// samples of uniform cubic B-splines (four per knot interval), formed in the
// kernel from the control points instead of read from q, qd, qdd.
struct SplineIn {
    float *U;                              // [d][T][K] control points, or null (states from io.q, qd, qdd)
    const float *th0, *dth0, *ddth0;       // [d][T] initial states (dth0, ddth0 may be null: at rest)
    int32_t T, K, H, printed;              // trajectories, control points, samples per trajectory, ghost reading
    float dt;
    // the control-point gradient reduced in the kernel (each workgroup owns
    // whole trajectories), then the step: g_U [d][T][K] (may be null), lr,
    // step rule (WB_STEP_*)
    float *g_U;
    float lr;
    int32_t rule;
};

// Arguments of the single-robot fused kernel (by value).
struct FusedArgs {
    DevRobot rb;
    DevFused fz;
    TreeIO io;
    SplineIn sp;
    StepScalars k;
    int64_t B;                // states (the arrays' row length is io.ld)
    int32_t chunk;            // states per four wavefronts (launch_fused takes each its share)
    int32_t lanes_per_state;  // G: 16, 32 or 64
};

// One robot of an uneven batch, and one unit of work of the persistent launch.
struct PlanTree {
    DevRobot rb;              // tables re-derived for the plan's slots per link
    DevFused fz;
    int64_t B;                // states (the arrays' row length is the run's io.ld)
    int32_t lanes_per_state;
    int32_t pad;
};
struct PlanItem {
    int64_t b0;
    int32_t tree, count;
};

#define WB_PLAN_MAX_TREES 16
struct PlanArgs {
    const PlanTree *trees;
    const PlanItem *items;        // grouped by workgroup
    const int32_t *item_start;    // [n_wg + 1]
    StepScalars k;
    TreeIO io[WB_PLAN_MAX_TREES];
};

hipError_t launch_fused(const FusedArgs &a, hipStream_t s);
hipError_t launch_plan(const PlanArgs &a, int nmax, int n_wg, size_t lds, bool ext, hipStream_t s);
// Workgroups of the plan kernel (variant nmax, ext, `lds` bytes of dynamic
// LDS) that one compute unit keeps resident; at least 1.
int plan_workgroups_per_cu(int nmax, bool ext, size_t lds);

// Kernel launchers (each defined next to its kernels).
hipError_t launch_fk(const DevRobot &rb, int64_t B, int64_t ld, const float *q, float *pose, float *spheres,
                     hipStream_t s);
hipError_t launch_fk_backward(const DevRobot &rb, int64_t B, int64_t ld, const float *q, const float *pose,
                              const float *g_pose, const float *g_sph, float *g_q, float *ws,
                              hipStream_t s);
hipError_t launch_rnea(const DevRobot &rb, int64_t B, int64_t ld, const float *q, const float *qd,
                       const float *qdd, const float *f_ext, float *tau, float *cache, hipStream_t s);
hipError_t launch_rnea_backward(const DevRobot &rb, int64_t B, int64_t ld, const float *q, const float *qd,
                                const float *qdd, const float *cache, const float *g_tau,
                                float *g_q, float *g_qd, float *g_qdd, float *g_fext, float *ws, hipStream_t s);
// A grid holds fewer than 2^32 threads.  Kernels with several threads a state
// are launched on slices of a batch, so that the batches that one thread a
// state reached (up to 2^31 - 1) still run: f(b0, n) for the states b0 .. b0 + n - 1.
constexpr int64_t SLICE_STATES = (int64_t)1 << 24;
template <typename F>
inline hipError_t in_slices(int64_t B, F f) {
    for (int64_t b0 = 0; b0 < B; b0 += SLICE_STATES) {
        f(b0, B - b0 < SLICE_STATES ? B - b0 : SLICE_STATES);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}
template <typename T>
inline T *from(T *rows, int64_t b0) {
    return rows ? rows + b0 : nullptr;
}

// The same level by level, one thread per (state, link), in tiles of 4 states
// (wide: 8); robots of at most 64 links.
hipError_t launch_rnea_levels(const DevRobot &rb, const DevFused &fz, int64_t B, int64_t ld, const float *q,
                              const float *qd, const float *qdd, const float *f_ext, float *tau, float *cache,
                              bool wide, hipStream_t s);
hipError_t launch_rnea_backward_levels(const DevRobot &rb, const DevFused &fz, int64_t B, int64_t ld, const float *q,
                                       const float *qd, const float *qdd, const float *cache, const float *g_tau,
                                       float *g_q, float *g_qd, float *g_qdd, float *g_fext, bool wide, hipStream_t s);
// Group-per-state RNEA and VJP without a cache (tree_kernels.hip); robots of
// at most 64 links.
hipError_t launch_rnea_lanes(const DevRobot &rb, const DevFused &fz, int64_t B, int64_t ld, const float *q,
                             const float *qd, const float *qdd, const float *f_ext, float *tau, hipStream_t s);
hipError_t launch_rnea_backward_lanes(const DevRobot &rb, const DevFused &fz, int64_t B, int64_t ld,
                                      const float *q, const float *qd, const float *qdd, const float *f_ext,
                                      const float *g_tau, float *g_q, float *g_qd, float *g_qdd, float *g_fext,
                                      hipStream_t s);
// FK and its adjoint through LDS tiles (tree_kernels.hip), robots of at most
// 64 links: a group of lanes per state (wide: tiles of 16, backward 8, states
// instead of 4), or level by level.
hipError_t launch_fk_levels(const DevRobot &rb, int64_t B, int64_t ld, const float *q, float *pose, float *spheres,
                            hipStream_t s);
hipError_t launch_fk_lanes(const DevRobot &rb, const DevFused &fz, int64_t B, int64_t ld, const float *q, float *pose,
                           float *spheres, bool wide, hipStream_t s);
hipError_t launch_fk_backward_lanes(const DevRobot &rb, const DevFused &fz, int64_t B, int64_t ld, const float *q,
                                    const float *g_pose, const float *g_sph, float *g_q, bool wide, hipStream_t s);
hipError_t launch_fk_backward_levels(const DevRobot &rb, const DevFused &fz, int64_t B, int64_t ld, const float *q,
                                     const float *g_pose, const float *g_sph, float *g_q, hipStream_t s);
// split: one state per workgroup with its pairs over the four wavefronts
// (else one state per wavefront).
hipError_t launch_self_collision(const DevRobot &rb, int64_t B, int64_t ld, const float *spheres,
                                 float *max_pen, int32_t *argmax, int32_t *n_coll, bool split, hipStream_t s);
hipError_t launch_self_collision_backward(const DevRobot &rb, int64_t B, int64_t ld, const float *spheres,
                                          const int32_t *argmax, const float *max_pen,
                                          float margin, const float *g_cost, float *g_sph,
                                          hipStream_t s);
hipError_t launch_cost_head(int64_t B, int64_t ld, int32_t n, const float *tau, const float *w, float tw,
                            const float *max_pen, float margin, float hw, float *cost,
                            float *g_tau, float *g_maxpen, hipStream_t s);
hipError_t launch_sgd_step(int64_t B, int64_t ld, int32_t n, float lr, float *q, float *qd, float *qdd,
                           const float *g_q, const float *g_q2, const float *g_qd,
                           const float *g_qdd, hipStream_t s);

hipError_t launch_bspline_eval(int64_t T, int32_t d, int32_t K, int32_t n_interp, float dt, int32_t printed,
                               const float *U, const float *th0, const float *dth0, const float *ddth0, float *q,
                               float *qd, float *qdd, hipStream_t s);
hipError_t launch_bspline_backward(int64_t T, int32_t d, int32_t K, int32_t n_interp, float dt, const float *g_q,
                                   const float *g_qd, const float *g_qdd, float *g_U, float lr, int32_t rule,
                                   float *U, hipStream_t s);

constexpr size_t LDS_LIMIT = 65536;

// LDS of one state's sweep: (L+1)*nmax sphere slots and L+1 link bounding
// spheres (float4 each); plus, per sweeping group, a list of surviving blocks
// and a ring of row codes (32-bit each).
// The list takes every block of a small robot and up to 512 at a time of a
// large one, the ring two rows per lane of the group (of G lanes).
constexpr int SWEEP_LIST = 512;       // a multiple of 128
__host__ __device__ inline int sweep_list(int n_blocks, int G) {
    const int all = (n_blocks + 2 * G - 1) / (2 * G) * (2 * G);
    return all < SWEEP_LIST ? all : SWEEP_LIST;
}
__host__ __device__ inline int sweep_ring(int G) { return 2 * G; }
__host__ __device__ inline size_t state_lds_bytes(int L, int nmax) { return (size_t)(L + 1) * (nmax + 1) * 16; }
__host__ __device__ inline size_t group_lds_bytes(int L, int nmax, int n_blocks, int G) {
    return state_lds_bytes(L, nmax) + (size_t)(sweep_list(n_blocks, G) + sweep_ring(G)) * 4;
}
// Blocks from which the one-state-per-wavefront fused sweep tests them on the
// matrix cores (sweep.h).  Direct / matrix form, us a fused launch of 16,384
// states: 946 blocks 74.4 / 77.0, 861 72.5 / 75.5, 780 70.3 / 71.4 to 73.2, 630
// 63.5 / 66.9, 253 52.5 / 58.0; 1,035 blocks 70.8 / 69.0, 1,128 (trees of 49
// links) 136.7 / 134.3, 79.9 / 79.5 and 78.4 / 78.6, a humanoid of as many x
// 24,576 92.6 / 88.0.  With one sphere a link the forms already cross at 650.
constexpr int BROAD_MATRIX_FROM = 1024;

// LDS copy of the block table (n_blocks_pad entries, a multiple of 128).
__host__ __device__ inline size_t tab_lds_bytes(int n_blocks_pad) { return (size_t)n_blocks_pad * 4; }
// Shapes of the standalone sweeps, all within LDS_LIMIT for every robot that
// wb_robot_create takes (one state and 4 KB fit).
constexpr int SC_RING = 128;          // row ring of a 64-lane group
struct SweepShape {
    int states;        // states side by side in a workgroup (wave form)
    int table, list;   // block table staged in LDS; entries of a wavefront's list
    size_t lds;
};
// One state per wavefront: four side by side with the block table beside them,
// or without it, or as many as fit, each with its own ring and list.
inline SweepShape sweep_wave_shape(int L, int nmax, int n_blocks_pad) {
    const size_t one = state_lds_bytes(L, nmax) + 4 * (SC_RING + SWEEP_LIST);
    if (4 * one + tab_lds_bytes(n_blocks_pad) <= LDS_LIMIT)
        return SweepShape{4, 1, SWEEP_LIST, 4 * one + tab_lds_bytes(n_blocks_pad)};
    const int fit = (int)(LDS_LIMIT / one), states = fit < 4 ? fit : 4;
    return SweepShape{states, 0, SWEEP_LIST, states * one};
}
// One state per workgroup: with the block table, without it, and with lists of
// one 128-entry chunk where those of two do not fit.  Two chunks: longer lists
// save sweeps of a few rows but cost workgroups on a compute unit (101 links
// of 7 spheres, 1,000 states, lists of 128 / 256 / 512 entries 48 / 45 / 54 us;
// 261 links of 5: 125 / 101 / 99; 49 of 24, 4,095 states: 207 / 202 / 226).
constexpr int SPLIT_LIST = 256;
inline SweepShape sweep_split_shape(int L, int nmax, int n_blocks_pad) {
    const size_t state = state_lds_bytes(L, nmax), full = state + 4 * 4 * (SC_RING + SPLIT_LIST);
    if (full + tab_lds_bytes(n_blocks_pad) <= LDS_LIMIT)
        return SweepShape{1, 1, SPLIT_LIST, full + tab_lds_bytes(n_blocks_pad)};
    if (full <= LDS_LIMIT) return SweepShape{1, 0, SPLIT_LIST, full};
    return SweepShape{1, 0, 128, state + 4 * 4 * (SC_RING + 128)};
}
// Rows (a block times the slots of its first link) up to which the wave form
// evaluates every row: testing and queueing so few takes longer (9 states, with
// the queue / without: 4 links of 5 spheres 5.40 / 5.10 us, 8 of 5 5.81 / 5.34,
// 9 of 2 4.64 / 4.29).
constexpr int DIRECT_ROWS = 128;
// Default threshold between the two, in states per compute unit: the split
// form below it.
//   0 for robots of at most DIRECT_ROWS rows and 16 slots (8 links of 5, wave /
//     split form: 5.3 / 6.0 us at 9 states, 5.9 / 6.2 at 138, 5.9 / 6.6 at 512);
//   2 with at most 128 link blocks, one chunk, which one wavefront sweeps in
//     either form; below, one state per wavefront leaves SIMDs without work;
//   6 with more (wave / split form, us, at 1,000 and 2,048 states: 41 links of
//     4 spheres 12.6 / 10.8, 14.5 / 15.9; 25 of 8: 13.6 / 12.6, 15.5 / 21.7;
//     101 of 1: 15.6 / 11.0, 16.3 / 19.6; a humanoid 13.3 / 11.9, 13.4 / 20.5);
//   16 for robots of more than 40,000 pairs, most of which stay ahead in the
//     split form to 4,096 states (61 links of 8: 46.8 / 43.5 at 2,048, 82 / 67
//     at 4,096; 61 of 12: 76 / 67, 139 / 107; 49 of 16: 99 / 81, 167 / 129; the
//     earliest, 21 of 16, crosses at 1,100), and for those of which 64 KB hold
//     fewer than four states, whose wave form leaves wavefronts idle (49 links
//     of 48: 533 / 223 at 512, 1,018 / 613 at 2,048).
inline int sweep_split_per_cu(int L, int nmax, int n_blocks, int64_t n_pairs) {
    if (nmax <= 16 && n_blocks * nmax <= DIRECT_ROWS) return 0;
    if (n_blocks <= 128) return 2;
    return n_pairs > 40000 || sweep_wave_shape(L, nmax, (n_blocks + 127) / 128 * 128).states < 4 ? 16 : 6;
}

// LDS of a workgroup of the fused kernel with G lanes per state and `waves`
// wavefronts: their group regions, then, for four, the block table.
inline size_t fused_lds_bytes(int L, int nmax, int n_blocks, int G, int waves) {
    return (size_t)waves * (64 / G) * group_lds_bytes(L, nmax, n_blocks, G) +
           (waves > 1 ? tab_lds_bytes((n_blocks + 127) / 128 * 128) : 0);
}
// What a fused shape or a plan is held against LDS_LIMIT by: a workgroup of
// four wavefronts with 16-bit lists of up to 2,048 blocks and a 16-bit table.
// It decides which robots and shapes are accepted, and is not what a launch
// takes: the fused and plan kernels' workgroups are one wavefront, of at most
// 17 KB; the one-launch B-spline step, four wavefronts with 32-bit lists and
// table, takes up to 7 KB more than is counted, 71 KB at most of the 160 KB
// that a workgroup may have, and two still share a compute unit.
inline size_t counted_group_bytes(int L, int nmax, int n_blocks_pad) {
    const int cap = n_blocks_pad < 128 ? 128 : (n_blocks_pad > 2048 ? 2048 : n_blocks_pad);
    return state_lds_bytes(L, nmax) + (size_t)cap * 2 + (size_t)128 * 4;
}
inline size_t counted_tab_bytes(int n_blocks_pad) { return (size_t)n_blocks_pad * 2; }
inline size_t counted_fused_bytes(int L, int nmax, int G, int n_blocks_pad) {
    return (size_t)4 * (64 / G) * counted_group_bytes(L, nmax, n_blocks_pad) + counted_tab_bytes(n_blocks_pad);
}
// LDS of the in-kernel control-point gradient beyond the fused kernel's:
// one partial sum per group of lanes (4 * 64 / G of them) over the
// d x (K + 6) extended knots, then the d x K reduced gradient.
inline size_t spline_lds_bytes(int G, int d, int K) {
    return ((size_t)(256 / G) * (K + 6) + (size_t)K) * d * 4;
}
// Sphere slots per link the fused kernels are instantiated for: 1 to 8, and
// 12 (links of up to 12 spheres are padded to 12 slots).
constexpr int FUSED_MAX_SLOTS = 12;

// Workspace floats per state needed by the backward kernels.
inline int64_t workspace_floats_per_state(int L) { return (int64_t)L * 18 + 8; }

}  // namespace wb
