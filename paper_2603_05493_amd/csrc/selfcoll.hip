// Standalone self-collision kernels (cuRoboV2 Sec. 6.2): a state's sphere
// centres are staged in LDS and swept by one wavefront, or by the four of a
// workgroup (sweep.h).
#include <algorithm>
#include "sweep.h"

namespace wb {

// The sphere slots' radii (they stay from state to state) and the padding
// link's empty bound.
template <int NMAX>
__device__ __forceinline__ void init_slots(const DevRobot &rb, float4 *P, int tid, int nt) {
    const int SL = (rb.L + 1) * NMAX;
    for (int i = tid; i < SL; i += nt) P[i] = make_float4(0.f, 0.f, 0.f, rb.slot_r[i]);
    if (tid == 0) P[SL + rb.L] = make_float4(0.f, 0.f, 0.f, -1e30f);
}

// The block table into LDS.
__device__ __forceinline__ void stage_blocks(const DevRobot &rb, uint32_t *tab, int tid, int nt) {
    for (int i = tid; i < rb.n_blocks_pad; i += nt) tab[i] = rb.blocks[i];
}

// One state per wavefront, four side by side: a workgroup takes `chunk`
// consecutive states (a multiple of four).  The slots' radii and the block
// table are staged once a workgroup, the centres of four states at a time by
// all its lanes, the rows in 16-byte pieces (chunks are dealt so that each
// XCD's L2 holds the rows' other pieces).  Bound by VALU issue of the sweep,
// as in the fused kernel; with the radii, the table and two integer
// divisions an element staged for every four states, and their rows fetched
// through every XCD, the humanoid's 24,576 states took 163 us.
// LDS: TS states x [(L+1)*NMAX slots | L+1 link bounds], then their row
// rings, (TAB_LDS) the block table and their lists.
// nb: states; B: row length of the sphere array (the ABI's ld >= nb).
// TS: 4, or 0 for robots of which 64 KB hold fewer than four states: a
// workgroup then takes `chunk` states (1 to 3), one a wavefront, the others
// helping to stage them.  DIRECT: rows are evaluated without a test.
template <int NMAX, bool TAB_LDS, int TS, bool DIRECT = false>
__global__ void __launch_bounds__(256) k_self_collision(DevRobot rb, int64_t nb, int64_t B, int chunk,
                                                        const float *__restrict__ sph,
                                                        float *__restrict__ max_pen,
                                                        int32_t *__restrict__ argmax,
                                                        int32_t *__restrict__ n_coll) {
    extern __shared__ float4 lds[];
    const int SL = (rb.L + 1) * NMAX;
    const int SLB = SL + rb.L + 1;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int ts = TS ? TS : chunk, rows = 256 / ts;   // rows staged at a time
    uint32_t *rings = reinterpret_cast<uint32_t *>(lds + ts * SLB), *t = rings + ts * SC_RING;
    const uint32_t *tab = TAB_LDS ? t : rb.blocks;
    uint32_t *lists = TAB_LDS ? t + rb.n_blocks_pad : t;
    if (TAB_LDS) stage_blocks(rb, t, tid, 256);
    float4 *P = lds + wave * SLB;
    if (wave < ts) init_slots<NMAX>(rb, P, lane, 64);
    const int64_t c0 = (int64_t)xcd_chunk() * chunk, c1 = min(c0 + chunk, nb);
    for (int64_t b0 = c0; b0 < c1; b0 += ts) {
        __syncthreads();   // the slots and the table are staged; the previous states are swept
        if (tid < rows * ts) {
            const int st = tid % ts;
            const int64_t b = min(b0 + st, nb - 1);
            float *slots = reinterpret_cast<float *>(lds + st * SLB);
#pragma unroll 4
            for (int row = tid / ts; row < 3 * rb.S; row += rows) {
                const int s = row / 3;
                slots[rb.sph_slot[s] * 4 + (row - 3 * s)] = sph[(int64_t)row * B + b];
            }
        }
        __syncthreads();
        const int64_t b = b0 + wave;
        if (wave >= ts || b >= c1) continue;
        float4 *Bd = P + SL;
        link_bounds<NMAX>(rb, P, Bd, lane, 64);
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        float M;
        int key;
        unsigned cnt;
        sweep_state<NMAX, true, false, false, DIRECT>(rb, tab, P, Bd, lists + wave * SWEEP_LIST, rings + wave * SC_RING, lane, 64,
                                0, M, key, cnt);
        if (lane == 0) {
            if (max_pen) max_pen[b] = M;
            if (argmax) argmax[b] = pair_index(rb, key);
            if (n_coll) n_coll[b] = (int32_t)cnt;
        }
    }
}

// One state per workgroup, its pairs split over the four wavefronts and
// reduced through LDS (sweep_state_wg): for batches too small to fill the
// chip with one state per wavefront, and for robots with many pairs.
// LDS: [(L+1)*NMAX slots | L+1 link bounds] (float4), 4 row rings, (TAB_LDS)
// the table and 4 lists of list_cap entries.
template <int NMAX, bool TAB_LDS>
__global__ void __launch_bounds__(256) k_self_collision_wg(DevRobot rb, int64_t nb, int64_t B, int list_cap,
                                                           const float *__restrict__ sph,
                                                           float *__restrict__ max_pen,
                                                           int32_t *__restrict__ argmax,
                                                           int32_t *__restrict__ n_coll) {
    extern __shared__ float4 lds[];
    const int SL = (rb.L + 1) * NMAX;
    float4 *P = lds;
    float4 *Bd = P + SL;
    uint32_t *rings = reinterpret_cast<uint32_t *>(Bd + rb.L + 1), *t = rings + 4 * SC_RING;
    const uint32_t *tab = TAB_LDS ? t : rb.blocks;
    uint32_t *lists = TAB_LDS ? t + rb.n_blocks_pad : t;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    if (TAB_LDS) stage_blocks(rb, t, tid, 256);
    init_slots<NMAX>(rb, P, tid, 256);
    for (int64_t b = blockIdx.x; b < nb; b += gridDim.x) {
        __syncthreads();   // staged; the previous state is swept
#pragma unroll 4
        for (int i = tid; i < rb.S * 3; i += 256) {
            const int s = i / 3;
            reinterpret_cast<float *>(P)[rb.sph_slot[s] * 4 + (i - 3 * s)] = sph[(int64_t)i * B + b];
        }
        __syncthreads();
        link_bounds<NMAX>(rb, P, Bd, tid, 256);
        __syncthreads();
        float M;
        int key;
        unsigned cnt;
        sweep_state_wg<NMAX>(rb, tab, P, Bd, lists + wave * list_cap, list_cap, rings, wave, lane, M, key, cnt);
        if (tid == 0) {
            if (max_pen) max_pen[b] = M;
            if (argmax) argmax[b] = pair_index(rb, key);
            if (n_coll) n_coll[b] = (int32_t)cnt;
        }
    }
}

// The shapes are in wb_internal.h.
template <int NMAX>
static hipError_t launch_sc(const DevRobot &rb, int64_t B, int64_t ld, const float *sph, float *mp, int32_t *am,
                            int32_t *nc, hipStream_t s) {
    const SweepShape w = sweep_wave_shape(rb.L, NMAX, rb.n_blocks_pad);
    // chunks of up to 32 states that leave 2,048 workgroups, or the states of one pass
    const int chunk = w.states < 4 ? w.states : (int)std::max<int64_t>(std::min<int64_t>(32, B / 2048) / 4 * 4, 4);
    const dim3 grid((unsigned)((B + chunk - 1) / chunk)), block(256);
    if (NMAX <= 16 && w.table && rb.n_blocks * NMAX <= DIRECT_ROWS)
        hipLaunchKernelGGL((k_self_collision<NMAX, true, 4, NMAX <= 16>), grid, block, w.lds, s, rb, B, ld, chunk, sph, mp, am, nc);
    else if (w.table)
        hipLaunchKernelGGL((k_self_collision<NMAX, true, 4>), grid, block, w.lds, s, rb, B, ld, chunk, sph, mp, am, nc);
    else if (w.states == 4)
        hipLaunchKernelGGL((k_self_collision<NMAX, false, 4>), grid, block, w.lds, s, rb, B, ld, chunk, sph, mp, am, nc);
    else
        hipLaunchKernelGGL((k_self_collision<NMAX, false, 0>), grid, block, w.lds, s, rb, B, ld, chunk, sph, mp, am, nc);
    return hipGetLastError();
}

template <int NMAX>
static hipError_t launch_sc_wg(const DevRobot &rb, int64_t B, int64_t ld, const float *sph, float *mp, int32_t *am,
                               int32_t *nc, hipStream_t s) {
    const SweepShape w = sweep_split_shape(rb.L, NMAX, rb.n_blocks_pad);
    const dim3 grid((unsigned)std::min<int64_t>(B, 1 << 20)), block(256);
    if (w.table)
        hipLaunchKernelGGL((k_self_collision_wg<NMAX, true>), grid, block, w.lds, s, rb, B, ld, w.list, sph, mp, am, nc);
    else
        hipLaunchKernelGGL((k_self_collision_wg<NMAX, false>), grid, block, w.lds, s, rb, B, ld, w.list, sph, mp, am, nc);
    return hipGetLastError();
}

template <int NMAX>
static hipError_t launch_sc_any(const DevRobot &rb, int64_t B, int64_t ld, const float *sph, float *mp, int32_t *am,
                                int32_t *nc, bool split, hipStream_t s) {
    return split ? launch_sc_wg<NMAX>(rb, B, ld, sph, mp, am, nc, s) : launch_sc<NMAX>(rb, B, ld, sph, mp, am, nc, s);
}

hipError_t launch_self_collision(const DevRobot &rb, int64_t B, int64_t ld, const float *spheres,
                                 float *max_pen, int32_t *argmax, int32_t *n_coll, bool split, hipStream_t s) {
    if (B == 0) return hipSuccess;
    switch (rb.nmax) {
        case 1: return launch_sc_any<1>(rb, B, ld, spheres, max_pen, argmax, n_coll, split, s);
        case 2: return launch_sc_any<2>(rb, B, ld, spheres, max_pen, argmax, n_coll, split, s);
        case 3: return launch_sc_any<3>(rb, B, ld, spheres, max_pen, argmax, n_coll, split, s);
        case 4: return launch_sc_any<4>(rb, B, ld, spheres, max_pen, argmax, n_coll, split, s);
        case 5: return launch_sc_any<5>(rb, B, ld, spheres, max_pen, argmax, n_coll, split, s);
        case 6: return launch_sc_any<6>(rb, B, ld, spheres, max_pen, argmax, n_coll, split, s);
        case 7: return launch_sc_any<7>(rb, B, ld, spheres, max_pen, argmax, n_coll, split, s);
        case 8: return launch_sc_any<8>(rb, B, ld, spheres, max_pen, argmax, n_coll, split, s);
        case 12: return launch_sc_any<12>(rb, B, ld, spheres, max_pen, argmax, n_coll, split, s);
        case 16: return launch_sc_any<16>(rb, B, ld, spheres, max_pen, argmax, n_coll, split, s);
        case 24: return launch_sc_any<24>(rb, B, ld, spheres, max_pen, argmax, n_coll, split, s);
        case 32: return launch_sc_any<32>(rb, B, ld, spheres, max_pen, argmax, n_coll, split, s);
        case 48: return launch_sc_any<48>(rb, B, ld, spheres, max_pen, argmax, n_coll, split, s);
        case 64: return launch_sc_any<64>(rb, B, ld, spheres, max_pen, argmax, n_coll, split, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace wb
