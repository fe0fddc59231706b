// The self-collision pair sweep of one state by a group of G lanes of a
// wavefront (cuRoboV2 Sec. 6.2: the "map" over pair blocks and the "reduce"
// to the most penetrating pair), shared by the standalone and fused kernels.
//
// The checked pair set is a union of dense link blocks: every allowed link
// pair (a < b) contributes all spheres of a times all spheres of b.  The
// state's sphere centres sit in LDS, padded to NMAX slots per link (empty
// slots carry radius -1e30, so they can neither be the maximum nor count as
// a collision), plus one all-empty row for padding.
//
// Broad phase (exact): each link gets a bounding sphere (centroid C_a of its
// sphere centres, reach R_a = max |c - C_a| + r), and no pair of block (a, b)
// can penetrate more than bound = R_a + R_b - |C_a - C_b|.  eps covers the
// FP32 rounding of both the bound and the pair penetrations (all computed
// from the same FP32 centres), so a block whose computed bound is below t -
// eps holds no pair whose computed penetration reaches t.
//   Pass 1 sweeps the blocks that may reach -eps, tested without a square
//   root as |C_a - C_b|^2 <= (R_a + R_b + eps)^2.  If their maximum M0 is
//   >= 0, every skipped pair penetrates less than 0 <= M0: none is the
//   maximum, ties it, or collides, and the result is that of the full sweep.
//   Otherwise (no collision) a lower bound of M -- M0, or the exact maximum
//   of the block with the largest bound when pass 1 found nothing -- sets
//   t1, and pass 2 sweeps the blocks that pass 1 skipped and whose bound is
//   >= t1 - eps (the two passes partition the blocks exactly).
// The surviving blocks of each pass are compacted into the group's LDS list
// (ballot + popcount), swept whenever it is full, and the pair loop runs over
// rows -- (block, sphere slot of the first link) against the NMAX slots of
// the second link -- so that the lanes stay dense whatever the number of
// survivors.
// Row test (the same broad phase one level down, in the per-group sweeps):
// no pair of a row penetrates more than r_A + R_b - |c_A - C_b|, sphere A of
// the first link against the second link's bounding sphere, so a row is
// evaluated only where that bound may reach the pass's threshold.  Passing
// rows are queued in an LDS ring of 2 G entries per group (ballot + popcount) and
// evaluated G at a time, so the lanes stay dense.  Pass 2 then takes every
// block whose bound reaches t1 - eps and, in it, the rows pass 1 did not
// evaluate whose row bound reaches t1 - eps: the rows of the two passes
// partition the rows of the table exactly, with the same eps argument.  The block
// table is read from LDS where the caller has staged it; it is padded to a
// multiple of 128 entries with the empty pair (L, L), whose bounding sphere
// Bd[L] has radius -1e30, so the pass-1 loop needs no range tests.  Entries
// and row codes are byte offsets: unpacking link numbers took 5 of a test's
// 28 vector instructions, and the fused kernel is bound by their issue.
//
// Reduce: the pair count is a scalar ballot popcount per pair (one state per
// wavefront) or a per-lane counter summed over the group; the maximum is a
// per-lane running max plus a group reduction.  The lowest pair index
// attaining the maximum is recovered exactly: lanes holding the maximum
// re-evaluate the row where their running max was set with the same
// arithmetic and report the lowest (s, t) whose penetration equals it; if
// any lane saw two of its rows tie the maximum, the group rescans every
// block instead.
#pragma once

#include <climits>
#include <type_traits>
#include "lanes.h"
#include "spatial.h"

namespace wb {

// Penetration depth of one sphere pair; .w is the radius.  Written with
// explicit fused multiply-adds so every evaluation rounds identically.
__device__ __forceinline__ float pair_pen(float4 A, float4 Bv) {
    const float dx = A.x - Bv.x, dy = A.y - Bv.y, dz = A.z - Bv.z;
    const float d2 = __builtin_fmaf(dx, dx, __builtin_fmaf(dy, dy, dz * dz));
    return (A.w + Bv.w) - __builtin_amdgcn_sqrtf(d2);
}

// A block table entry holds the byte offsets of its two links' bounding
// spheres, (16 a) << 16 | 16 b, so that one add each forms an address.
__device__ __forceinline__ const float4 &bound_of(const float4 *Bd, uint32_t off) {
    return *reinterpret_cast<const float4 *>(reinterpret_cast<const char *>(Bd) + off);
}
__device__ __forceinline__ int entry_a(uint32_t e) { return (int)(e >> 20); }
__device__ __forceinline__ int entry_b(uint32_t e) { return (int)((e >> 4) & 0xfffu); }

__device__ __forceinline__ float block_bound(const float4 *Bd, uint32_t e) {
    const float4 A = bound_of(Bd, e >> 16), Bv = bound_of(Bd, e & 0xffffu);
    const float dx = A.x - Bv.x, dy = A.y - Bv.y, dz = A.z - Bv.z;
    return (A.w + Bv.w) - __builtin_amdgcn_sqrtf(__builtin_fmaf(dx, dx, __builtin_fmaf(dy, dy, dz * dz)));
}

// Lowest sphere key s*S + t in row i of link pair (a, bb) whose penetration
// equals M.
template <int NMAX>
__device__ __forceinline__ int row_min_key(const DevRobot &rb, const float4 *P, int a, int bb, int i, float M) {
    if (a >= rb.L) return INT_MAX;
    const float4 A = P[a * NMAX + i];
    const int s = rb.li[a].sph_first + i, fb = rb.li[bb].sph_first;
#pragma unroll
    for (int j = 0; j < NMAX; ++j)
        if (pair_pen(A, P[bb * NMAX + j]) == M) return s * rb.S + (fb + j);
    return INT_MAX;
}

template <int NMAX>
__device__ __forceinline__ int block_min_key(const DevRobot &rb, const float4 *P, int a, int bb, float M) {
    int key = INT_MAX;
#pragma unroll
    for (int i = 0; i < NMAX; ++i) key = min(key, row_min_key<NMAX>(rb, P, a, bb, i, M));
    return key;
}

// Bounding sphere of every link's (non-empty) sphere slots, into Bd[0..L).
template <int NMAX>
__device__ __forceinline__ void link_bounds(const DevRobot &rb, const float4 *P, float4 *Bd, int glane, int G) {
    for (int a = glane; a < rb.L; a += G) {
        float cx = 0.f, cy = 0.f, cz = 0.f, n = 0.f;
#pragma unroll
        for (int i = 0; i < NMAX; ++i) {
            const float4 s = P[a * NMAX + i];
            if (s.w > -1e29f) {
                cx += s.x;
                cy += s.y;
                cz += s.z;
                n += 1.f;
            }
        }
        float R = -1e30f;
        if (n > 0.f) {
            const float inv = 1.f / n;
            cx *= inv;
            cy *= inv;
            cz *= inv;
#pragma unroll
            for (int i = 0; i < NMAX; ++i) {
                const float4 s = P[a * NMAX + i];
                if (s.w > -1e29f) {
                    const float dx = s.x - cx, dy = s.y - cy, dz = s.z - cz;
                    R = fmaxf(R, __builtin_amdgcn_sqrtf(__builtin_fmaf(dx, dx, __builtin_fmaf(dy, dy, dz * dz))) + s.w);
                }
            }
        }
        Bd[a] = make_float4(cx, cy, cz, R);
    }
}

// Pass-1 test: block (a, b) may hold a pair whose penetration reaches -eps,
// |C_a - C_b| <= R_a + R_b + eps, as one compare without a square root:
// d2 <= s |s| is false for every s < 0 (d2 >= 0), so the empty pair (L, L)
// never passes.  PADDED: the bounds' radii hold the margin already.
template <bool PADDED>
__device__ __forceinline__ bool may_reach(const float4 *Bd, uint32_t e, float eps) {
    const float4 A = bound_of(Bd, e >> 16), Bv = bound_of(Bd, e & 0xffffu);
    const float dx = A.x - Bv.x, dy = A.y - Bv.y, dz = A.z - Bv.z;
    const float s = PADDED ? A.w + Bv.w : (A.w + Bv.w) + eps;
    const float d2 = __builtin_fmaf(dx, dx, __builtin_fmaf(dy, dy, dz * dz));
    return d2 <= s * fabsf(s);
}

// Bits of the group's ballot m (its lanes' predicate, shifted down to the
// group) below this lane.
template <bool FULL>
__device__ __forceinline__ int bits_below(uint64_t m, uint64_t below) {
    if (FULL) return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
    return __popcll(m & below);
}

// Appends to the list of nl entries those of 2 G blocks (e0 and e1 of each
// lane) that pass the pass's test; returns the new length.  PASS2: every
// block with bound >= lo (the row sweep filters the rows itself), else the
// pass-1 test.
template <bool PASS2, bool FULL, bool PADDED>
__device__ __forceinline__ int append_blocks(uint32_t e0, uint32_t e1, const float4 *Bd, uint32_t *list, int nl,
                                             float eps, float lo, int glane, int G, int gshift, uint64_t gmask) {
    const uint64_t below = (1ull << glane) - 1ull;
    const bool s0 = PASS2 ? block_bound(Bd, e0) >= lo : may_reach<PADDED>(Bd, e0, eps);
    const bool s1 = PASS2 ? block_bound(Bd, e1) >= lo : may_reach<PADDED>(Bd, e1, eps);
    const uint64_t m0 = FULL ? __ballot(s0) : (__ballot(s0) >> gshift) & gmask;
    const uint64_t m1 = FULL ? __ballot(s1) : (__ballot(s1) >> gshift) & gmask;
    const int n0 = nl + __popcll(m0);
    if (s0) list[nl + bits_below<FULL>(m0, below)] = e0;
    if (s1) list[n0 + bits_below<FULL>(m1, below)] = e1;
    return n0 + __popcll(m1);
}

// The pass-1 test of every link pair of a robot of at most 64 links on the
// matrix cores: with n = |C|^2 - R^2 - tol / 2 the test |C_a - C_b| <= R_a +
// R_b reads
//   n_a + n_b - 2 (C_a . C_b + R_a R_b) <= 0,
// a product of the rows [x y z R n 1] and the columns [-2x -2y -2z -2R 1 n]:
// three 32x32x2 FP32 products (K = 6) for each of the tiles (links 0-31,
// 0-31), (0-31, 32-63) and (32-63, 32-63).  tol (rb.broad_tol, 1e-5 of the
// squared reach of any state) exceeds the rounding of this form and of the
// direct test's, so every block that the direct test passes has its sign bit
// set here; the few more that do are dropped by the row test.  A lane gathers
// the signs of its 48 results in two words, masks the checked pairs and
// appends its survivors behind those of the lanes below.  The direct test
// costs 25 vector instructions for 64 blocks, 450 for a humanoid's 1,128;
// this takes about 220 and the idle matrix cores.
// Taken from BROAD_MATRIX_FROM blocks on.
// Returns the number of survivors; the list holds them if they are at most
// cap.  Every lane of the wavefront calls this.
typedef float floatx16 __attribute__((ext_vector_type(16)));
__device__ __forceinline__ int broad_phase(const DevRobot &rb, const float4 *Bd, uint32_t *list, int cap, int lane) {
    const bool lo = lane < 32;
    const float *f = reinterpret_cast<const float *>(Bd);
    const int l0 = min(lane & 31, rb.L) * 4 + (lo ? 0 : 1), l1 = min((lane & 31) + 32, rb.L) * 4 + (lo ? 0 : 1);
    // component 2 s + (lane >= 32) of link 32 h + lane % 32
    const float a00 = f[l0], a01 = f[l0 + 2], a10 = f[l1], a11 = f[l1 + 2];
    const float4 c = Bd[min(lane, rb.L)];
    const float n = __builtin_fmaf(c.x, c.x, __builtin_fmaf(c.y, c.y, c.z * c.z)) - __builtin_fmaf(c.w, c.w, 0.5f * rb.broad_tol);
    unsigned u, v;
    swap32(__builtin_bit_cast(unsigned, n), u, v);   // the lower half's n in every lane, then the upper's
    const float nl = __builtin_bit_cast(float, u), nu = __builtin_bit_cast(float, v);
    const float a02 = lo ? nl : 1.f, a12 = lo ? nu : 1.f, b02 = lo ? 1.f : nl, b12 = lo ? 1.f : nu;
    const float b00 = -2.f * a00, b01 = -2.f * a01, b10 = -2.f * a10, b11 = -2.f * a11;
    auto tile = [](float p0, float p1, float p2, float q0, float q1, float q2) {
        floatx16 d = {};
        d = __builtin_amdgcn_mfma_f32_32x32x2f32(p0, q0, d, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_32x32x2f32(p1, q1, d, 0, 0, 0);
        return __builtin_amdgcn_mfma_f32_32x32x2f32(p2, q2, d, 0, 0, 0);
    };
    // result r of a lane is row 8 (r / 4) + 4 (lane / 32) + r % 4, column lane % 32
    auto signs = [](uint32_t w, const floatx16 &d) {
#pragma unroll
        for (int r = 15; r >= 0; --r) {
            const float x = d[r];
            w = __builtin_amdgcn_alignbit(w, __builtin_bit_cast(uint32_t, x), 31);
        }
        return w;
    };
    uint32_t w0 = signs(0u, tile(a00, a01, a02, b10, b11, b12));
    w0 = signs(w0, tile(a00, a01, a02, b00, b01, b02)) & rb.allow[lane];
    uint32_t w1 = signs(0u, tile(a10, a11, a12, b10, b11, b12)) & rb.allow[64 + lane];
    const int mine = __popc(w0) + __popc(w1);
    int at = mine;   // inclusive prefix sum over the wavefront
    at += dpp_i<DPP_ROW_SHR + 1>(at);
    at += dpp_i<DPP_ROW_SHR + 2>(at);
    at += dpp_i<DPP_ROW_SHR + 4>(at);
    at += dpp_i<DPP_ROW_SHR + 8>(at);
    at += __builtin_amdgcn_update_dpp(0, at, DPP_ROW_BCAST15, 0xa, 0xf, false);
    at += __builtin_amdgcn_update_dpp(0, at, DPP_ROW_BCAST31, 0xc, 0xf, false);
    const int total = __builtin_amdgcn_readlane(at, 63);
    if (total > cap) return total;
    uint32_t *out = list + (at - mine);
    const uint32_t base = ((uint32_t)(lane >> 5) << 22) | (uint32_t)(lane & 31) << 4;
    while (w0 | w1) {
        const bool first = w0 != 0;
        const uint32_t w = first ? w0 : w1, q = (uint32_t)__builtin_ctz(w), rest = w & (w - 1);
        // row 8 (r / 4) + r % 4 of the tile; bit 4 of q: the second tile's columns
        const uint32_t e = base + (((q & 3u) | (q & 12u) << 1) << 20) + ((q & 16u) << 5);
        *out++ = first ? e : e + ((32u << 20) | (32u << 4));
        w0 = first ? rest : 0u;
        w1 = first ? w1 : rest;
    }
    return total;
}

// Row test: sphere slot A against link bound Bb may hold a pair reaching
// -eps (squared, as may_reach; an empty slot never passes), and the row
// bound itself.
template <bool PADDED>
__device__ __forceinline__ bool row_may_reach(float4 A, float4 Bb, float eps) {
    const float dx = A.x - Bb.x, dy = A.y - Bb.y, dz = A.z - Bb.z;
    const float s = PADDED ? A.w + Bb.w : (A.w + Bb.w) + eps;
    const float d2 = __builtin_fmaf(dx, dx, __builtin_fmaf(dy, dy, dz * dz));
    return d2 <= s * fabsf(s);
}
__device__ __forceinline__ float row_bound(float4 A, float4 Bb) {
    const float dx = A.x - Bb.x, dy = A.y - Bb.y, dz = A.z - Bb.z;
    return (A.w + Bb.w) - __builtin_amdgcn_sqrtf(__builtin_fmaf(dx, dx, __builtin_fmaf(dy, dy, dz * dz)));
}

constexpr uint32_t NO_ROW = ~0u;           // no row code (offsets are multiples of 16)

// Evaluates the row that a code names -- the byte offset of slot A << 16 | that
// of the second link's first slot -- in the calling lanes; best_code keeps the
// code of the row that set the running max.  BALLOT: cnt is the wavefront's
// count, held by the lanes that call, else the lane's.
template <int NMAX, bool BALLOT>
__device__ __forceinline__ void eval_row(const float4 *P, uint32_t code, float &best, uint32_t &best_code, bool &tie,
                                         unsigned &cnt) {
    const float4 A = bound_of(P, code >> 16);
    const float4 *Bp = &bound_of(P, code & 0xffffu);
    float m = -INFINITY;
#pragma unroll
    for (int k = 0; k < NMAX; ++k) {
        const float pen = pair_pen(A, Bp[k]);
        m = fmaxf(m, pen);
        if (BALLOT) cnt += (unsigned)__popcll(__ballot(pen > 0.0f));
        else cnt += pen > 0.0f ? 1u : 0u;
    }
    if (m > best) {
        best = m;
        best_code = code;
        tie = false;
    } else if (m == best) {
        tie = true;
    }
}

// Evaluates the n queued rows at ring[head, head + n) (mod 2 G), one per lane.
template <int NMAX, bool FULL>
__device__ __forceinline__ void eval_rows(const float4 *P, const uint32_t *ring, int head, int n, int glane, int G,
                                          float &best, uint32_t &best_code, bool &tie, unsigned &cnt) {
    if (glane < n) eval_row<NMAX, FULL>(P, ring[(head + glane) & (2 * G - 1)], best, best_code, tie, cnt);
}

// Every row of the blocks list[0, nl), by a wavefront (PASS2: of those that
// pass 1 left out), for robots of at most DIRECT_ROWS rows.
template <int NMAX, bool PASS2>
__device__ __forceinline__ void sweep_rows_direct(const float4 *P, const float4 *Bd, const uint32_t *list, int nl,
                                                  float eps, int lane, float &best, uint32_t &best_code, bool &tie,
                                                  unsigned &cnt) {
    for (int j = lane; j < nl * NMAX; j += 64) {
        const int i = j / NMAX, row = j - i * NMAX;
        const uint32_t e = list[i];
        if (PASS2 && may_reach<false>(Bd, e, eps)) continue;
        eval_row<NMAX, false>(P, (((e >> 16) * NMAX + row * 16) << 16) | ((e & 0xffffu) * NMAX), best, best_code, tie, cnt);
    }
}

// The rows of the blocks list[0, nl) that pass the row test (pass 1: may
// reach -eps; PASS2: row bound >= lo and not evaluated by pass 1), queued in
// the ring and evaluated G at a time: running maximum, its row code, ties,
// count.  Lane i takes rows i, i + G, ...: its list entry and slot advance by
// the quotient and remainder of G by NMAX.
template <int NMAX, bool FULL, bool PASS2, bool PADDED>
__device__ __forceinline__ void sweep_rows_culled(const float4 *P, const float4 *Bd, const uint32_t *list, int nl,
                                                  uint32_t *ring, float eps, float lo, int glane, int G, int gshift, uint64_t gmask, float &best,
                                                  uint32_t &best_code, bool &tie, unsigned &cnt) {
    const uint64_t below = (1ull << glane) - 1ull;
    const int items = nl * NMAX, dq = G / NMAX, dr = G - dq * NMAX;
    int head = 0, pending = 0;   // the same in every lane of the group
    int i = glane / NMAX, row = glane - i * NMAX;
    for (int j0 = 0; j0 < items; j0 += G) {
        bool pass = false;
        uint32_t code = 0;
        if (i < nl) {
            const uint32_t e = list[i];
            const uint32_t a = (e >> 16) * NMAX + row * 16;
            const float4 A = bound_of(P, a), Bb = bound_of(Bd, e & 0xffffu);
            const bool may = row_may_reach<PADDED>(A, Bb, eps);
            pass = PASS2 ? (row_bound(A, Bb) >= lo && !(may && may_reach<PADDED>(Bd, e, eps))) : may;
            code = (a << 16) | ((e & 0xffffu) * NMAX);
        }
        i += dq;
        row += dr;
        if (row >= NMAX) {
            row -= NMAX;
            ++i;
        }
        const uint64_t m = FULL ? __ballot(pass) : (__ballot(pass) >> gshift) & gmask;
        if (pass) ring[(head + pending + bits_below<FULL>(m, below)) & (2 * G - 1)] = code;
        pending += __popcll(m);
        if (pending >= G) {
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
            eval_rows<NMAX, FULL>(P, ring, head, G, glane, G, best, best_code, tie, cnt);
            head = (head + G) & (2 * G - 1);
            pending -= G;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (pending > 0) eval_rows<NMAX, FULL>(P, ring, head, pending, glane, G, best, best_code, tie, cnt);
}

// Lowest key of the row that best_code names.
template <int NMAX>
__device__ __forceinline__ int code_min_key(const DevRobot &rb, const float4 *P, uint32_t code, float M) {
    const int sa = (int)(code >> 20), a = sa / NMAX;
    return row_min_key<NMAX>(rb, P, a, (int)((code & 0xffffu) >> 4) / NMAX, sa - a * NMAX, M);
}

// Sweep one state.  tab: the robot's block table (or its LDS copy); P: the
// state's (L+1)*NMAX sphere slots; Bd: its link bounding spheres; list:
// sweep_list entries of LDS scratch for this group, swept whenever it is
// full.
// Every lane of the group returns the maximum penetration M, the sphere key
// s*S + t of the lowest pair attaining it (INT_MAX if none) and the number
// of pairs with positive penetration.  FULL: G == 64.  ring: sweep_ring
// words of LDS scratch for this group.  PADDED: the bounds' radii hold the rounding
// margin of any state already, else it is formed from the state's extent.
// MATRIX (with PADDED, at most 64 links): pass 1 on the matrix cores where
// the robot has blocks enough.  DIRECT (with FULL, not PADDED): no row tests.
template <int NMAX, bool FULL, bool PADDED, bool MATRIX, bool DIRECT = false>
__device__ __forceinline__ void sweep_state(const DevRobot &rb, const uint32_t *tab, const float4 *P,
                                            const float4 *Bd, uint32_t *list, uint32_t *ring, int glane, int G,
                                            int grp, float &M_out, int &key_out, unsigned &cnt_out) {
    const int n = rb.n_blocks;
    const int nb = (n + 2 * G - 1) / (2 * G) * (2 * G);   // <= n_blocks_pad, a multiple of 128
    const int cap = min(nb, SWEEP_LIST);                  // sweep_list
    const uint64_t gmask = FULL ? ~0ull : ((1ull << G) - 1ull);
    const int gshift = FULL ? 0 : grp * G;
    float eps = 0.f;
    if (!PADDED) {   // extent of the robot in this state, for the rounding margin
        float ext = 0.f;
        for (int a = glane; a < rb.L; a += G) {
            const float4 c = Bd[a];
            if (c.w > -1e29f)
                ext = fmaxf(ext, __builtin_amdgcn_sqrtf(__builtin_fmaf(c.x, c.x, __builtin_fmaf(c.y, c.y, c.z * c.z))) + c.w);
        }
        eps = 4e-6f * (1.f + group_reduce_max(ext, G));
    }

    float best = -INFINITY;
    uint32_t best_code = NO_ROW;
    bool tie = false;
    unsigned cnt = 0;
    auto sweep_blocks = [&](auto pass2, float lo) {
        constexpr bool PASS2 = decltype(pass2)::value;
        int nl = 0;
        // the next entries are fetched beside the test of these: a table read
        // through the L1 costs a wavefront alone on its SIMD its whole latency
        // (a plan of 3,165 states of four trees 30.1 -> 29.4 us)
        uint32_t n0 = nb > 0 ? tab[glane] : 0u, n1 = nb > 0 ? tab[glane + G] : 0u;
        for (int k = 0; k < nb; k += 2 * G) {
            const uint32_t e0 = n0, e1 = n1;
            const int next = min(k + 2 * G, nb - 2 * G) + glane;
            n0 = tab[next];
            n1 = tab[next + G];
            nl = append_blocks<PASS2, FULL, PADDED>(e0, e1, Bd, list, nl, eps, lo, glane, G, gshift, gmask);
            const bool full = nl + 2 * G > cap;
            if (k + 2 * G >= nb || (FULL ? full : __ballot(full) != 0)) {
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                __builtin_amdgcn_wave_barrier();
                if (DIRECT) sweep_rows_direct<NMAX, PASS2>(P, Bd, list, nl, eps, glane, best, best_code, tie, cnt);
                else
                    sweep_rows_culled<NMAX, FULL, PASS2, PADDED>(P, Bd, list, nl, ring, eps, lo, glane, G, gshift,
                                                                 gmask, best, best_code, tie, cnt);
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                __builtin_amdgcn_wave_barrier();
                nl = 0;
            }
        }
    };
    // pass 1: blocks that may hold a collision
    int found = -1;
    if (MATRIX && FULL && n >= BROAD_MATRIX_FROM) {
        found = broad_phase(rb, Bd, list, cap, glane);
        if (found > cap) found = -1;
    }
    if (found < 0) sweep_blocks(std::false_type{}, 0.f);
    else {
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        sweep_rows_culled<NMAX, FULL, false, PADDED>(P, Bd, list, found, ring, eps, 0.f, glane, G, gshift, gmask, best,
                                                     best_code, tie, cnt);
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    float M = group_reduce_max(best, G);
    if (!(M >= 0.f) && n > 0) {
        // pass 2 (no collision): a lower bound of M, then the skipped blocks that can reach it
        float lb = M;
        if (lb == -INFINITY) {
            float bmax = -INFINITY;
            int bblk = INT_MAX;
            for (int k = glane; k < n; k += G) {
                const float d = block_bound(Bd, tab[k]);
                if (d > bmax) {
                    bmax = d;
                    bblk = k;
                }
            }
            const float gbmax = group_reduce_max(bmax, G);
            const int cand = group_reduce_min(bmax == gbmax ? bblk : INT_MAX, G);
            float seed = -INFINITY;
            if (cand != INT_MAX) {   // no candidate only when every bound is NaN
                const uint32_t e = tab[cand];
                const int a = entry_a(e), bb = entry_b(e);
                for (int j = glane; j < NMAX * NMAX; j += G) {
                    const int i = j / NMAX, k = j - i * NMAX;
                    seed = fmaxf(seed, pair_pen(P[a * NMAX + i], P[bb * NMAX + k]));
                }
            }
            lb = group_reduce_max(seed, G);
        }
        const float theta1 = lb - eps;
        sweep_blocks(std::true_type{}, theta1);
        M = group_reduce_max(best, G);
    }
    int key = INT_MAX;
    const bool holder = best == M && M > -INFINITY && best_code != NO_ROW;
    const bool rescan = group_reduce_min((holder && tie) ? 0 : 1, G) == 0;
    if (rescan) {
        for (int blk = glane; blk < n; blk += G) {
            const uint32_t e = tab[blk];
            key = min(key, block_min_key<NMAX>(rb, P, entry_a(e), entry_b(e), M));
        }
    } else if (holder) {
        key = code_min_key<NMAX>(rb, P, best_code, M);
    }
    M_out = M;
    key_out = group_reduce_min(key, G);
    cnt_out = FULL && !DIRECT ? cnt : group_reduce_sum_u(cnt, G);
}

// Sweep one state with the four wavefronts of a workgroup (the map of the
// paper's two-stage self-collision split over wavefronts, then a second
// reduce through LDS): the block table's 128-entry chunks are dealt
// round-robin to the wavefronts (chunk c to wavefront c % 4); each compacts
// its chunks into its list (list_cap entries) and sweeps their rows as
// sweep_state does with G = 64, and the workgroup combines the wavefronts'
// maxima, counts and argmax keys.  Pass 2, the seed block and the tie rescan
// follow the single-wavefront rules with workgroup-wide values, so the result
// is the full sweep's.  rings: the four wavefronts' row rings; the values to
// reduce pass through the first word of each, which its wavefront alone uses
// between the barriers.  Every thread of the workgroup must call this (it
// synchronizes the workgroup).
__device__ __forceinline__ float wg_max4(float v, uint32_t *rings, int wave, int lane) {
    float *red = reinterpret_cast<float *>(rings);
    if (lane == 0) red[wave * SC_RING] = v;
    __syncthreads();
    const float m = fmaxf(fmaxf(red[0], red[SC_RING]), fmaxf(red[2 * SC_RING], red[3 * SC_RING]));
    __syncthreads();
    return m;
}
__device__ __forceinline__ int wg_min4(int v, uint32_t *rings, int wave, int lane) {
    int *red = reinterpret_cast<int *>(rings);
    if (lane == 0) red[wave * SC_RING] = v;
    __syncthreads();
    const int m = min(min(red[0], red[SC_RING]), min(red[2 * SC_RING], red[3 * SC_RING]));
    __syncthreads();
    return m;
}

template <int NMAX>
__device__ __forceinline__ void sweep_state_wg(const DevRobot &rb, const uint32_t *tab, const float4 *P, const float4 *Bd,
                                               uint32_t *list, int list_cap, uint32_t *rings, int wave, int lane,
                                               float &M_out, int &key_out, unsigned &cnt_out) {
    const int n = rb.n_blocks;
    const int nb = (n + 127) / 128 * 128;   // <= n_blocks_pad
    uint32_t *ring = rings + wave * SC_RING;
    float ext = 0.f;
    for (int a = lane; a < rb.L; a += 64) {
        const float4 c = Bd[a];
        if (c.w > -1e29f)
            ext = fmaxf(ext, __builtin_amdgcn_sqrtf(__builtin_fmaf(c.x, c.x, __builtin_fmaf(c.y, c.y, c.z * c.z))) + c.w);
    }
    const float eps = 4e-6f * (1.f + group_reduce_max(ext, 64));

    float best = -INFINITY;
    uint32_t best_code = NO_ROW;
    bool tie = false;
    unsigned cnt = 0;
    // the wavefront's chunks through its list, the rows swept when it is full
    auto sweep_chunks = [&](auto pass2, float lo) {
        constexpr bool PASS2 = decltype(pass2)::value;
        int nl = 0;
        for (int k = wave * 128; k < nb; k += 4 * 128) {
            nl = append_blocks<PASS2, true, false>(tab[k + lane], tab[k + lane + 64], Bd, list, nl, eps, lo, lane, 64, 0, ~0ull);
            if (k + 4 * 128 >= nb || nl + 128 > list_cap) {
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                __builtin_amdgcn_wave_barrier();
                sweep_rows_culled<NMAX, true, PASS2, false>(P, Bd, list, nl, ring, eps, lo, lane, 64, 0, ~0ull, best,
                                                            best_code, tie, cnt);
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                __builtin_amdgcn_wave_barrier();
                nl = 0;
            }
        }
    };
    sweep_chunks(std::false_type{}, 0.f);
    float M = wg_max4(group_reduce_max(best, 64), rings, wave, lane);
    if (!(M >= 0.f) && n > 0) {
        float lb = M;
        if (lb == -INFINITY) {
            // the block with the largest bound over the whole table (lowest index among equals)
            float bmax = -INFINITY;
            int bblk = INT_MAX;
            for (int c0 = wave * 128; c0 < nb; c0 += 4 * 128)
                for (int k = c0 + lane; k < min(c0 + 128, n); k += 64) {
                    const float d = block_bound(Bd, tab[k]);
                    if (d > bmax) {
                        bmax = d;
                        bblk = k;
                    }
                }
            const float gbmax = wg_max4(group_reduce_max(bmax, 64), rings, wave, lane);
            const int cand = wg_min4(group_reduce_min(bmax == gbmax ? bblk : INT_MAX, 64), rings, wave, lane);
            float seed = -INFINITY;
            if (cand != INT_MAX) {
                const uint32_t e = tab[cand];
                const int a = entry_a(e), bb = entry_b(e);
                for (int j = lane; j < NMAX * NMAX; j += 64) {
                    const int i = j / NMAX, k = j - i * NMAX;
                    seed = fmaxf(seed, pair_pen(P[a * NMAX + i], P[bb * NMAX + k]));
                }
            }
            lb = group_reduce_max(seed, 64);   // the same in every wavefront
        }
        const float theta1 = lb - eps;
        sweep_chunks(std::true_type{}, theta1);
        M = wg_max4(group_reduce_max(best, 64), rings, wave, lane);
    }
    int key = INT_MAX;
    const bool holder = best == M && M > -INFINITY && best_code != NO_ROW;
    const bool rescan = wg_min4(group_reduce_min((holder && tie) ? 0 : 1, 64), rings, wave, lane) == 0;
    if (rescan) {
        for (int c0 = wave * 128; c0 < nb; c0 += 4 * 128)
            for (int blk = c0 + lane; blk < min(c0 + 128, n); blk += 64) {
                const uint32_t e = tab[blk];
                key = min(key, block_min_key<NMAX>(rb, P, entry_a(e), entry_b(e), M));
            }
    } else if (holder) {
        key = code_min_key<NMAX>(rb, P, best_code, M);
    }
    M_out = M;
    key_out = wg_min4(group_reduce_min(key, 64), rings, wave, lane);
    // counts: the wavefronts' (uniform) counts summed in a fixed order
    if (lane == 0) ring[0] = cnt;
    __syncthreads();
    cnt_out = rings[0] + rings[SC_RING] + rings[2 * SC_RING] + rings[3 * SC_RING];
    __syncthreads();
}

// Pair index (lexicographic in (s, t)) of a sphere key s*S + t.
__device__ __forceinline__ int32_t pair_index(const DevRobot &rb, int key) {
    if (key == INT_MAX) return -1;
    const int s = (int)((unsigned)key / (unsigned)rb.S), t = key - s * rb.S;
    const int a = rb.sph_link[s], bt = rb.sph_link[t];
    return rb.pair_off[s] + rb.pair_cnt[a * rb.L + bt] + (t - rb.li[bt].sph_first);
}

}  // namespace wb
