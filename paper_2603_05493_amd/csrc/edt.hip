// Exact Euclidean distance transform of a site grid (cuRoboV2 Sec. 5,
// "Stage 2: Distance Propagation"): the nearest site of every voxel by
// three separable axis passes, as the PBA+ decomposition of the paper, each
// line's owners found by monotone search instead of an envelope stack.
// Integer arithmetic throughout, so the result is exact.
//
// Grid [nz][ny][nx], x fastest.  A site is stored packed as
// x | y << 10 | z << 20 (coordinates below 1024), NONE (-1) when there is
// none.  The axes are taken in the order x, y, z so that every pass keeps
// its lanes along x, the contiguous axis: loads and stores are coalesced
// and no transpose is needed.  Three launches, fixed for a grid size
// (graph-capturable, no atomics):
//   1. along x, one wavefront per row (y, z): the nearest site of the row,
//      from a forward and a backward flood, each an inclusive max-scan over
//      the wavefront (DPP; the backward one toward lower lanes) carried
//      across chunks -> A (rows of a multiple of 4 voxels: 4 voxels per
//      lane, in registers, one read and one write of the row);
//   2. along y, a workgroup per tile of lines (x0 .. x0+TL-1, z) held in
//      LDS: every voxel's nearest of the row sites, by (y - y')^2 + (x - x*)^2
//      -> B;
//   3. along z, the same on tiles (x0 .. x0+TL-1, y) with the plane sites and
//      (z - z')^2 + (x - x*)^2 + (y - y*)^2 -> the nearest site and
//      voxel_size * sqrt(d2).
// Each pass reads its input grid once and writes its output once.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "edt.h"

namespace wb {
namespace {

constexpr int32_t EDT_NONE = -1;
constexpr int EDT_BIG = 1 << 20; // above any coordinate

__device__ __forceinline__ int32_t pack(int x, int y, int z) { return x | (y << 10) | (z << 20); }
__device__ __forceinline__ int cx(int32_t c) { return c & 1023; }
__device__ __forceinline__ int cy(int32_t c) { return (c >> 10) & 1023; }
__device__ __forceinline__ int cz(int32_t c) { return c >> 20; }

// Inclusive max-scan over the 64 lanes of a wavefront, for values >= 0 (0 is
// the identity): row_shr 1, 2, 4, 8 inside each row of 16, then row_bcast15
// and row_bcast31 carry the row maxima upward.
template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ int dpp_up(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, ROW_MASK, 0xf, false);
}
__device__ __forceinline__ int wave_max_scan(int v) {
    v = max(v, dpp_up<0x111>(v));
    v = max(v, dpp_up<0x112>(v));
    v = max(v, dpp_up<0x114>(v));
    v = max(v, dpp_up<0x118>(v));
    v = max(v, dpp_up<0x142, 0xa>(v));
    v = max(v, dpp_up<0x143, 0xc>(v));
    return v;
}
// Inclusive max-scan toward lower lanes (lane i: max over lanes >= i):
// row_shl 1, 2, 4, 8 inside each row, then the maxima of the rows above,
// read from the first lane of each row.
__device__ __forceinline__ int wave_max_suffix_scan(int v, int lane) {
    v = max(v, dpp_up<0x101>(v));
    v = max(v, dpp_up<0x102>(v));
    v = max(v, dpp_up<0x104>(v));
    v = max(v, dpp_up<0x108>(v));
    const int r1 = __builtin_amdgcn_readlane(v, 16), r2 = __builtin_amdgcn_readlane(v, 32),
              r3 = __builtin_amdgcn_readlane(v, 48);
    const int row = lane >> 4;
    if (row < 3) v = max(v, r3);
    if (row < 2) v = max(v, r2);
    if (row < 1) v = max(v, r1);
    return v;
}

// ---- pass 1: nearest site along x, one wavefront per row (y, z)
__global__ void __launch_bounds__(256) k_edt_x(const uint8_t *__restrict__ sites, int32_t *__restrict__ A, int nx,
                                               int ny, int nz) {
    const int64_t w = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 6;
    const int lane = threadIdx.x & 63;
    if (w >= (int64_t)ny * nz) return;   // uniform over the wavefront
    const int y = (int)(w % ny), z = (int)(w / ny);
    const int64_t base = w * nx;
    // forward: 1 + the last site at or before x (0: none)
    int carry = 0;
    for (int x0 = 0; x0 < nx; x0 += 64) {
        const int x = x0 + lane;
        const int s = x < nx && sites[base + x] ? x + 1 : 0;
        const int v = max(wave_max_scan(s), carry);
        carry = __builtin_amdgcn_readlane(v, 63);
        if (x < nx) A[base + x] = v - 1;
    }
    // backward: BIG - the next site at or after x (0: none); each lane reads
    // back only what it stored itself
    carry = 0;
    for (int x0 = ((nx - 1) >> 6) << 6; x0 >= 0; x0 -= 64) {
        const int x = x0 + lane;
        const int s = x < nx && sites[base + x] ? EDT_BIG - x : 0;
        const int v = max(wave_max_suffix_scan(s, lane), carry);
        carry = __builtin_amdgcn_readlane(v, 0);
        if (x < nx) {
            const int prev = A[base + x], next = v > 0 ? EDT_BIG - v : EDT_NONE;
            const int best = prev < 0 ? next : (next < 0 ? prev : (x - prev <= next - x ? prev : next));
            A[base + x] = best < 0 ? EDT_NONE : pack(best, y, z);
        }
    }
}

// Pass 1 for rows whose length is a multiple of 4 (up to 1024): lane i of
// the row's wavefront holds voxels 4i .. 4i + 3 of each 256-voxel chunk in
// registers, read as one 4-byte word per chunk.  Both floods run on those
// registers (a 4-voxel scan inside the lane, a wavefront scan of the lane
// totals, a carry across chunks), and each chunk's result leaves as one
// 16-byte store per lane: the site row is read once and A written once.
template <int NC>
__global__ void __launch_bounds__(256) k_edt_x4(const uint8_t *__restrict__ sites, int32_t *__restrict__ A, int nx,
                                                int ny, int nz) {
    const int64_t w = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 6;
    const int lane = threadIdx.x & 63;
    if (w >= (int64_t)ny * nz) return;   // uniform over the wavefront
    const int y = (int)(w % ny), z = (int)(w / ny);
    const int n4 = nx >> 2;
    const uint32_t *row = reinterpret_cast<const uint32_t *>(sites + w * nx);
    int4 *out = reinterpret_cast<int4 *>(A + w * nx);
    uint32_t sb[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int i = c * 64 + lane;
        sb[c] = i < n4 ? row[i] : 0u;
    }
    // forward: 1 + the last site at or before x (0: none)
    int prev[NC][4];
    int carry = 0;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int x0 = (c * 64 + lane) * 4;
        int v = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            v = (sb[c] >> (8 * j)) & 0xffu ? x0 + j + 1 : v;
            prev[c][j] = v;
        }
        const int incl = wave_max_scan(v);
        const int up = __shfl_up(incl, 1, 64);
        const int excl = max(lane > 0 ? up : 0, carry);
#pragma unroll
        for (int j = 0; j < 4; ++j) prev[c][j] = max(prev[c][j], excl);
        carry = max(carry, __builtin_amdgcn_readlane(incl, 63));
    }
    // backward: BIG - the next site at or after x (0: none), then the nearer
    carry = 0;
#pragma unroll
    for (int c = NC - 1; c >= 0; --c) {
        const int x0 = (c * 64 + lane) * 4;
        int nxt[4];
        int v = 0;
#pragma unroll
        for (int j = 3; j >= 0; --j) {
            v = (sb[c] >> (8 * j)) & 0xffu ? EDT_BIG - (x0 + j) : v;
            nxt[j] = v;
        }
        const int incl = wave_max_suffix_scan(v, lane);
        const int down = __shfl_down(incl, 1, 64);
        const int excl = max(lane < 63 ? down : 0, carry);
        carry = max(carry, __builtin_amdgcn_readlane(incl, 0));
        int r[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int x = x0 + j;
            const int pv = prev[c][j] - 1;
            const int nv = max(nxt[j], excl);
            const int nx_ = nv > 0 ? EDT_BIG - nv : EDT_NONE;
            const int best = pv < 0 ? nx_ : (nx_ < 0 ? pv : (x - pv <= nx_ - x ? pv : nx_));
            r[j] = best < 0 ? EDT_NONE : pack(best, y, z);
        }
        const int i = c * 64 + lane;
        if (i < n4) out[i] = make_int4(r[0], r[1], r[2], r[3]);
    }
}

// Squared offset across the line of a candidate c: AX == 1 runs along y (a
// line (x, z); the candidate is the row's nearest site (x*, y', z)), AX == 2
// along z (a line (x, y); the plane's nearest site (x*, y*, z')).
template <int AX>
__device__ __forceinline__ int height(int32_t c, int qx, int qy) {
    const int dx = qx - cx(c);
    if (AX == 1) return dx * dx;
    const int dy = qy - cy(c);
    return dx * dx + dy * dy;
}

// ---- passes 2 and 3: one workgroup per tile of TL lines (consecutive x)
// at a fixed z (AX == 1) or y (AX == 2).  The owner of position s is the
// candidate p with the least (s - p)^2 + h_p, the last one where several
// tie.  Both rules are one unsigned comparison of keys
//   ((s - p)^2 + h_p) << 10 | (1023 - p)
// (values below 2^22: h_p <= 2 * 1023^2, and an empty position's EMPTY_H
// exceeds every real value, so it owns only where the line is empty), so LDS
// holds h_p << 10 | (1023 - p) and a candidate costs one 24-bit multiply-add
// and one minimum.  Owners never decrease along the line, so they are found
// by halving: the owner of a position lies between those of its solved
// neighbours.  A stretch of candidates between them is searched by blocks of
// eight, each skipped where its least key at its least distance exceeds the
// best so far: a jump over candidates that own nothing costs one bound per
// eight of them.  The coarse levels, whose positions end the threads' 16-
// position segments, synchronize the workgroup; inside its segment (l, j)
// each thread goes on alone.  What bounds it is the issue of these searches
// (about 230 VALU instructions a solved position for 64 lanes of different
// jumps, 24.0 M and 37.5 M a pass; without the block bounds a wavefront of
// the room's y pass takes 720 candidate steps a segment, 2,900 at worst,
// with them 41 blocks, 79 at worst).  Room of 256 x 256 x 128: y pass 70 us,
// z pass 74 us; the form before, an envelope stack per band and a merge
// whose slowest tile set the time, 85 and 78 us.  The owners' packed sites
// are read again from the input grid, rows the workgroup has just read.
constexpr uint32_t EMPTY_H = 3 * 1023 * 1023 + 1;
constexpr int EDT_BLK = 8;   // candidates under one bound

// Tiles of few candidates.  A row (AX == 1) or a plane holds a candidate for
// every line of the tile or for none; with at most few_limit(n) of them every
// position takes the least of all, at one multiply-add and one minimum each:
// about 0.6 us a candidate on 256 x 256 x 128 voxels over the 15 us of reading
// and writing, where the search, whose intervals the empty positions widen,
// takes 45 to 77.  y and z pass there, by the search / so: no site 48, 45 / 16,
// 20 us; one voxel in 10^5 a site 57, 68 / 17, 51; in 10^4 66, 74 / 21, 74; in
// 10^3 77, 72 / 51, 72.
constexpr int EDT_FEW = 88, EDT_SEG = 16;
__host__ __device__ constexpr int few_limit(int n) { return n * 7 / 16 < EDT_FEW ? n * 7 / 16 : EDT_FEW; }

// LDS of a line: its keys, padded to whole groups of four blocks and four
// words apart in banks, one least key per block, and the owners.
__host__ __device__ constexpr int edt_padded(int n) { return (n + 31) & ~31; }
__host__ __device__ constexpr int edt_key_pitch(int n) { return edt_padded(n) + 4; }
__host__ __device__ constexpr int edt_min_pitch(int n) { return edt_padded(n) / EDT_BLK + 4; }

template <int AX, int TL, int NT, typename Own>
__global__ void __launch_bounds__(NT) k_edt_tile(const int32_t *__restrict__ in, int32_t *__restrict__ out,
                                                 float *__restrict__ dist, float voxel_size, int nx, int ny,
                                                 int nz) {
    extern __shared__ uint4 lds4[];
    constexpr int NB = NT / TL;   // segments per line (a power of two)
    const int n = AX == 1 ? ny : nz;
    const int kp = edt_key_pitch(n), mp = edt_min_pitch(n);
    const int l = threadIdx.x % TL, seg = threadIdx.x / TL;
    uint32_t *keys = reinterpret_cast<uint32_t *>(lds4), *key = keys + l * kp;   // this thread's line
    uint32_t *mins = keys + TL * kp, *least = mins + l * mp;
    Own *own = reinterpret_cast<Own *>(mins + TL * mp) + l;                       // [n][TL]
    const int ntx = (nx + TL - 1) / TL;
    const int o = (int)(blockIdx.x / ntx);   // z for AX == 1, y for AX == 2
    const int x = (int)(blockIdx.x % ntx) * TL + l;
    // element p of line x: AX == 1 (x, p, o), AX == 2 (x, o, p)
    auto gidx = [&](int p) -> uint32_t {
        return AX == 1 ? ((uint32_t)o * ny + p) * nx + x : ((uint32_t)p * ny + o) * nx + x;
    };
    // the tile into LDS, one block per thread and trip
    for (int p0 = seg * EDT_BLK; p0 < edt_padded(n); p0 += NB * EDT_BLK) {
        int32_t v[EDT_BLK];
        uint32_t k[EDT_BLK];
#pragma unroll
        for (int j = 0; j < EDT_BLK; ++j) v[j] = p0 + j < n && x < nx ? in[gidx(p0 + j)] : EDT_NONE;
#pragma unroll
        for (int j = 0; j < EDT_BLK; ++j)
            k[j] = ((v[j] < 0 ? EMPTY_H : (uint32_t)height<AX>(v[j], x, o)) << 10) | (uint32_t)(1023 - (p0 + j));
        uint32_t m = k[0];
#pragma unroll
        for (int j = 1; j < EDT_BLK; ++j) m = min(m, k[j]);
        *reinterpret_cast<uint4 *>(key + p0) = make_uint4(k[0], k[1], k[2], k[3]);
        *reinterpret_cast<uint4 *>(key + p0 + 4) = make_uint4(k[4], k[5], k[6], k[7]);
        least[p0 / EDT_BLK] = m;
    }
    __syncthreads();
    // the square of a distance given in 32nds, in key units
    auto sq = [](int d32) -> uint32_t { return (uint32_t)__mul24(d32, d32); };
    const int bw = (n + NB - 1) / NB, t0 = seg * bw, t1 = min(t0 + bw, n);   // the thread's segment
    // ---- few candidates: every wavefront counts the first line's
    const int lane = threadIdx.x & 63;
    auto has = [&](int p) { return p < n && keys[min(p, n - 1)] >> 10 != EMPTY_H; };
    int m = 0;
    for (int p0 = 0; p0 < n; p0 += 64) m += __popcll(__ballot(has(p0 + lane)));
    if (m <= few_limit(n)) {
        // their positions, where the search would keep the owners
        uint16_t *few = reinterpret_cast<uint16_t *>(mins + TL * mp);
        if (threadIdx.x < 64)
            for (int p0 = 0, at0 = 0; p0 < n; p0 += 64) {
                const bool one = has(p0 + lane);
                const uint64_t some = __ballot(one);
                if (one) few[at0 + __popcll(some & ((1ull << lane) - 1ull))] = (uint16_t)(p0 + lane);
                at0 += __popcll(some);
            }
        __syncthreads();
        if (t0 >= t1 || x >= nx) return;
        // (s - p)^2 + h_p - s^2 + 1023^2 = (h_p + p^2 + 1023^2) - 2 p s, below 2^22 still
        uint32_t best[EDT_SEG];
#pragma unroll
        for (int j = 0; j < EDT_SEG; ++j) best[j] = ~0u;
        for (int c = 0; c < m; ++c) {
            const int p = few[c], q = -2048 * p;
            const uint32_t k = key[p] + sq(32 * p) + sq(32 * 1023);
#pragma unroll
            for (int j = 0; j < EDT_SEG; ++j) best[j] = min(best[j], (uint32_t)__mul24(q, t0 + j) + k);
        }
#pragma unroll
        for (int h = 0; h < EDT_SEG; h += 8) {   // eight gathers in flight
            int32_t c[8];
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (t0 + h + j < t1) c[j] = m ? in[gidx(1023 - (int)(best[h + j] & 1023))] : EDT_NONE;
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (t0 + h + j < t1) {
                    const int s = t0 + h + j;
                    out[gidx(s)] = c[j];
                    const uint32_t d2 = (best[h + j] - sq(32 * 1023) + sq(32 * s)) >> 10;
                    if (dist) dist[gidx(s)] = m ? voxel_size * sqrtf((float)d2) : INFINITY;
                }
        }
        return;
    }
    // the owner of s, which lies in [a, b]
    auto solve = [&](int s, int a, int b) -> int {
        const int s32 = s * 32;
        uint32_t best = min(key[s], min(key[a] + sq(s32 - a * 32), key[b] + sq(b * 32 - s32)));
        if (b - a > 1) {
            // the open interval's blocks, no farther than the best value's distance (the root rounded up)
            const int r = min((int)__builtin_amdgcn_sqrtf((float)(best >> 10)) + 1, n);
            const unsigned b0 = (unsigned)max(a + 1, s - r) / EDT_BLK, b1 = (unsigned)min(b - 1, s + r) / EDT_BLK;
            for (unsigned g = b0 & ~3u; g <= b1; g += 4) {   // four blocks at a time
                const uint4 m4 = *reinterpret_cast<const uint4 *>(least + g);
                const uint32_t m[4] = {m4.x, m4.y, m4.z, m4.w};
                const int d = (int)(g * (32 * EDT_BLK)) - s32;
                unsigned todo = 0;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int dj = d + j * 32 * EDT_BLK;
                    todo |= m[j] + sq(max(0, max(dj, -32 * (EDT_BLK - 1) - dj))) <= best ? 1u << j : 0u;
                }
                todo &= (15u << max((int)(b0 - g), 0)) & (15u >> max((int)(g + 3 - b1), 0));
                while (todo) {
                    const unsigned blk = g + __builtin_ctz(todo);
                    todo &= todo - 1;
                    const uint4 *kb = reinterpret_cast<const uint4 *>(key + blk * EDT_BLK);
                    const uint4 u = kb[0], w = kb[1];
                    const int e = (int)(blk * (32 * EDT_BLK)) - s32;
                    best = min(best, min(min(min(u.x + sq(e), u.y + sq(e + 32)), min(u.z + sq(e + 64), u.w + sq(e + 96))),
                                         min(min(w.x + sq(e + 128), w.y + sq(e + 160)), min(w.z + sq(e + 192), w.w + sq(e + 224)))));
                }
            }
        }
        return 1023 - (int)(best & 1023);
    };
    // ---- the segments' last positions: level st solves every second multiple of st segments
    for (int st = NB; st > 0; st >>= 1) {
        if (t0 < t1 && (seg + 1) % (2 * st) == st) {
            const int lo = (seg + 1 - st) * bw, hi = (seg + 1 + st) * bw;   // the ends of the solved neighbours
            own[(t1 - 1) * TL] = (Own)solve(t1 - 1, lo > 0 ? own[(lo - 1) * TL] : 0, hi <= n ? own[(hi - 1) * TL] : n - 1);
        }
        __syncthreads();
    }
    if (t0 >= t1 || x >= nx) return;
    // ---- inside the segment
    const int first = t0 > 0 ? own[(t0 - 1) * TL] : 0, last = own[(t1 - 1) * TL];
    for (int st = 8; st > 0; st >>= 1)
        for (int s = t0 + st - 1; s < t1 - 1; s += 2 * st)
            own[s * TL] = (Own)solve(s, s - st < t0 ? first : own[(s - st) * TL], s + st >= t1 - 1 ? last : own[(s + st) * TL]);
    // ---- output, eight gathers in flight per thread
    for (int s0 = t0; s0 < t1; s0 += 8) {
        int32_t c[8];
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (s0 + j < t1) c[j] = in[gidx(own[(s0 + j) * TL])];
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (s0 + j < t1) {
                const int s = s0 + j, p = own[s * TL];
                out[gidx(s)] = c[j];
                if (dist) dist[gidx(s)] = c[j] < 0 ? INFINITY : voxel_size * sqrtf((float)((key[p] + sq((s - p) * 32)) >> 10));
            }
    }
}

template <int AX, int TL, int NT, typename Own>
void launch_tile(const int32_t *in, int32_t *out, float *dist, float voxel_size, int nx, int ny, int nz, hipStream_t s) {
    const int n = AX == 1 ? ny : nz, o_n = AX == 1 ? nz : ny;
    const dim3 grid((unsigned)(((nx + TL - 1) / TL) * (int64_t)o_n));
    const size_t lds = (size_t)TL * (4 * (edt_key_pitch(n) + edt_min_pitch(n)) + n * sizeof(Own));
    hipLaunchKernelGGL((k_edt_tile<AX, TL, NT, Own>), grid, dim3(NT), lds, s, in, out, dist, voxel_size, nx, ny, nz);
}

// Segments of at most 16 positions; 32 lines per tile up to n = 256, 16 up to
// 512, 8 up to 1024, an owner one byte up to n = 256 and two above: at most 46
// KB of LDS up to 256 and 52.5 KB above, three workgroups a compute unit.  At
// 512 and 1024 they fill its 160 KB to the last piece, so the kernel declares
// none besides: with 192 bytes more only two fit (512 x 512 x 32, a tenth of the
// voxels sites: 140 against 135 us, comb 171 against 156).
template <int AX>
void tile_pass(const int32_t *in, int32_t *out, float *dist, float voxel_size, int nx, int ny, int nz, hipStream_t s) {
    const int n = AX == 1 ? ny : nz;
    if (n <= 128) launch_tile<AX, 32, 256, uint8_t>(in, out, dist, voxel_size, nx, ny, nz, s);
    else if (n <= 256) launch_tile<AX, 32, 512, uint8_t>(in, out, dist, voxel_size, nx, ny, nz, s);
    else if (n <= 512) launch_tile<AX, 16, 512, uint16_t>(in, out, dist, voxel_size, nx, ny, nz, s);
    else launch_tile<AX, 8, 512, uint16_t>(in, out, dist, voxel_size, nx, ny, nz, s);
}

}  // namespace

hipError_t launch_edt(int nx, int ny, int nz, const uint8_t *sites, float voxel_size, int32_t *nearest, float *dist,
                      int32_t *A, int32_t *B, hipStream_t s) {
    const int64_t rows = (int64_t)ny * nz;
    const dim3 xgrid((unsigned)((rows * 64 + 255) / 256));
    // the 4-voxel form needs rows of whole 4-byte words and 16-byte aligned rows of A
    if (nx % 4 != 0 || reinterpret_cast<uintptr_t>(sites) % 4 != 0 || reinterpret_cast<uintptr_t>(A) % 16 != 0)
        hipLaunchKernelGGL(k_edt_x, xgrid, dim3(256), 0, s, sites, A, nx, ny, nz);
    else if (nx <= 256)
        hipLaunchKernelGGL(k_edt_x4<1>, xgrid, dim3(256), 0, s, sites, A, nx, ny, nz);
    else if (nx <= 512)
        hipLaunchKernelGGL(k_edt_x4<2>, xgrid, dim3(256), 0, s, sites, A, nx, ny, nz);
    else if (nx <= 768)
        hipLaunchKernelGGL(k_edt_x4<3>, xgrid, dim3(256), 0, s, sites, A, nx, ny, nz);
    else
        hipLaunchKernelGGL(k_edt_x4<4>, xgrid, dim3(256), 0, s, sites, A, nx, ny, nz);
    tile_pass<1>(A, B, nullptr, voxel_size, nx, ny, nz, s);
    tile_pass<2>(B, nearest, dist, voxel_size, nx, ny, nz, s);
    return hipGetLastError();
}

}  // namespace wb
