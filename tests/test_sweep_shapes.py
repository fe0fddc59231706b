"""Host: the LDS shapes of the standalone self-collision sweeps fit the 64 KB
limit for every robot that wb_robot_create takes, with a ring and a list for
each state in flight (the header's functions, compiled and swept over the
accepted sizes); so do the fused and plan launches, one wavefront a workgroup,
and the one-launch B-spline step, four, takes at most 72 KB; and the default threshold of the split form follows the
measured crossings, as does the matrix-core broad phase."""
import os
import subprocess

from paper_2603_05493_amd import build

SOURCE = r"""
#include "wb_internal.h"
#include <cstdio>
using namespace wb;
int main() {
    const int sizes[] = {1, 2, 3, 4, 5, 6, 7, 8, 12, 16, 24, 32, 48, 64};
    long shapes = 0;
    int worst = 0;
    for (int nmax : sizes)
        for (int L = 1; L <= 1024; ++L) {
            if (state_lds_bytes(L, nmax) + 4 * 4 * (SC_RING + 128) > LDS_LIMIT) continue;   // refused at creation
            const long most = (long)L * (L - 1) / 2;
            for (long blocks : {0L, 1L, most / 3, most}) {
                const int pad = (int)((blocks + 127) / 128 * 128);
                const SweepShape w = sweep_wave_shape(L, nmax, pad), s = sweep_split_shape(L, nmax, pad);
                const size_t state = state_lds_bytes(L, nmax);
                const size_t need_w = w.states * (state + 4 * (SC_RING + w.list)) + (w.table ? tab_lds_bytes(pad) : 0);
                const size_t need_s = state + 4 * 4 * (SC_RING + s.list) + (s.table ? tab_lds_bytes(pad) : 0);
                const bool ok = w.states >= 1 && w.states <= 4 && (!w.table || w.states == 4) && s.states == 1 &&
                                w.list >= 128 && s.list >= 128 && w.list % 128 == 0 && s.list % 128 == 0 &&
                                need_w <= w.lds && need_s <= s.lds && w.lds <= LDS_LIMIT && s.lds <= LDS_LIMIT;
                if (!ok) {
                    printf("L %d nmax %d blocks %ld: wave %d states %zu B, split %zu B\n", L, nmax, blocks, w.states, w.lds, s.lds);
                    return 1;
                }
                if ((int)state > worst) worst = (int)state;
                ++shapes;
            }
        }
    printf("%ld shapes, largest state %d B\n", shapes, worst);
    return worst == 61440 ? 0 : 2;
}
"""


FUSED = r"""
#include "wb_internal.h"
#include <algorithm>
#include <cstdio>
using namespace wb;
int main() {
    size_t one = 0, four = 0;
    for (int nmax : {1, 2, 3, 4, 5, 6, 7, 8, 12})
        for (int L = 1; L <= 64; ++L)
            for (int blocks = 0; blocks <= L * (L - 1) / 2; ++blocks)
                for (int G : {16, 32, 64}) {
                    const int pad = (blocks + 127) / 128 * 128;
                    const size_t counted = counted_fused_bytes(L, nmax, G, pad);
                    if (G < L || counted > LDS_LIMIT) continue;   // refused
                    one = std::max(one, fused_lds_bytes(L, nmax, blocks, G, 1));
                    // the spline's own part is counted as it is launched
                    four = std::max(four, LDS_LIMIT + fused_lds_bytes(L, nmax, blocks, G, 4) - counted);
                }
    printf("one wavefront %zu B, four %zu B\n", one, four);
    return one <= LDS_LIMIT && four <= 72 * 1024 ? 0 : 1;
}
"""


# links, slots, blocks, pairs and the threshold in states per compute unit, of
# robots whose two forms were timed from 256 to 8,192 states
SPLIT = r"""
#include "wb_internal.h"
#include <cstdio>
int main() {
    const struct { int L, nmax, blocks; long pairs; int per_cu; } robots[] = {
        {4, 5, 3, 75, 0},             {8, 5, 21, 525, 0},          {9, 2, 28, 112, 0},
        {13, 6, 66, 2376, 2},        {16, 12, 105, 15120, 2},      {11, 16, 45, 11520, 2},      {8, 64, 21, 86016, 2},
        {41, 4, 780, 12480, 6},      {25, 8, 276, 17664, 6},       {101, 1, 4950, 4950, 6},     {49, 5, 1128, 28000, 6},      {101, 3, 4950, 44550, 16},
        {61, 8, 1770, 113280, 16},   {61, 12, 1770, 254880, 16},   {49, 16, 1128, 288768, 16},  {101, 7, 4950, 242550, 16},
        {49, 24, 1128, 649728, 16},  {49, 48, 1128, 2598912, 16},  {261, 5, 33670, 841750, 16}};
    // 101 links of 7 spheres: four workgroups of the split form in a compute unit's 160 KB
    if (4 * wb::sweep_split_shape(101, 7, 4992).lds > 160 * 1024) return 2;
    // link blocks on the two sides of the broad phase's crossing
    for (int blocks : {253, 378, 496, 561, 630, 703, 780, 861, 946})
        if (blocks >= wb::BROAD_MATRIX_FROM) return 3;
    for (int blocks : {1035, 1128})
        if (blocks < wb::BROAD_MATRIX_FROM) return 4;
    for (const auto &r : robots) {
        const int got = wb::sweep_split_per_cu(r.L, r.nmax, r.blocks, r.pairs);
        if (got != r.per_cu) {
            printf("L %d nmax %d: %d, not %d\n", r.L, r.nmax, got, r.per_cu);
            return 1;
        }
    }
    return 0;
}
"""


def _run(tmp_path, text):
    src, exe = tmp_path / "shapes.cpp", tmp_path / "shapes"
    src.write_text(text)
    subprocess.run([build.hipcc(), *build.flags(), str(src), "-o", str(exe)], check=True, capture_output=True, text=True,
                   env=dict(os.environ))
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    print(r.stdout)
    assert r.returncode == 0, r.stdout


def test_shapes_fit(tmp_path):
    _run(tmp_path, SOURCE)


def test_fused_launches(tmp_path):
    _run(tmp_path, FUSED)


def test_default_split_threshold(tmp_path):
    _run(tmp_path, SPLIT)
