"""Where a drawn point falls in a row's running sum: the decision functions of the sampling kernels, compiled for the host.

The kernels add a row's weights level by level (waves, tiles, lanes, four values) and every level in its own order, so a level's sums may
fall a rounding short of, or past, what the level above saw.  The driver below repeats those orders on weights that spread over
50 binary orders of magnitude, with many zeros, and asks for the points where the levels disagree; what must hold is the rule of
inverse-CDF sampling: an index of positive weight, the last one of its level where no running sum exceeds the point."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>
#include <hip/hip_runtime.h>
#include "asd_sample.h"
#define REQUIRE(c) do { if (!(c)) { printf("failed: %s (line %d)\n", #c, __LINE__); return 1; } } while (0)

static double butterfly(const double* v) {                     // wave_sum: lane 0's value after xor 32, 16, .. 1
    double x[64], y[64];
    for (int l = 0; l < 64; ++l) x[l] = v[l];
    for (int o = 32; o > 0; o >>= 1) { for (int l = 0; l < 64; ++l) y[l] = x[l] + x[l ^ o]; for (int l = 0; l < 64; ++l) x[l] = y[l]; }
    return x[0];
}
static void scan(const double* v, double* incl) {              // the kernels' inclusive scan over the lanes
    double y[64];
    for (int l = 0; l < 64; ++l) incl[l] = v[l];
    for (int o = 1; o < 64; o <<= 1) {
        for (int l = 0; l < 64; ++l) y[l] = l >= o ? incl[l] + incl[l - o] : incl[l];
        for (int l = 0; l < 64; ++l) incl[l] = y[l];
    }
}

int main() {
    std::mt19937_64 rng(1);
    std::uniform_real_distribution<double> ex(-50.0, 0.0), un(0.0, 1.0);
    int zero_first = 0, tile_short = 0, lane_short = 0;
    for (int trial = 0; trial < 20000; ++trial) {
        const double zeros = 0.3 + 0.6 * un(rng);
        float e[8][64][4];
        double sl[8][64], sum[8], all[64];
        for (int l = 0; l < 64; ++l) all[l] = 0.0;
        for (int k = 0; k < 8; ++k) {
            for (int l = 0; l < 64; ++l) {
                for (int j = 0; j < 4; ++j) e[k][l][j] = un(rng) < zeros ? 0.f : (float)std::exp2(ex(rng));
                sl[k][l] = ((double)e[k][l][0] + e[k][l][1]) + ((double)e[k][l][2] + e[k][l][3]);
                all[l] += sl[k][l];
            }
            sum[k] = butterfly(sl[k]);
        }
        const double total = butterfly(all);                   // this wave's share, as the level above sees it
        double run = 0.0;
        for (int k = 0; k < 8; ++k) run += sum[k];
        std::vector<double> points = {un(rng) * total, std::nextafter(total, 0.0)};
        for (int k = 0; k < 8; ++k) {                          // the ends of every lane's interval, as its scan has them
            double incl[64], before = 0.0;
            for (int i = 0; i < k; ++i) before += sum[i];
            scan(sl[k], incl);
            for (int l = 0; l < 64; ++l) points.push_back(before + incl[l]);
        }
        for (const double t : points) {
            if (!(t < total)) continue;
            IntervalSearch tiles(t, 0.0);
            for (int k = 0; k < 8; ++k) tiles.visit(k, sum[k]);
            const int kt = tiles.index();
            double incl[64];
            scan(sl[kt], incl);
            uint64_t over = 0, some = 0;
            for (int l = 0; l < 64; ++l) { over |= (uint64_t)(t < tiles.before + incl[l]) << l; some |= (uint64_t)(sl[kt][l] > 0.0) << l; }
            REQUIRE(some);
            const int lane = sample_lane(over, some);
            const int j = sample_of_four(e[kt][lane], tiles.before + (lane ? incl[lane - 1] : 0.0), t);
            REQUIRE(lane >= 0 && lane < 64 && j >= 0 && j < 4);
            REQUIRE(e[kt][lane][j] > 0.f);                      // never an index of weight zero
            if (over && !(some >> __builtin_ctzll(over) & 1)) ++zero_first;
            if (!(over & some)) { ++lane_short; REQUIRE(lane == 63 - __builtin_clzll(some)); }
            if (!(t < run)) {                                   // no running sum exceeds t: the last positive weight of all
                ++tile_short;
                int lk = 7, ll = 63, lj = 3;
                while (!(e[lk][ll][lj] > 0.f)) if (--lj < 0) { lj = 3; if (--ll < 0) { ll = 63; --lk; } }
                REQUIRE(kt == lk && lane == ll && j == lj);
            }
        }
    }
    printf("zero_first %d tile_short %d lane_short %d\n", zero_first, tile_short, lane_short);
    REQUIRE(zero_first > 0 && tile_short > 0 && lane_short > 0);      // the points did reach the places where the levels disagree
    printf("all draws valid\n");
    return 0;
}
"""


@pytest.mark.slow
def test_points_on_rounding_boundaries_draw_a_positive_weight(tmp_path):
    hipcc = shutil.which("hipcc")
    if not hipcc:
        pytest.skip("no hipcc")
    src, exe = tmp_path / "pick.hip", tmp_path / "pick"
    src.write_text(DRIVER)
    subprocess.run([hipcc, "--offload-arch=gfx950", "-O1", "-ffp-contract=off", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    "-I", os.path.join(ROOT, "paper_2410_01028_amd", "csrc"), str(src), "-o", str(exe)], check=True, capture_output=True, timeout=300)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "all draws valid" in r.stdout, r.stdout[-2000:]
