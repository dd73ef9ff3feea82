"""Lane arithmetic of the dense blocked body (csrc/lbm_lanes.h), compiled with
the host C++ compiler: where lanes pull from, and what becomes of the lanes
that hold no cell."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1303_0107_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include <algorithm>
#include <cmath>
#include <random>
#include <vector>
#include "lbm_lanes.h"
using namespace lbm::sweep;
// argv: rows halo seed fraction-solid stripes offsets.  A region of random
// cells (with stripes: rows of cells four apart, the others solid) is advanced
// as the body advances it, every lane of a row while one of its cells has the
// depth, on full populations (double form) or offsets.  Prints a fault, or the smallest and
// largest density that any advanced lane met.
int main(int argc, char **argv) {
    const int RH = std::atoi(argv[1]), H = std::atoi(argv[2]), RW = 64, PL = RW * RH;
    std::mt19937 rng(std::atoi(argv[3]));
    const double p_solid = std::atof(argv[4]);
    const bool stripes = std::atoi(argv[5]) != 0, offsets = std::atoi(argv[6]) != 0;
    std::uniform_real_distribution<double> u(0.0, 1.0);
    std::vector<int> solid(PL);
    for (int n = 0; n < PL; ++n) solid[n] = u(rng) < p_solid || (stripes && n / RW % 4 != 1);
    auto is_solid = [&](int x, int y) {
        return x < 0 || x >= RW || y < 0 || y >= RH || solid[y * RW + x];
    };
    std::vector<uint32_t> word(PL, 0);
    for (int y = 0; y < RH; ++y)
        for (int x = 0; x < RW; ++x)
            if (!solid[y * RW + x])
                for (int i = 1; i < 9; ++i)
                    // beyond the region lies more lattice: a wall only where a solid cell is
                    if (x - kCx[i] >= 0 && x - kCx[i] < RW && y - kCy[i] >= 0 && y - kCy[i] < RH &&
                        is_solid(x - kCx[i], y - kCy[i]))
                        word[y * RW + x] |= 1u << (i - 1);
    const double w[9] = {4. / 9, 1. / 9, 1. / 9, 1. / 9, 1. / 9, 1. / 36, 1. / 36, 1. / 36, 1. / 36};
    // two copies, interleaved by plane; the second holds what an earlier region left
    std::vector<double> L(18 * PL);
    for (int n = 0; n < 18 * PL; ++n) L[n] = idle_population(offsets, n / (2 * PL));
    for (int n = 0; n < PL; ++n)
        for (int i = 0; i < 9; ++i)
            L[2 * i * PL + n] = solid[n] ? idle_population(offsets, i)
                                         : w[i] * (1.0 + 0.1 * (u(rng) - 0.5)) - (offsets ? w[i] : 0.0);
    const std::vector<double> first(L.begin(), L.begin() + PL);
    std::vector<double> rest = first;
    // largest depth of a row's cells (the distance to the region's edge)
    std::vector<int> reach(RH, 0);
    for (int n = 0; n < PL; ++n) {
        const int x = n % RW, y = n / RW;
        if (!solid[n]) reach[y] = std::max(reach[y], std::min({x, RW - 1 - x, y, RH - 1 - y}));
    }
    for (int y = 0; y < RH; ++y) {
        uint64_t lanes = 0;
        for (int x = 0; x < RW; ++x) lanes |= (uint64_t)!solid[y * RW + x] << x;
        if (row_reach(lanes, y, RH) != reach[y]) {
            std::printf("row %d reach %d for %d\n", y, row_reach(lanes, y, RH), reach[y]);
            return 0;
        }
    }
    double lo = 1.0, hi = 1.0;
    for (int s = 1; s <= H; ++s) {
        const int B = (s - 1) & 1;
        for (int y = 0; y < RH; ++y) {
            if (reach[y] < s) continue;
            for (int x = 0; x < RW; ++x) {
                double f[9];
                f[0] = rest[y * RW + x];
                for (int i = 1; i < 9; ++i) {
                    const int pos = y * RW + x, e = pull_entry(word[pos], i, pos, PL, RW);
                    if (e < 0 || e + B * PL >= 18 * PL) {
                        std::printf("row %d lane %d population %d leaves the region\n", y, x, i);
                        return 0;
                    }
                    const bool wall = (word[pos] >> (i - 1)) & 1u;
                    const int xs = x - kCx[i], ys = y - kCy[i];
                    if (e != (wall ? 2 * kOpp[i] * PL + pos : 2 * i * PL + ys * RW + xs) &&
                        xs >= 0 && xs < RW) {
                        std::printf("row %d lane %d population %d wrong source\n", y, x, i);
                        return 0;
                    }
                    f[i] = L[e + B * PL];
                }
                double r = offsets ? 1.0 : 0.0, jx = 0, jy = 0;
                for (int i = 0; i < 9; ++i) {
                    r += f[i];
                    jx += kCx[i] * f[i];
                    jy += kCy[i] * f[i];
                }
                if (!(r > -1e300 && r < 1e300)) {
                    std::printf("step %d row %d lane %d density not finite\n", s, y, x);
                    return 0;
                }
                lo = std::fmin(lo, r);
                hi = std::fmax(hi, r);
                const double ux = jx / r, uy = jy / r, om = 1.0 / 0.6;
                for (int i = 0; i < 9; ++i) {
                    const double cu = kCx[i] * ux + kCy[i] * uy;
                    const double feq = w[i] * r * (1 + 3 * cu + 4.5 * cu * cu - 1.5 * (ux * ux + uy * uy)) -
                                       (offsets ? w[i] : 0.0);
                    f[i] = f[i] - om * (f[i] - feq);
                    if (i > 0) L[(2 * i + 1 - B) * PL + y * RW + x] = f[i];
                }
                rest[y * RW + x] = f[0];
            }
        }
    }
    // lanes of a row without walls: all of them in different columns
    for (int i = 1; i < 9; ++i) {
        std::vector<int> seen(RW, 0);
        for (int x = 0; x < RW; ++x) ++seen[pull_entry(0, i, RH / 2 * RW + x, PL, RW) % RW];
        for (int x = 0; x < RW; ++x)
            if (seen[x] != 1) {
                std::printf("population %d: two lanes in one column\n", i);
                return 0;
            }
    }
    std::printf("%.17g %.17g\n", lo, hi);
    return 0;
}
"""


@pytest.fixture(scope="module")
def region(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp("lanes")
    src = d / "lanes.cpp"
    src.write_text(DRIVER)
    exe = d / "lanes"
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-I", CSRC, str(src), "-o", str(exe)],
                   check=True)

    def advance(rows, halo, seed, solid, stripes, offsets):
        out = subprocess.run([str(exe), str(rows), str(halo), str(seed), str(solid),
                              str(int(stripes)), str(int(offsets))], check=True, capture_output=True, text=True).stdout
        try:
            return [float(v) for v in out.split()]
        except ValueError:
            pytest.fail(out)
    return advance


# every dense shape that is compiled, from no solid cell to nothing but solid
@pytest.mark.parametrize("offsets", [False, True])
@pytest.mark.parametrize("solid,stripes", [(0.0, 0), (0.02, 0), (0.5, 0), (1.0, 0), (0.0, 1),
                                           (0.3, 1)])
@pytest.mark.parametrize("rows,halo", [(16, 4), (32, 8), (32, 9)])
def test_lanes_without_a_cell_stay_near_rest(region, rows, halo, solid, stripes, offsets):
    """A dense row is advanced whole.  Its lanes without a cell pull inside
    the region, from other columns than their neighbours, and their density
    stays near that of rest (a density of zero would take every lane of the
    double form's wave through two divisions).  The cells start within 5 % of rest; nine steps of a
    scheme that conserves what it does not reflect leave the densities far
    inside a factor of two."""
    lo, hi = region(rows, halo, 3, solid, stripes, offsets)
    assert 0.5 < lo <= hi < 2.0


REACH = r"""
#include <algorithm>
#include <cstdio>
#include "lbm_lanes.h"
// Every row of one or two cells, in each row of a region.
int main() {
    for (int rh : {16, 32})
        for (int ry = 0; ry < rh; ++ry)
            for (int a = 0; a <= 64; ++a)
                for (int b = a; b <= 64; ++b) {
                    uint64_t lanes = 0;
                    int want = 0;
                    for (int x : {a, b})
                        if (x < 64) {
                            lanes |= 1ull << x;
                            want = std::max(want, std::min({x, 63 - x, ry, rh - 1 - ry}));
                        }
                    if (lbm::sweep::row_reach(lanes, ry, rh) != want)
                        return std::printf("%d %d %d %d\n", rh, ry, a, b), 1;
                }
    return 0;
}
"""


def test_row_reach_is_the_deepest_cell(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    (tmp_path / "reach.cpp").write_text(REACH)
    exe = tmp_path / "reach"
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", CSRC, str(tmp_path / "reach.cpp"), "-o",
                    str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
