"""How the marching sweep cuts a lattice into waves (host code,
csrc/lbm_march_plan.h), compiled with the host C++ compiler."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1303_0107_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include "lbm_march_plan.h"
using namespace lbm;
// argv: step counts.  Lattices of every width from the narrowest that marches
// up to 1500 columns, and some wide ones, in a few heights.
int main(int argc, char **argv) {
    for (int k = 1; k < argc; ++k) {
        const int S = std::atoi(argv[k]);
        for (int nx = 128; nx <= 65536; nx = nx < 1500 ? nx + 1 : nx * 3 / 2 + 1)
            for (int ny : {3, 37, 760, 9000, -760}) {
                const int cus = 256, fill = 2;
                const bool in_cache = ny > 0;
                ny = std::abs(ny);
                const MarchPlan p = march_plan(nx, ny, S, cus, fill, in_cache);
                auto bad = [&](const char *what) {
                    std::printf("%s: S %d nx %d ny %d strips %d\n", what, S, nx, ny, p.strips);
                    return 1;
                };
                if (p.strips < 3 || p.strips * p.width < nx || (p.strips - 1) * p.width >= nx)
                    return bad("cover");
                if (p.width < 1 || p.width > 64 - 2 * S) return bad("width");
                // the columns of the interior strips' lanes
                const int first = p.width - S, last = (p.strips - 2) * p.width - S + 63;
                if (in_cache && (first <= 0 || last >= nx - 1)) return bad("boundary column in an interior strip");
                if (p.segs * p.rows < ny || (p.segs - 1) * p.rows >= ny ||
                    p.edge_segs * p.edge_rows < ny || (p.edge_segs - 1) * p.edge_rows >= ny)
                    return bad("segments");
                if (p.waves != 2 * p.edge_segs + (p.strips - 2) * p.segs ||
                    p.blocks * (kMarchThreads / 64) < p.waves)
                    return bad("waves");
                if (p.waves > fill * cus * 4 && p.rows < ny) return bad("more waves than run at once");
            }
    }
    return 0;
}
"""


@pytest.mark.parametrize("steps", [1, 2, 4, 6, 7])
def test_strips_cover_the_lattice_and_only_edge_strips_see_a_boundary(tmp_path, steps):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    (tmp_path / "plan.cpp").write_text(DRIVER)
    exe = tmp_path / "plan"
    subprocess.run([cxx, "-std=c++17", "-O2", "-Wall", "-Werror", "-I", CSRC,
                    str(tmp_path / "plan.cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe), str(steps)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


RULE = r"""
#include <cstdio>
#include <cstdlib>
#include "lbm_march_plan.h"
// argv: value_bytes cells nonsolid nx; prints from, steps, and the waves per
// SIMD of launches of that many steps and of two
int main(int, char **argv) {
    const int bytes = std::atoi(argv[1]), nx = std::atoi(argv[4]);
    const long long cells = std::atoll(argv[2]), nonsolid = std::atoll(argv[3]);
    const lbm::MarchRule r = lbm::march_rule(bytes, cells, nonsolid, nx);
    const bool c = lbm::clear(cells, nonsolid, nx);
    std::printf("%lld %d %d %d\n", (long long)r.from, r.steps, lbm::march_fill(bytes, r.steps, c),
                lbm::march_fill(bytes, 2, c));
    return 0;
}
"""


# channels, channels with solid cells up to and past one in a thousand, and the
# step count of the largest
@pytest.mark.parametrize("value_bytes,nx,ny,solid,want", [
    (8, 1024, 512, 0, [500000, 4, 2, 2]),
    (8, 4096, 2048, 80000, [500000, 4, 2, 2]),
    (4, 1500, 760, 0, [1100000, 6, 2, 2]),
    (4, 1500, 760, 1140, [1100000, 6, 2, 2]),
    (4, 1500, 760, 1141, [2400000, 6, 3, 2]),
    (4, 2048, 2047, 0, [1100000, 6, 2, 2]),
    (4, 2048, 2048, 0, [1100000, 7, 2, 2]),
    (4, 2048, 2048, 90000, [2400000, 7, 2, 2]),
    (2, 1500, 760, 0, [1100000, 4, 3, 3]),
    (2, 4096, 2048, 90000, [2400000, 4, 3, 3]),
])
def test_which_lattices_march(tmp_path, value_bytes, nx, ny, solid, want):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    (tmp_path / "rule.cpp").write_text(RULE)
    exe = tmp_path / "rule"
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC,
                    str(tmp_path / "rule.cpp"), "-o", str(exe)], check=True)
    cells = nx * ny
    out = subprocess.run([str(exe), str(value_bytes), str(cells), str(cells - 2 * nx - solid),
                          str(nx)], check=True, capture_output=True, text=True).stdout
    assert [int(v) for v in out.split()] == want
