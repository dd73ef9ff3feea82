"""The region shape of a new lattice and the tilings a lattice keeps (host
code, csrc/lbm_tiles.h), compiled with the host C++ compiler."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_1303_0107_amd import inputs as I

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1303_0107_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include "lbm_tiles.h"
// argv: nx ny value_bytes variants; the mask on stdin.  Prints the shape
// (rows halo kind), the tilings kept after its tiles were listed, and, for
// limits around the true count of its tiles, what tiles_within says.
int main(int argc, char **argv) {
    using namespace lbm;
    const int nx = std::atoi(argv[1]), ny = std::atoi(argv[2]), bytes = std::atoi(argv[3]);
    const bool variants = std::atoi(argv[4]) != 0;
    std::vector<uint8_t> t((size_t)nx * ny);
    if (std::fread(t.data(), 1, t.size(), stdin) != t.size()) return 1;
    const std::vector<TbVariant> shapes =
        bytes == 8 ? std::vector<TbVariant>{{16, 4, kTbCompact}, {16, 4, kTbDense},
                                            {16, 2, kTbCompact}, {32, 8, kTbInPlace}}
                   : std::vector<TbVariant>{{32, 8, kTbCompact}, {32, 8, kTbDense},
                                            {32, 4, kTbCompact}, {16, 4, kTbCompact},
                                            {16, 4, kTbDense},   {32, 9, kTbDense}};
    std::vector<size_t> resident;
    for (const TbVariant &v : shapes) resident.push_back(v.rows == 16 && bytes < 8 ? 512 : 256);
    int64_t nonsolid = 0;
    for (uint8_t v : t) nonsolid += v != 0;
    Tilings kept;
    const int v = start_shape(shapes, resident, bytes, variants, nonsolid, t.data(), nx, ny);
    const int tw = 64 - 2 * shapes[v].halo, th = shapes[v].rows - 2 * shapes[v].halo;
    const size_t n = kept.list(t.data(), nx, ny, tw, th).size();
    std::printf("%d %d %d %zu", shapes[v].rows, shapes[v].halo, shapes[v].kind, kept.kept.size());
    for (long d = -1; d <= 1; ++d)
        std::printf(" %d", tiles_within(t.data(), nx, ny, tw, th, (size_t)std::max(0l, (long)n + d)));
    std::printf(" %zu\n", n);
    return 0;
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp("start")
    src = d / "start.cpp"
    src.write_text(DRIVER)
    exe = d / "start"
    subprocess.run([cxx, "-std=c++17", "-O2", "-Wall", "-Werror", "-I", CSRC, str(src), "-o",
                    str(exe)], check=True)

    def ask(t, value_bytes, variants=0):
        t = np.ascontiguousarray(t, np.uint8)
        out = subprocess.run([str(exe), str(t.shape[1]), str(t.shape[0]), str(value_bytes),
                              str(variants)], input=t.tobytes(), check=True,
                             capture_output=True).stdout.split()
        return [int(v) for v in out]
    return ask


def _tiles(t, tw, th):
    ny, nx = t.shape
    return sum(bool(t[y:y + th, x:x + tw].any()) for y in range(0, ny, th)
               for x in range(0, nx, tw))


@pytest.mark.parametrize("value_bytes", [2, 4, 8])
@pytest.mark.parametrize("size", [(128, 64, 2), (773, 391, 3), (1024, 512, 3), (2048, 1024, 4)])
def test_a_new_lattice_keeps_one_tiling(rule, size, value_bytes):
    """Every exchange step updates and relists each tiling a handle keeps, so
    the shapes the rule only looks at leave none behind."""
    t = I.distributor(*size, None)
    rows, halo, kind, kept, below, equal, above, n = rule(t, value_bytes)
    assert kept == 1
    assert n == _tiles(t, 64 - 2 * halo, rows - 2 * halo)
    assert (below, equal, above) == (0, 1, 1)


def test_tiles_of_an_empty_and_a_full_lattice(rule):
    t = np.zeros((40, 200), np.uint8)
    assert rule(t, 4)[-4:] == [1, 1, 1, 0]
    t[:] = 1
    assert rule(t, 4)[-4:-1] == [0, 1, 1]
