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
// (rows halo kind), the tilings kept after its tiles were listed, for limits
// around the true count of its tiles what tiles_within says, that count, and
// the fill of the densest region of three shapes.
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
    Tilings kept;
    const int v = start_shape(shapes, 256, bytes, variants, t.data(), nx, ny);
    const int tw = 64 - 2 * shapes[v].halo, th = shapes[v].rows - 2 * shapes[v].halo;
    const size_t n = kept.list(t.data(), nx, ny, tw, th).size();
    std::printf("%d %d %d %zu", shapes[v].rows, shapes[v].halo, shapes[v].kind, kept.kept.size());
    for (long d = -1; d <= 1; ++d)
        std::printf(" %d", tiles_within(t.data(), nx, ny, tw, th, (size_t)std::max(0l, (long)n + d)));
    std::printf(" %zu", n);
    for (int s = 0; s < 3; ++s) {
        const int rows = s ? 32 : 16, halo = s == 0 ? 4 : 7 + s;
        const RegionFill r = densest_region(t.data(), nx, ny, rows, halo, rows * 64);
        std::printf(" %d %d", r.cells, r.live_rows);
    }
    std::printf("\n");
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
    rows, halo, kind, kept, below, equal, above, n = rule(t, value_bytes)[:8]
    assert kept == 1
    assert n == _tiles(t, 64 - 2 * halo, rows - 2 * halo)
    assert (below, equal, above) == (0, 1, 1)


def test_tiles_of_an_empty_and_a_full_lattice(rule):
    t = np.zeros((40, 200), np.uint8)
    assert rule(t, 4)[4:] == [1, 1, 1] + [0] * 7
    t[:] = 1
    assert rule(t, 4)[4:7] == [0, 1, 1]


def _fill(t, rows, halo):
    ny, nx = t.shape
    iw, ih = 64 - 2 * halo, rows - 2 * halo
    cells, live = 0, 0
    for y in range(0, ny, ih):
        for x in range(0, nx, iw):
            r = t[max(0, y - halo):y + ih + halo, max(0, x - halo):x + iw + halo] != 0
            cells, live = max(cells, int(r.sum())), max(live, int(r.any(axis=1).sum()))
    return [cells, live]


@pytest.mark.parametrize("size", [(3, 3), (64, 17), (57, 16), (113, 41), (300, 97)])
@pytest.mark.parametrize("share", [0.002, 0.1, 1.0])
def test_densest_region(rule, size, share):
    t = (np.random.default_rng(size[0]).random(size[::-1]) < share).astype(np.uint8)
    t[0, 0] = 1
    assert rule(t, 2)[8:] == _fill(t, 16, 4) + _fill(t, 32, 8) + _fill(t, 32, 9)


def _lines(nx, ny, w, every):
    t = np.zeros((ny, nx), np.uint8)
    for y in range(w, ny - w, every):
        t[y:y + w] = 1
    return t


DENSE, COMPACT = 0, 1


# Both sides of every line of the rule: few rows of cells, few cells, a region
# full of them, more tiles than CUs, and the boundary variants.
@pytest.mark.parametrize("value_bytes,variants,t,shape", [
    (4, 0, I.channel(130, 60), (32, 9, DENSE)),
    (4, 0, I.channel(700, 400), (16, 4, DENSE)),
    (2, 0, I.channel(100, 18), (32, 9, DENSE)),          # 16 rows of cells
    (2, 0, I.channel(100, 20), (16, 4, DENSE)),          # 18
    (2, 0, _lines(600, 600, 4, 48), (32, 9, DENSE)),
    (2, 0, _lines(2400, 2400, 4, 48), (16, 4, DENSE)),   # more tiles than CUs
    (2, 0, I.distributor(1024, 512, 3, None), (32, 9, DENSE)),
    (2, 0, I.distributor(128, 64, 2, None), (32, 8, COMPACT)),
    (2, 0, I.distributor(256, 128, 2, None), (16, 4, DENSE)),
    (2, 1, I.collector(128, 64, 2, None), (32, 8, COMPACT)),
    (4, 1, I.collector(128, 64, 2, None), (32, 8, COMPACT)),
    (4, 1, I.collector(300, 160, 3, None), (16, 4, DENSE)),
    (8, 0, I.distributor(112, 64, 1, None), (16, 4, COMPACT)),
    (8, 0, I.distributor(144, 90, 1, None), (16, 4, DENSE)),
    (8, 0, _lines(300, 300, 3, 36), (16, 4, DENSE)),
    (8, 1, I.collector(300, 160, 3, None), (16, 4, COMPACT)),
])
def test_start_shapes(rule, value_bytes, variants, t, shape):
    assert tuple(rule(t, value_bytes, variants)[:3]) == shape
