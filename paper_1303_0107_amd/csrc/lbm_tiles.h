// Tiles of the temporally blocked sweep: which hold a non-solid cell, their
// launch order, and the choice of a region shape (host code only).
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <utility>
#include <vector>

namespace lbm {

// Region bodies: dense (a lane per region column), compacted (lanes take
// consecutive entries of a list of the region's non-solid cells), or dense
// with one region copy updated in place (half the LDS, so taller regions).
enum TbKind : int { kTbDense = 0, kTbCompact = 1, kTbInPlace = 2 };
struct TbVariant {
    int rows, halo, kind;
};

// Non-solid cell counts per tile of a tw x th tiling and the tiles that hold
// one, row-major, packed (tile row << 16 | tile column).
struct Tiling {
    int tw = 0, th = 0, ntx = 0, nty = 0;
    std::vector<int32_t> count, list;
    void relist() {
        list.clear();
        for (int ty = 0; ty < nty; ++ty)
            for (int tx = 0; tx < ntx; ++tx)
                if (count[(size_t)ty * ntx + tx] > 0) list.push_back((ty << 16) | tx);
    }
};

// A lattice's tilings (type 0: solid): each is built once, by a scan of the
// mask, when a sweep needs it, and kept current from the cells every exchange
// step flips.  What is kept costs every exchange step, so a tiling that is
// only asked about is counted instead (tiles_within).
struct Tilings {
    std::vector<Tiling> kept;

    const std::vector<int32_t> &list(const uint8_t *types, int nx, int ny, int tw, int th) {
        for (const auto &t : kept)
            if (t.tw == tw && t.th == th) return t.list;
        Tiling t;
        t.tw = tw;
        t.th = th;
        t.ntx = (nx + tw - 1) / tw;
        t.nty = (ny + th - 1) / th;
        t.count.assign((size_t)t.ntx * t.nty, 0);
        for (int y = 0; y < ny; ++y) {
            const uint8_t *row = types + (size_t)y * nx;
            int32_t *c = t.count.data() + (size_t)(y / th) * t.ntx;
            for (int tx = 0; tx < t.ntx; ++tx) {
                int n = 0;
                const int x1 = std::min(nx, (tx + 1) * tw);
                for (int x = tx * tw; x < x1; ++x) n += row[x] != 0;
                c[tx] += n;
            }
        }
        t.relist();
        kept.push_back(std::move(t));
        return kept.back().list;
    }

    // Cells made solid (removed) and fluid (added) by an exchange step.
    void flip(int nx, const std::vector<int32_t> &removed, const std::vector<int32_t> &added) {
        for (auto &t : kept) {
            for (int32_t n : removed) --t.count[(size_t)((n / nx) / t.th) * t.ntx + (n % nx) / t.tw];
            for (int32_t n : added) ++t.count[(size_t)((n / nx) / t.th) * t.ntx + (n % nx) / t.tw];
            t.relist();
        }
    }
};

// Whether at most `limit` tiles of a tw x th tiling hold a non-solid cell.
inline bool tiles_within(const uint8_t *types, int nx, int ny, int tw, int th, size_t limit) {
    const int ntx = (nx + tw - 1) / tw, nty = (ny + th - 1) / th;
    if ((size_t)ntx * nty <= limit) return true;
    size_t n = 0;
    std::vector<uint8_t> any(ntx);
    for (int ty = 0; ty < nty; ++ty) {
        std::fill(any.begin(), any.end(), 0);
        for (int y = ty * th; y < std::min(ny, (ty + 1) * th); ++y) {
            const uint8_t *row = types + (size_t)y * nx;
            for (int tx = 0; tx < ntx; ++tx) {
                uint8_t v = 0;
                const int x1 = std::min(nx, (tx + 1) * tw);
                for (int x = tx * tw; x < x1; ++x) v |= row[x];
                any[tx] |= v;
            }
        }
        for (int tx = 0; tx < ntx; ++tx) n += any[tx] != 0;
        if (n > limit) return false;
    }
    return true;
}

// Workgroup g of a launch runs on XCD g mod 8, and each XCD has its own L2.
// The row-major tile list is cut into `runs` contiguous runs (a multiple of
// 8, sizes differing by at most one) and XCD k takes runs k, k + 8, ...:
// tiles whose regions overlap (the halo cells) then mostly read them through
// the same L2.  Measured: one run per XCD (bands of tile rows) is fastest
// for the two-copy bodies; the in-place body is fastest with 32 runs, its
// densest tiles spread over the XCDs.
inline std::vector<int32_t> dealt_tiles(const std::vector<int32_t> &list, size_t runs) {
    const size_t n = list.size(), rb = n / runs, re = n % runs;
    std::vector<std::vector<int32_t>> xcd(8);
    size_t at = 0;
    for (size_t r = 0; r < runs; ++r) {
        const size_t len = rb + (r < re ? 1 : 0);
        xcd[r % 8].insert(xcd[r % 8].end(), list.begin() + at, list.begin() + at + len);
        at += len;
    }
    // XCD sizes differ by at most one, the larger ones first: slots 8j + k
    // cover [0, n) exactly
    std::vector<int32_t> out(n);
    for (size_t k = 0; k < 8; ++k)
        for (size_t j = 0; j < xcd[k].size(); ++j) out[8 * j + k] = xcd[k][j];
    return out;
}

// Region shape to run after the mask has changed.  The autotuner's timings
// (ms[v] per step for shape v) hold while a shape's active tiles all run in
// one round of workgroups: tiles(v) <= resident[v], the workgroups of shape v
// the chip holds at once (CUs x workgroups per CU by LDS).  The tuned shape is
// kept (or taken back) whenever it fits; otherwise the fastest timed shape
// that fits; the tuned shape when none does.  tiles(v) is called only for
// shapes that are considered, in order of their timings.
template <typename TileCount>
int fitted_shape(int tuned, const std::vector<double> &ms,
                 const std::vector<size_t> &resident, TileCount tiles) {
    const int nv = (int)ms.size();
    if (tuned < 0 || tuned >= nv || (int)resident.size() != nv) return tuned;
    if (tiles(tuned) <= resident[tuned]) return tuned;
    std::vector<int> order(nv);
    for (int v = 0; v < nv; ++v) order[v] = v;
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return ms[a] < ms[b]; });
    for (int v : order)
        if (v != tuned && tiles(v) <= resident[v]) return v;
    return tuned;
}

// Region shape a new lattice starts with (until one is set or tuned): a rule
// on the precision, the variants and the tile count, never on a size by
// itself.  resident: as for fitted_shape.  value_bytes: of a stored
// population.
//   float   (32,9) dense while its tiles run in one round of workgroups, since
//           a launch's fixed cost is then spread over most steps; else, and
//           with boundary variants, (16,4) dense, of which two workgroups
//           share a CU.  us per step, compacted (32,8) / (16,4) / (32,9):
//           256 x 128 distributor 1.43 / 1.24 / 1.21; 773 x 391 1.83 / 1.38 /
//           1.33; 2200 x 1400 7.05 / 4.51 / 5.47; 1000 x 600 channel 7.23 /
//           4.41 / 4.84; 360 x 180 half collector 1.91 / 1.51 / 1.75.
//   16-bit  (16,4) dense: 256 x 128 1.51 / 1.38 / 1.43, 2200 x 1400 7.27 /
//           4.84 / 6.22.
//   double  (16,4) dense, but compacted with boundary variants (2.30 against
//           2.68) and on a few wave rows of cells (128 x 64: 1.74 against
//           1.96; 773 x 391: 2.33 against 2.23).
inline int start_shape(const std::vector<TbVariant> &shapes, const std::vector<size_t> &resident,
                       int value_bytes, bool variants, int64_t nonsolid, const uint8_t *types,
                       int nx, int ny) {
    auto find = [&](int rows, int halo, int kind) {
        for (size_t v = 0; v < shapes.size(); ++v)
            if (shapes[v].rows == rows && shapes[v].halo == halo && shapes[v].kind == kind)
                return (int)v;
        return 0;
    };
    if (value_bytes == 8)
        return find(16, 4, variants || nonsolid < 40 * 64 ? kTbCompact : kTbDense);
    if (value_bytes == 4 && !variants) {
        const int v = find(32, 9, kTbDense);
        if (tiles_within(types, nx, ny, 64 - 2 * shapes[v].halo,
                         shapes[v].rows - 2 * shapes[v].halo, resident[v]))
            return v;
    }
    return find(16, 4, kTbDense);
}

}  // namespace lbm
