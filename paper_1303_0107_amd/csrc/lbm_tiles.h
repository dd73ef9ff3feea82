// Tiles of the temporally blocked sweep: which hold a non-solid cell, their
// launch order, and the choice of a region shape (host code only).
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <cstring>
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

// Non-solid cells (types 1 to 3) among n, eight at a time.
inline int cells_in(const uint8_t *p, int n) {
    constexpr uint64_t kOnes = 0x0101010101010101u;
    int c = 0;
    for (; n >= 8; p += 8, n -= 8) {
        uint64_t w;
        std::memcpy(&w, p, 8);
        c += (int)((((w | w >> 1) & kOnes) * kOnes) >> 56);
    }
    for (; n > 0; ++p, --n) c += *p != 0;
    return c;
}

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
            for (int tx = 0; tx < t.ntx; ++tx)
                c[tx] += cells_in(row + tx * tw, std::min(tw, nx - tx * tw));
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
            for (int tx = 0; tx < ntx; ++tx)
                if (!any[tx]) any[tx] = cells_in(row + tx * tw, std::min(tw, nx - tx * tw)) > 0;
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

// The most non-solid cells, and the most rows with one, in any region of a
// shape (64 columns, `rows` rows).  Stops, with what it has found so far, once
// a region holds more than `enough` cells; it starts at half the height, where
// an opening is likely.
struct RegionFill {
    int cells = 0, live_rows = 0;
};
inline RegionFill densest_region(const uint8_t *types, int nx, int ny, int rows, int halo,
                                 int enough) {
    const int iw = 64 - 2 * halo, ih = rows - 2 * halo;
    const int ntx = (nx + iw - 1) / iw, nty = (ny + ih - 1) / ih;
    std::vector<uint8_t> cells((size_t)ny * ntx), counted(ny);  // per row and 64 columns
    RegionFill most;
    for (int k = 0; k < nty; ++k) {
        const int ty = (nty / 2 + k) % nty;
        const int y0 = std::max(0, ty * ih - halo), y1 = std::min(ny, ty * ih - halo + rows);
        for (int y = y0; y < y1; ++y) {
            if (counted[y]) continue;
            counted[y] = 1;
            const uint8_t *row = types + (size_t)y * nx;
            for (int tx = 0; tx < ntx; ++tx) {
                const int x0 = std::max(0, tx * iw - halo);
                cells[(size_t)y * ntx + tx] =
                    (uint8_t)cells_in(row + x0, std::min(nx, tx * iw + iw + halo) - x0);
            }
        }
        for (int tx = 0; tx < ntx; ++tx) {
            RegionFill r;
            for (int y = y0; y < y1; ++y) {
                const int c = cells[(size_t)y * ntx + tx];
                r.cells += c;
                r.live_rows += c != 0;
            }
            most.cells = std::max(most.cells, r.cells);
            most.live_rows = std::max(most.live_rows, r.live_rows);
        }
        if (most.cells > enough) return most;
    }
    return most;
}

// Region shape a new lattice starts with (until one is set or tuned): a rule
// on the storage, the variants, the tiles and what the densest region holds,
// never on a size by itself.  cus: compute units; a 32-row region, and an FP64
// one, takes a whole CU.  value_bytes: of a stored population.
//   What a launch does besides its steps (5 us) is spread over nine of them by
//   (32,9) and over four by (16,4), but a wave of a 32-row region advances two
//   rows a step, and rows without a cell cost nothing.  us per step, checks
//   every 100 steps included, compacted (32,8) / (16,4) / (32,9):
//   float   (32,9) while its tiles run at once, else (16,4): 256 x 128
//           distributor 1.57 / 1.52 / 1.38; 1200 x 300 2.01 / 1.62 / 1.51; 130
//           x 60 channel 2.00 / 1.55 / 1.61; lines of 4 rows in 600 x 600
//           1.27 / 1.42 / 1.04.
//   16-bit  the conversions make the second row dearer: (32,9) while its tiles
//           run at once and either no region has more live rows than waves
//           (FP16: lines of 4 rows 1.39 / 1.52 / 1.17, 100 x 16 channel 1.69 /
//           1.57 / 1.41, but 40 x 20, 18 rows, 1.60 / 1.63 / 1.63; 256 x 128
//           distributor, 32 rows, 1.68 / 1.58 / 1.61) or those of (16,4) do
//           not (1024 x 512: 2.02 / 1.97 / 1.67).
//   16-bit, and any offset form with boundary variants: compacted while no
//           region holds over 640 cells, ten waves' worth (FP16 / BF16 against
//           (16,4): 64 x 48, 399 cells, 0.92 / 0.94; 144 x 90, 625, 0.99 /
//           0.97; 160 x 80, 670, 1.03 / 1.03; 160 x 100, 792, 1.08 / 1.12; FP32
//           128 x 64 collector, 440, 0.96); else (16,4).
//   double  a compacted list packs a region's cells into few waves, a dense
//           row takes one each: compacted while the tiles run at once and the
//           densest region has at most 40 cells per live row (compacted against dense: 64 x 48
//           distributor, 18, 0.91; 24 x 12 channel, 24, 0.90; 112 x 64, 31,
//           0.98; 160 x 80, 34, 0.99; 40 x 20 channel, 40, 0.97; 144 x 90, 41,
//           1.09; 256 x 128, 45, 1.08; lines of 4 rows, 64, 1.10), and with
//           boundary variants (360 x 180 half collector 0.90).
inline int start_shape(const std::vector<TbVariant> &shapes, int cus, int value_bytes,
                       bool variants, const uint8_t *types, int nx, int ny) {
    auto find = [&](int rows, int halo, int kind) {
        for (size_t v = 0; v < shapes.size(); ++v)
            if (shapes[v].rows == rows && shapes[v].halo == halo && shapes[v].kind == kind)
                return (int)v;
        return 0;
    };
    auto one_each = [&](int rows, int halo) {
        return tiles_within(types, nx, ny, 64 - 2 * halo, rows - 2 * halo, cus);
    };
    if (value_bytes == 8) {
        if (variants) return find(16, 4, kTbCompact);
        if (!one_each(16, 4)) return find(16, 4, kTbDense);
        const RegionFill r = densest_region(types, nx, ny, 16, 4, 40 * 16);
        return find(16, 4, r.cells <= 40 * r.live_rows ? kTbCompact : kTbDense);
    }
    if (!variants && one_each(32, 9) &&
        (value_bytes == 4 || !one_each(16, 4) ||
         densest_region(types, nx, ny, 32, 9, 64 * 16).live_rows <= 16))
        return find(32, 9, kTbDense);
    if ((value_bytes == 2 || variants) && one_each(32, 8) &&
        densest_region(types, nx, ny, 32, 8, 640).cells <= 640)
        return find(32, 8, kTbCompact);
    return find(16, 4, kTbDense);
}

}  // namespace lbm
