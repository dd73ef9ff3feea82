// Lane arithmetic of the dense blocked body.  Plain functions, so that they
// also compile, and can be checked, on the host.
#pragma once

#include <stdint.h>

#ifdef __HIPCC__
#define LBM_LANE_FN __host__ __device__ __forceinline__
#define LBM_LANE_CONST __device__ constexpr
#else
#define LBM_LANE_FN inline
#define LBM_LANE_CONST constexpr
#endif

namespace lbm {
namespace sweep {

// D2Q9 numbering of Sec. 2.1, and the opposite of each population.
LBM_LANE_CONST int kCx[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
LBM_LANE_CONST int kCy[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
LBM_LANE_CONST int kOpp[9] = {0, 3, 4, 1, 2, 7, 8, 5, 6};

// Element from which the region cell at `pos` pulls population i >= 1 in copy
// 0 of a region of `rw` columns, whose plane j starts at element 2 j pl.
// Every lane of an advanced row pulls this way, also those that hold no cell
// to advance (solid cells, the region's edge): a pull from the lane's own
// cell, as a wall's is, would meet its neighbour's pull in the same LDS bank.
// Rows 0 and the last are never advanced, so the element lies in the region
// whatever the lane; the edge's lanes read one element beyond their row,
// which is the next row's or, for the corners, the next copy's.
LBM_LANE_FN int pull_entry(uint32_t word, int i, int pos, int pl, int rw) {
    const bool wall = ((word >> (i - 1)) & 1u) != 0;
    return wall ? 2 * kOpp[i] * pl + pos : 2 * i * pl + pos - kCy[i] * rw - kCx[i];
}

// What a lane without a cell (solid, or off the lattice) starts with: the
// rest equilibrium, stored as populations or as offsets from it.  Nothing
// reads these lanes, but they are relaxed with their row, and a density of
// zero there would send the whole wave to the divisions of the double form.
LBM_LANE_FN double idle_population(bool offsets, int i) {
    return offsets ? 0.0 : i == 0 ? 4.0 / 9.0 : i < 5 ? 1.0 / 9.0 : 1.0 / 36.0;
}

// The 64 lanes' flags in the opposite order.
LBM_LANE_FN uint64_t mirrored(uint64_t lanes) {
#if defined(__HIPCC__)
    return __builtin_bitreverse64(lanes);
#else
    uint64_t r = 0;
    for (int l = 0; l < 64; ++l) r |= (lanes >> l & 1u) << (63 - l);
    return r;
#endif
}

// Largest depth (distance to the region's edge) of a row's cells: row ry of a
// region of 64 columns and rh rows, `lanes` the columns that hold a cell; 0
// without one.  Lanes l and 63 - l have the same distance, so the row is
// folded onto its first half, where the highest column set has the largest.
LBM_LANE_FN int row_reach(uint64_t lanes, int ry, int rh) {
    const uint32_t cols = (uint32_t)(lanes | mirrored(lanes));
    const int col = cols ? 31 - __builtin_clz(cols) : 0, row = ry < rh - 1 - ry ? ry : rh - 1 - ry;
    return col < row ? col : row;
}

}  // namespace sweep
}  // namespace lbm
