// How a launch of the marching sweep is cut into waves, and which lattices
// march (host code).
#pragma once

#include <stdint.h>

#include <algorithm>

namespace lbm {

// `steps` (1, 2, 4; in float also 6, 7) time steps a launch, one wave per
// strip of `width` columns and segment of rows.  Interior strips are cut into
// `segs` segments of `rows` rows, the two edge strips into `edge_segs` of
// `edge_rows`; `blocks` workgroups of kMarchThreads hold the waves.
constexpr int kMarchThreads = 256;
struct MarchPlan {
    int steps, width, strips, segs, rows, edge_segs, edge_rows, waves, blocks;
};

// The widest strips, up to the 64 - 2 steps columns that a wave can own, for
// which no lane of an interior strip lies on the last column.  With a thin
// last strip its neighbour, whose segments are the long ones, has the outlet
// in its halo, and its rows take half as long again: FP32, 6 steps, us per
// step, 1200 x 760, in strips of 52, the last of 4 columns, 8.0, of 51 7.0;
// 1150 x 1050 9.4 and 7.6; FP16, 4 steps, 2300 x 2000 24.1 and 20.2.
inline int strip_width(int nx, int steps) {
    const int widest = 64 - 2 * steps;
    for (int w = widest; w > widest / 2; --w) {
        const int last = nx - (nx - 1) / w * w;
        if (last > 64 - steps - w) return w;
    }
    return widest;
}

// The shortest segments (at least four rows) for which all workgroups run at
// once with `fill` waves on each SIMD.  Fewer waves do not hide the latency of
// their own instructions, more only lengthen the launch by the rows that each
// segment advances beyond its ends.  in_cache: whether both population
// buffers fit the 256 MB cache; beyond it HBM bounds the launch, and strips
// that start off its lines cost more than the neighbour of a thin last one
// (FP64 2300 x 2000 52.1 in strips of 55, 50.4 of 56).
inline MarchPlan march_plan(int nx, int ny, int steps, int cus, int fill, bool in_cache) {
    const int target = fill * cus * (kMarchThreads / 64);
    MarchPlan p{};
    p.steps = steps;
    p.width = in_cache ? strip_width(nx, steps) : 64 - 2 * steps;
    p.strips = (nx + p.width - 1) / p.width;
    for (p.rows = std::max(4, (int)((int64_t)ny * p.strips / target));; ++p.rows) {
        p.segs = (ny + p.rows - 1) / p.rows;
        p.edge_rows = (p.rows + 1) / 2;
        p.edge_segs = (ny + p.edge_rows - 1) / p.edge_rows;
        p.waves = 2 * p.edge_segs + (p.strips - 2) * p.segs;
        if (p.waves <= target || p.rows >= ny) break;
    }
    p.blocks = (p.waves + kMarchThreads / 64 - 1) / (kMarchThreads / 64);
    return p;
}

}  // namespace lbm
