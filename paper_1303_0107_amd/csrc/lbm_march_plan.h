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

// Which lattices march, and how, unless the environment says otherwise.
struct MarchRule {
    int64_t from;  // cells, in tiles with a non-solid one, from which an untuned lattice marches
    int steps;     // of a launch
};
// value_bytes: of a stored population; cells: of the lattice.
//   from   Below it a segment has too few rows for what it advances beyond its
//          ends.  The sweep advances solid cells as well, where the blocked one
//          skips tiles without others, and the rows near one take the longer
//          path, so a lattice with more in it than its two walls and one cell
//          in a thousand marches later: `clear` tells.  us per step, checks
//          every 100 steps included, blocked / marching:
//          FP64  800 x 700, 0.2 to 20 % of its cells solid, 10.3 / 9.6-9.9, two
//                solid blocks (470,000 cells in tiles) 8.7 / 9.6; 1024 x 512
//                channel 9.1 / 7.6; 1500 x 900, 20 % solid, 21.0 / 16.0.
//          FP32  channels 1000 x 1000 7.0 / 7.1, 1500 x 740 7.6 / 7.1, 1150 x
//                1050 8.2 / 7.6, 2000 x 1000 12.6 / 10.0; 1 % solid, 1500 x 900
//                9.0 / 10.0, 2000 x 1400 17.0 / 15.7; two blocks 2000 x 1400
//                (2.3 M in tiles) 14.4 / 15.4, 2800 x 2000 32.5 / 30.7.
//          FP16  channels 1000 x 1000 7.6 / 7.7, 1500 x 740 8.4 / 7.7, 2000 x
//                1000 14.1 / 11.1; 1 % solid, 1500 x 900 9.9 / 10.8, 2000 x 1400
//                19.2 / 17.2.
//   steps  In double the registers end at 4 (eight spill in float).  On 16-bit
//          storage 4, since the conversions make every step beyond a segment's
//          ends and in the halo dearer (4 and 6 steps: 2000 x 1000 11.1 and
//          11.9, 4096 x 2048 34.5 and 37.0).  FP32 6 (2000 x 1000 10.5 and
//          10.0), and 7 on the largest, which HBM bounds (6 and 7: 2300 x 2000
//          19.9 and 19.9, 4096 x 2048 38.1 and 34.3).
inline bool clear(int64_t cells, int64_t nonsolid, int nx) {
    return cells - nonsolid - 2 * (int64_t)nx <= cells / 1000;
}
inline MarchRule march_rule(int value_bytes, int64_t cells, int64_t nonsolid, int nx) {
    if (value_bytes == 8) return {500000, 4};
    const int64_t from = clear(cells, nonsolid, nx) ? 1100000 : 2400000;
    if (value_bytes == 2) return {from, 4};
    return {from, cells < (int64_t)4 << 20 ? 6 : 7};
}

// Waves per SIMD of a launch of `steps` steps.  us per step with 2 and 3: FP64
// 1024 x 512 7.7 and 9.6, 2000 x 1000 20.6 and 23.0; FP32, 4 steps, 2000 x 1000
// 10.4 and 11.0, 6 steps 10.0 and 10.2, but with 1 % solid 2000 x 1400 16.9 and
// 15.7 and 2800 x 2000 30.1 and 27.4 (rows on the longer path wait more); FP16,
// 4 steps, 2000 x 1000 11.2 and 11.1, 3000 x 1500 21.2 and 19.6, 2000 x 1400
// with 1 % solid 18.8 and 17.2.
inline int march_fill(int value_bytes, int steps, bool is_clear) {
    if (value_bytes == 8) return 2;
    return (value_bytes == 2 && steps <= 4) || (steps == 6 && !is_clear) ? 3 : 2;
}

}  // namespace lbm
