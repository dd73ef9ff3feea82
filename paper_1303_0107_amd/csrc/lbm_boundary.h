// The boundary sums of the outlet statistics (Sec. 2.3 step 5, Eqs. 9-11; the
// pressure drop of Eq. 4), shared by the storage forms.
//
// One launch sums over the stored state and over the state one time step
// later.  Only the boundary columns of the later state are needed, so their
// cells take the step here, from the stored state, and nothing is written
// back.  Workgroup (k, s) of the grid (n_out + 1, 2): outlet k (k < n_out) or
// the ends (k == n_out: the inlet cells and all outlet cells) of state s.
//
// Every sum is a running sum in increasing y, the order of a sequential loop
// over the rows.  What bounds it is that chain of double additions, so the
// rows' values are first read by all lanes at once, and then one wave adds
// 64 of them at a time, taking lane after lane as a scalar operand: three
// instructions a row, none of them waiting for memory.  Rows without a
// boundary cell add 0.0, which leaves the sum as it is, and 64 rows without
// any are passed over.  The three sums of the ends run in three waves.
// Before, each state had a launch of its own (18-160 us), with the rows'
// values taken from LDS one by one in a single thread and a whole time step in
// between: a call of lbm_outlet_stats on the 1024 x 512 FP32 distributor takes
// 38 us in place of 82, on the 2048 x 1024 one 64 in place of 149, on the 128
// x 64 one 24 in place of 35.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lbm_internal.h"

namespace lbm {

constexpr int kBoundaryThreads = 256, kBoundaryRowsPerThread = 4,
              kBoundarySpan = kBoundaryThreads * kBoundaryRowsPerThread;

// sum + v of lane 0 + v of lane 1 + ... + v of lane m - 1, one after another.
__device__ __forceinline__ double add_lanes(double sum, double v, int m) {
    const uint64_t w = (uint64_t)__double_as_longlong(v);
    const int lo = (int)(uint32_t)w, hi = (int)(uint32_t)(w >> 32);
    auto lane = [&](int t) {
        const uint64_t b = (uint64_t)(uint32_t)__builtin_amdgcn_readlane(lo, t) |
                           ((uint64_t)(uint32_t)__builtin_amdgcn_readlane(hi, t) << 32);
        return __longlong_as_double((long long)b);
    };
    if (m == 64) {
#pragma unroll 16
        for (int t = 0; t < 64; ++t) sum += lane(t);
    } else {
        for (int t = 0; t < m; ++t) sum += lane(t);
    }
    return sum;
}

// at(x, y, rho, jx): density and x momentum of the boundary cell (x, y).
// out: [flow_0 .. flow_{n-1}, rho_0 .. rho_{n-1}, flow_in, rho_in, count_in,
//       count_out, rho_out]
template <class At>
__device__ __forceinline__ void boundary_sums(const uint16_t *cell, int nx, int ny, int pitch,
                                              const int32_t *out_y0, const int32_t *out_y1,
                                              int n_out, double *out, At at) {
    const int k = blockIdx.x, t = threadIdx.x, lane = t & 63, wave = t >> 6;
    if (k < n_out) {
        if (t >= 64) return;  // one wave per outlet
        const int y0 = out_y0[k], y1 = out_y1[k];
        double fl = 0.0, rs = 0.0;
        for (int c = y0; c <= y1; c += 64) {
            double r = 0.0, j = 0.0;
            if (c + lane <= y1) at(nx - 1, c + lane, r, j);
            const int m = min(64, y1 - c + 1);
            fl = add_lanes(fl, j, m);
            rs = add_lanes(rs, r, m);
        }
        if (lane == 0) {
            out[k] = fl;
            out[n_out + k] = rs;
        }
        return;
    }
    __shared__ double s_v[3][kBoundarySpan];  // outlet rho, inlet rho, inlet jx of each row
    double sum = 0.0;
    int64_t count = 0;
    for (int c0 = 0; c0 < ny; c0 += kBoundarySpan) {
        // The cell words of all of a thread's rows first, then their
        // populations.  Rows that hold no boundary cell are not read.
        bool is_out[kBoundaryRowsPerThread], is_in[kBoundaryRowsPerThread];
#pragma unroll
        for (int q = 0; q < kBoundaryRowsPerThread; ++q) {
            const int y = c0 + q * kBoundaryThreads + t;
            const size_t n0 = (size_t)min(y, ny - 1) * pitch;
            is_out[q] = (y < ny) & (cell_type(cell[n0 + nx - 1]) == kOutlet);
            is_in[q] = (y < ny) & (cell_type(cell[n0]) == kInlet);
        }
#pragma unroll
        for (int q = 0; q < kBoundaryRowsPerThread; ++q) {
            const int r = q * kBoundaryThreads + t;
            double ro = 0.0, jo, ri = 0.0, ji = 0.0;
            if (is_out[q]) at(nx - 1, c0 + r, ro, jo);
            if (is_in[q]) at(0, c0 + r, ri, ji);
            s_v[0][r] = ro;
            s_v[1][r] = ri;
            s_v[2][r] = ji;
        }
        __syncthreads();
        if (wave < 3) {
            const int m = min(kBoundarySpan, ny - c0);
            for (int r = 0; r < m; r += 64) {
                const int y = c0 + r + lane;
                const size_t n0 = (size_t)min(y, ny - 1) * pitch;
                const bool has = (y < ny) & (wave == 0 ? cell_type(cell[n0 + nx - 1]) == kOutlet
                                                       : cell_type(cell[n0]) == kInlet);
                const uint64_t any = __ballot(has);
                if (any == 0) continue;
                count += __popcll(any);
                sum = add_lanes(sum, has ? s_v[wave][r + lane] : 0.0, 64);
            }
        }
        __syncthreads();
    }
    if (lane == 0 && wave < 3) {
        double *o = out + 2 * n_out;  // flow_in, rho_in, count_in, count_out, rho_out
        o[wave == 0 ? 4 : wave == 1 ? 1 : 0] = sum;
        if (wave == 0) o[3] = (double)count;
        if (wave == 1) o[2] = (double)count;
    }
}

}  // namespace lbm
