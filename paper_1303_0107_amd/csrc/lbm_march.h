// The marching sweep: several time steps of a dense lattice in registers.
//
// One wavefront owns a strip of 64 lattice columns (at most 64 - 2S of them its
// own, the others a halo) over a segment of rows, and walks up the rows with
// all S time steps in flight: when row t of the input arrives, step 1 is
// carried out on row t - 1, step 2 on row t - 2, and so on to step S on row
// t - S, which is written out.  Step s of a row needs the rows below, at and
// above it of step s - 1, so each step keeps the last row whole and of the
// one before it the three populations that move up: 12 registers a step.
// Horizontal neighbours are neighbouring lanes.  Nothing goes through LDS,
// no wave waits for another, and each population crosses HBM once per S
// steps; the next row is read a whole iteration (S cell updates) ahead.
//
// What it costs beyond the cell update: six lane shifts per cell, the halo
// lanes (S of 64 on each side) and the rows S - s beyond both ends of the
// segment that step s also has to advance.  The blocked sweep pays for its
// barrier a step (two in place), 16 LDS accesses a cell and a halo on regions
// of 16 or 32 rows; it remains the better one where many cells are solid,
// since it skips the tiles and rows without fluid and shares one region's work
// among sixteen waves.  Which lattices march: march_rule (lbm_march_plan.h).
//
// The cells' arithmetic is the shared Cell policy on the same operands, so
// the populations have the bits of one launch per step.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "lbm_internal.h"
#include "lbm_sweep.h"

namespace lbm {
namespace sweep {

// Lane l reads lane l - 1 (lane 0: zero), and lane l + 1 (lane 63: zero).
__device__ __forceinline__ uint32_t from_left(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x138, 0xf, 0xf, true);  // wave_shr:1
}
__device__ __forceinline__ uint32_t from_right(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x130, 0xf, 0xf, true);  // wave_shl:1
}
template <typename CT, class F>
__device__ __forceinline__ CT by_words(CT v, F f) {
    uint32_t w[sizeof(CT) / 4];
    __builtin_memcpy(w, &v, sizeof v);
#pragma unroll
    for (unsigned k = 0; k < sizeof(CT) / 4; ++k) w[k] = f(w[k]);
    __builtin_memcpy(&v, w, sizeof v);
    return v;
}
// Population i as a cell pulls it from the lane x - c_i.
template <int I, typename CT>
__device__ __forceinline__ CT shifted(CT v) {
    if constexpr (kCx[I] > 0) return by_words(v, [](uint32_t w) { return from_left(w); });
    if constexpr (kCx[I] < 0) return by_words(v, [](uint32_t w) { return from_right(w); });
    return v;
}

// The stored bits (the 16-bit formats are classes, which have no assignment
// outside the generic address space).
template <typename T>
using Bits = typename std::conditional<
    sizeof(T) == 8, uint64_t,
    typename std::conditional<sizeof(T) == 4, uint32_t, uint16_t>::type>::type;

// Element col of a row of global memory whose address p is the same in every
// lane: p in scalar registers, and the 32-bit column added by the access.
template <typename T>
__device__ __forceinline__ T load_at(uint64_t p, uint32_t col) {
    using G = const __attribute__((address_space(1))) Bits<T>;
    const Bits<T> w =
        *(G *)((const __attribute__((address_space(1))) char *)p + col * (uint32_t)sizeof(T));
    T v;
    __builtin_memcpy(&v, &w, sizeof(T));
    return v;
}
// Store v at byte offset `off` of the row of `bytes` bytes at p (the same in
// every lane), or nothing where off == kNoStore: a buffer store drops lanes
// beyond its range.  Lanes are left out that way and not by a branch, because
// a branch around the stores would hide from the compiler how many memory
// operations are in flight, and every wait for a row on its way would become
// a wait for all of them, the stores just issued included.
constexpr uint32_t kNoStore = 0xffffffffu;
template <typename T>
__device__ __forceinline__ void store_in(uint64_t p, uint32_t bytes, uint32_t off, T v) {
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, (int)bytes, 0x00027000);
    if constexpr (sizeof(T) == 8) {
        typedef uint32_t Pair __attribute__((ext_vector_type(2)));
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(Pair, v), rsrc, (int)off, 0, 0);
    } else if constexpr (sizeof(T) == 4) {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(Bits<T>, v), rsrc, (int)off, 0, 0);
    } else {
        __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(Bits<T>, v), rsrc, (int)off, 0, 0);
    }
}
template <typename CT>
__device__ __forceinline__ CT pinned(CT v) {
    asm volatile("" : "+v"(v));
    return v;
}
// A register as it is.
template <typename CT>
__device__ __forceinline__ CT any_value() {
    CT v;
    asm("" : "=v"(v));
    return v;
}
// A value the compiler takes as new here.  Plane strides: as nine
// loop-invariant addresses the planes would not fit the scalar registers.
__device__ __forceinline__ uint64_t opaque(uint64_t v) {
    asm volatile("" : "+s"(v));
    return v;
}

// f(0) .. f(N - 1) with constant arguments.  (Loops over the arrays below
// would be unrolled only after their boundary branches had been merged into
// stores through a selected address, and the arrays would live in memory.)
template <int N, class F>
__device__ __forceinline__ void static_for(F &&f) {
    if constexpr (N > 0) {
        static_for<N - 1>(f);
        f(std::integral_constant<int, N - 1>{});
    }
}

// Wave w of the grid: its strip and rows.  The two edge strips, whose every
// row has inlet, outlet or wall cells and takes the longer path, are cut into
// twice as many segments; their waves come first.
struct MarchWave {
    int strip, y0, y1;
};
__device__ __forceinline__ MarchWave march_wave(const MarchPlan &p, int w, int ny) {
    MarchWave m;
    const int edge = 2 * p.edge_segs;
    if (w < edge) {
        m.strip = w < p.edge_segs ? 0 : p.strips - 1;
        const int k = w < p.edge_segs ? w : w - p.edge_segs;
        m.y0 = k * p.edge_rows;
        m.y1 = min(ny, m.y0 + p.edge_rows);
    } else {
        const int k = w - edge;
        m.strip = 1 + k / p.segs;
        m.y0 = (k % p.segs) * p.rows;
        m.y1 = min(ny, m.y0 + p.rows);
    }
    if (w >= p.waves) m.y1 = m.y0 = 0;  // padding of the last workgroup
    return m;
}

template <class Cell, int S, bool CHECK>
__global__ __launch_bounds__(kMarchThreads, march_waves(S, sizeof(typename Cell::CT), CHECK)) void march_kernel(const int *__restrict__ stop,
                                                              MarchPlan plan,
                                                              SweepArgs<typename Cell::T> a) {
    using T = typename Cell::T;
    using CT = typename Cell::CT;
    const int lane = threadIdx.x & 63;
    if (__builtin_amdgcn_readfirstlane(stop[lane])) return;  // the run has ended (all lanes alike)

    // Workgroup g runs on XCD g mod 8: each XCD takes one contiguous run of
    // the waves, so that strips and segments that share halo cells mostly
    // read them through one L2.
    const int nb = gridDim.x, xcd = blockIdx.x & 7, per = nb >> 3, rest = nb & 7;
    const int g = xcd * per + min(xcd, rest) + (int)(blockIdx.x >> 3);
    const int w = __builtin_amdgcn_readfirstlane(g * (kMarchThreads / 64) + (threadIdx.x >> 6));
    const MarchWave m = march_wave(plan, w, a.ny);
    const int y0 = m.y0, y1 = m.y1;

    const int gx = m.strip * plan.width - S + lane;
    const bool col_in = gx >= 0 && gx < a.nx;
    const uint32_t col = col_in ? (uint32_t)gx : 0u;
    const bool own = lane >= S && lane < S + plan.width && col_in;
    const int lo = max(0, y0 - S), hi = min(a.ny, y1 + S);  // rows to read

    // Slots of step s - 1's rows as step s sees them in phase p: row y + 1 in
    // slot p, row y in slot p + 2, row y - 1 in slot p + 1 (mod 3).
    CT r[S][3][9];
    // Cell words of the last 16 rows (the boundary path's only, so they keep
    // no registers): written and read by the same lane.
    __shared__ uint16_t s_words[kMarchThreads / 64][16][64];
    uint16_t(&words)[16][64] = s_words[threadIdx.x >> 6];
    uint32_t plain = 0;         // bit s: row t - s holds only fluid cells without walls
    T raw[3][9];                // rows on their way: row t of phase t mod 3
    uint32_t raw_word[3];
    CT uv = CT(0);              // inlet velocities of rows uv_base + lane (strip 0)
    int uv_base = -(1 << 20);
    double part[4] = {0.0, 0.0, 0.0, 0.0};

    static_for<S * 27>([&](auto j) { r[j / 27][j / 9 % 3][j % 9] = CT(0); });

    // Rows outside [lo, hi) are not used: row lo or hi - 1 is read instead, so
    // that every iteration issues the same loads.
    auto fetch = [&](auto slot, const int row) {
        constexpr int Q = decltype(slot)::value;
        const size_t at = (size_t)min(max(row, lo), hi - 1) * a.pitch;
        raw_word[Q] = load_at<uint16_t>((uint64_t)(a.cell + at), col);
        const uint64_t stride = opaque(a.plane * sizeof(T));
        uint64_t p = (uint64_t)(a.fin + at);
        static_for<9>([&](auto i) {
            raw[Q][i] = load_at<T>(p, col);
            p += stride;
        });
    };

    // One iteration: row t arrives.  The first 2 S iterations of a segment
    // (warm) fill the steps up, step s from the row S - s below the segment
    // on; after them every step advances a row and the last one writes it.
    auto iteration = [&](auto warming, auto phase, const int t) {
        constexpr bool WARM = decltype(warming)::value;
        constexpr int P = decltype(phase)::value, C = (P + 2) % 3, O = (P + 1) % 3;
        static_for<9>([&](auto i) { r[0][P][i] = Cell::load(raw[P][i]); });
        const uint32_t word = col_in && t >= lo && t < hi ? raw_word[P] : 0u;  // here: the load is waited for now
        words[t & 15][lane] = (uint16_t)word;
        plain = (plain << 1) | (__all(word == (kFluid << 8)) ? 1u : 0u);
        if (m.strip == 0 && t - 1 - uv_base > 63) {
            uv_base = t - S;
            uv = (CT)a.uin[min(max(uv_base + lane, 0), a.ny - 1)];
            asm volatile("" : "+v"(uv));  // waited for here, not at each use
        }
        static_for<S>([&](auto step) {
            constexpr int s = decltype(step)::value + 1;
            const int y = t - s;
            if (!WARM || (s < S && y >= max(0, y0 - (S - s)))) {
                const CT(&nw)[9] = r[s - 1][P];
                const CT(&cu)[9] = r[s - 1][C];
                const CT(&od)[9] = r[s - 1][O];
                CT f[9] = {cu[0], shifted<1>(cu[1]), od[2], shifted<3>(cu[3]), nw[4],
                           shifted<5>(od[5]), shifted<6>(od[6]), shifted<7>(nw[7]),
                           shifted<8>(nw[8])};
                bool live = own;
                if (!((plain >> s) & 1u)) {
                    const uint32_t cw = words[y & 15][lane];
                    static_for<8>([&](auto j) {
                        constexpr int i = decltype(j)::value + 1;
                        f[i] = ((cw >> (i - 1)) & 1u) ? cu[kOpp[i]] : f[i];
                    });
                    const uint32_t type = cell_type(cw);
                    const CT u = m.strip == 0 ? by_words(uv, [&](uint32_t x) {
                        return (uint32_t)__builtin_amdgcn_readlane((int)x, y - uv_base);
                    }) : CT(0);
                    // by selects: stores under branches would be merged into
                    // stores through a selected address
                    CT k1 = f[1], k2 = f[5], k3 = f[8];
                    if (type == kInlet) Cell::inlet(f, u, k1, k2, k3);
                    CT q1 = f[3], q2 = f[7], q3 = f[6];
                    if (type == kOutlet) Cell::outlet(f, a, q1, q2, q3);
                    f[1] = k1;
                    f[5] = k2;
                    f[8] = k3;
                    f[3] = q1;
                    f[7] = q2;
                    f[6] = q3;
                    live = own && type != kSolid;
                }
                double mass, ux, uy;
                Cell::relax(f, a, mass, ux, uy);
                if constexpr (s < S) {
                    // each value is made opaque: moved across the steps by the
                    // compiler, their parts held 50 registers more
                    static_for<9>([&](auto i) {
                        r[s][P][i] = pinned(Cell::load(Cell::store(f[i])));
                    });
                } else if constexpr (!WARM) {
                    live = live && y < y1;
                    const uint64_t stride = opaque(a.plane * sizeof(T));
                    uint64_t p = (uint64_t)(a.fout + (size_t)y * a.pitch);
                    const uint32_t off = live ? col * (uint32_t)sizeof(T) : kNoStore;
                    static_for<9>([&](auto i) {
                        store_in(p, (uint32_t)a.pitch * (uint32_t)sizeof(T), off,
                                 Cell::store(f[i]));
                        p += stride;
                    });
                    if (CHECK && live)
                        check_terms(a, (size_t)y * a.pitch + col, mass, ux, uy, part);
                }
            } else if constexpr (s < S) {
                // any value: the slot's old row need not be kept
                static_for<9>([&](auto i) { r[s][P][i] = any_value<CT>(); });
            }
            if constexpr (s == 1) fetch(std::integral_constant<int, (P + 2) % 3>{}, t + 2);
        });
    };

    if (y1 > y0) {
        const std::integral_constant<int, 0> p0;
        const std::integral_constant<int, 1> p1;
        const std::integral_constant<int, 2> p2;
        const int steady = y0 + S, last = y1 - 1 + S;
        int t = steady - (steady - lo + 2) / 3 * 3;  // whole turns of the three phases
        fetch(p0, t);
        fetch(p1, t + 1);
        for (; t < steady; t += 3) {
            iteration(std::true_type{}, p0, t);
            iteration(std::true_type{}, p1, t + 1);
            iteration(std::true_type{}, p2, t + 2);
        }
        for (;; t += 3) {
            iteration(std::false_type{}, p0, t);
            if (t + 1 > last) break;
            iteration(std::false_type{}, p1, t + 1);
            if (t + 2 > last) break;
            iteration(std::false_type{}, p2, t + 2);
            if (t + 3 > last) break;
        }
    }
    if (CHECK) {
        block_sum<4, kMarchThreads>(part);
        if (threadIdx.x == 0) {
            double *out = a.partials + (size_t)blockIdx.x * 4;
#pragma unroll
            for (int k = 0; k < 4; ++k) out[k] = part[k];
        }
    }
}

template <class Cell, int S>
hipError_t launch_march_steps(const SweepArgs<typename Cell::T> &a, const MarchPlan &p,
                              bool check, hipStream_t s) {
    const dim3 grid((unsigned)p.blocks), block(kMarchThreads);
    if (check)
        hipLaunchKernelGGL((march_kernel<Cell, S, true>), grid, block, 0, s, a.stop, p, a);
    else
        hipLaunchKernelGGL((march_kernel<Cell, S, false>), grid, block, 0, s, a.stop, p, a);
    return hipGetLastError();
}

template <class Cell>
hipError_t launch_march(const SweepArgs<typename Cell::T> &a, const MarchPlan &p, bool check,
                        hipStream_t s) {
    if (a.flags != 0 || !a.stop) return hipErrorInvalidValue;
    switch (p.steps) {
        case 1: return launch_march_steps<Cell, 1>(a, p, check, s);
        case 2: return launch_march_steps<Cell, 2>(a, p, check, s);
        case 4: return launch_march_steps<Cell, 4>(a, p, check, s);
    }
    if constexpr (sizeof(typename Cell::CT) == 4) {  // in double the registers end at 4
        if (p.steps == 6) return launch_march_steps<Cell, 6>(a, p, check, s);
        if (p.steps == 7) return launch_march_steps<Cell, 7>(a, p, check, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace sweep
}  // namespace lbm
