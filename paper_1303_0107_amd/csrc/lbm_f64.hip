// Double-precision kernels of the D2Q9 sweep, in the reference arithmetic
// form: populations stored as full f_i (post-collision), and every
// floating-point expression evaluated in the order the method's definition
// writes it (moments summed in population order, equilibrium of Sec. 2.1
// expanded as written, relaxation f - (1/tau)(f - feq) of Eq. 1, Zou-He
// closures as printed).  This file is compiled with -ffp-contract=off, so no
// multiply-add is fused and each operation rounds once, as IEEE-754 double
// arithmetic on any conforming machine does: results are reproducible bit
// for bit.  Wang, Fan & Luo, Sec. 2.1 (Eqs. 1-2), Sec. 3.3 (boundaries),
// Sec. 4.2 (Eqs. 9-11), Eq. 4.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lbm_boundary.h"
#include "lbm_internal.h"
#include "lbm_keys.h"

#pragma clang fp contract(off)

#include "lbm_march.h"
#include "lbm_sweep.h"

namespace lbm {
namespace f64 {

__device__ constexpr int kCx[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
__device__ constexpr int kCy[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
__device__ constexpr int kOpp[9] = {0, 3, 4, 1, 2, 7, 8, 5, 6};

__device__ __forceinline__ double weight(int i) {
    return i == 0 ? 4.0 / 9.0 : (i < 5 ? 1.0 / 9.0 : 1.0 / 36.0);
}

// rho = sum f_i, j = sum c_i f_i (Eq. 2), each summed in population order.
__device__ __forceinline__ void moments(const double (&f)[9], double &r,
                                        double &mx, double &my) {
    r = 0.0;
    mx = 0.0;
    my = 0.0;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        r += f[i];
        mx += kCx[i] * f[i];
        my += kCy[i] * f[i];
    }
}

// Density and velocity of cell n (pitched) of the stored state: the
// macroscopic export and the exchange-step keys both use this.
struct Moments {
    using T = double;
    __device__ static __forceinline__ void at(const double *f, size_t plane, size_t n,
                                              double &r, double &ux, double &uy) {
        double g[9], mx, my;
#pragma unroll
        for (int i = 0; i < 9; ++i) g[i] = f[(size_t)i * plane + n];
        moments(g, r, mx, my);
        ux = mx / r;
        uy = my / r;
    }
};

template <int NV>
__device__ __forceinline__ void block_sum(double (&v)[NV], int tid) {
    __shared__ double red[4][NV];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
#pragma unroll
        for (int k = 0; k < NV; ++k) v[k] += __shfl_xor(v[k], off, 64);
    if ((tid & 63) == 0)
#pragma unroll
        for (int k = 0; k < NV; ++k) red[tid >> 6][k] = v[k];
    __syncthreads();
    if (tid == 0)
#pragma unroll
        for (int k = 0; k < NV; ++k) v[k] = ((red[0][k] + red[1][k]) + red[2][k]) + red[3][k];
}

// a / r and b / r, rounded as the divisions round them, with one reciprocal:
// Newton steps bring the hardware estimate of 1/r within an ulp, and one
// exact-remainder correction then rounds each quotient correctly (Markstein,
// IBM J. Res. Dev. 34, 1990).  Where r is far from 1 the remainder or the
// reciprocal could leave the normal range, so those waves divide.  A quotient
// below 2^-500 may differ in its last place; it is lost entirely in the sums
// 1 + 3 c.u and in the squares it enters.  Eleven instructions for the pair,
// the two divisions take 22.  (Lanes relaxed without a cell of their own are
// kept near rest, so that they do not decide the vote.)
__device__ __forceinline__ void divide_pair(double a, double b, double r, double &qa,
                                            double &qb) {
    // biased exponent of r within 512 of that of 1, and r positive
    const uint32_t hi = (uint32_t)((uint64_t)__double_as_longlong(r) >> 32);
    if (__builtin_expect(__any(hi - (511u << 20) >= (1024u << 20)), 0)) {
        qa = a / r;
        qb = b / r;
        return;
    }
    double y = __builtin_amdgcn_rcp(r);
    y = __builtin_fma(__builtin_fma(-r, y, 1.0), y, y);
    y = __builtin_fma(__builtin_fma(-r, y, 1.0), y, y);
    qa = a * y;
    qb = b * y;
    qa = __builtin_fma(__builtin_fma(-r, qa, a), y, qa);
    qb = __builtin_fma(__builtin_fma(-r, qb, b), y, qb);
}

// One cell of one time step on full populations: Zou-He closure on inlet
// (velocity u_in, unknowns 1, 5, 8) and outlet cells (density rho_out, zero
// transverse velocity, unknowns 3, 6, 7), moments (Eq. 2), relaxation
// f - (1/tau)(f - feq) (Eq. 1) to the equilibrium of Sec. 2.1.
struct Cell {
    using T = double;
    using CT = ArithT<double>;
    static constexpr bool kOffsets = false;
    __device__ static __forceinline__ double load(double v) { return v; }
    __device__ static __forceinline__ double store(double v) { return v; }
    // Velocity (Eq. 2) of a stored population set, formed as the oracle does.
    __device__ static __forceinline__ void velocity(double (&g)[9], double &ux, double &uy) {
        double r, mx, my;
        moments(g, r, mx, my);
        ux = mx / r;
        uy = my / r;
    }
    // Zou-He closures: the three unknown populations, 1, 5, 8 of an inlet
    // cell (velocity bx) and 3, 7, 6 of an outlet cell (fixed density, or the
    // velocity (bx, by) of its x-1 neighbour's stored state).
    __device__ static __forceinline__ void inlet(const double (&f)[9], double bx, double &k1,
                                                 double &k5, double &k8) {
        const double rho = (f[0] + f[2] + f[4] + 2.0 * (f[3] + f[6] + f[7])) / (1.0 - bx);
        const double ru = rho * bx;
        k1 = f[3] + (2.0 / 3.0) * ru;
        k5 = f[7] - 0.5 * (f[2] - f[4]) + (1.0 / 6.0) * ru;
        k8 = f[6] + 0.5 * (f[2] - f[4]) + (1.0 / 6.0) * ru;
    }
    __device__ static __forceinline__ void outlet(const double (&f)[9], const SweepArgs<double> &a,
                                                  double &k3, double &k7, double &k6) {
        const double uo = -1.0 + (f[0] + f[2] + f[4] + 2.0 * (f[1] + f[5] + f[8])) / a.rho_out;
        const double ru = a.rho_out * uo;
        k3 = f[1] - (2.0 / 3.0) * ru;
        k7 = f[5] + 0.5 * (f[2] - f[4]) - (1.0 / 6.0) * ru;
        k6 = f[8] - 0.5 * (f[2] - f[4]) - (1.0 / 6.0) * ru;
    }
    __device__ static __forceinline__ void neumann(const double (&f)[9], double bx, double by,
                                                   double &k3, double &k7, double &k6) {
        const double rho = (f[0] + f[2] + f[4] + 2.0 * (f[1] + f[5] + f[8])) / (1.0 + bx);
        const double ru = rho * bx, rv = rho * by;
        k3 = f[1] - (2.0 / 3.0) * ru;
        k7 = f[5] + 0.5 * (f[2] - f[4]) - (1.0 / 6.0) * ru - 0.5 * rv;
        k6 = f[8] - 0.5 * (f[2] - f[4]) - (1.0 / 6.0) * ru + 0.5 * rv;
    }
    __device__ static __forceinline__ void update(double (&f)[9], uint32_t type, double bx,
                                                  double by, const SweepArgs<double> &a,
                                                  double &mass, double &ux, double &uy) {
        closure(f, type, bx, by, a);
        relax(f, a, mass, ux, uy);
    }
    __device__ static __forceinline__ void closure(double (&f)[9], uint32_t type, double bx,
                                                   double by, const SweepArgs<double> &a) {
        if (type == kInlet)
            inlet(f, bx, f[1], f[5], f[8]);
        else if (type == kOutlet)
            outlet(f, a, f[3], f[7], f[6]);
        else if (type == kOutletNeumann)
            neumann(f, bx, by, f[3], f[7], f[6]);
    }
    __device__ static __forceinline__ void relax(double (&f)[9], const SweepArgs<double> &a,
                                                 double &mass, double &ux, double &uy) {
        // Moments and relaxation in the definition's order, without the
        // operations that cannot change a result: terms with a zero velocity
        // component are left out, opposite populations share 3 c.u and
        // 4.5 (c.u)^2 (their c.u differ in sign alone), and 0.5 x 9 and
        // 0.5 x 3 are one product (halving is exact).  Every population keeps
        // the bits of the expressions as the definition writes them.  With
        // the shared reciprocal 117 vector instructions a cell in place of
        // 205; 1024 x 512 distributor, 4000 steps: 15.2 -> 13.0 ms (in-place
        // regions, whose pulls also lost their address arithmetic).
        const double r = f[0] + f[1] + f[2] + f[3] + f[4] + f[5] + f[6] + f[7] + f[8];
        const double mx = f[1] - f[3] + f[5] - f[6] - f[7] + f[8];
        const double my = f[2] - f[4] + f[5] + f[6] - f[7] - f[8];
        divide_pair(mx, my, r, ux, uy);
        const double v = 1.5 * (ux * ux + uy * uy), om = a.omega;
        const double w0 = weight(0) * r, w1 = weight(1) * r, w5 = weight(5) * r;
        f[0] = f[0] - om * (f[0] - w0 * (1.0 - v));
        auto relax_pair = [&](int i, int j, double cu, double w) {  // c_j = -c_i
            const double c3 = cu * 3.0, s = 4.5 * (cu * cu);
            f[i] = f[i] - om * (f[i] - w * (1.0 + c3 + s - v));
            f[j] = f[j] - om * (f[j] - w * (1.0 - c3 + s - v));
        };
        relax_pair(1, 3, ux, w1);
        relax_pair(2, 4, uy, w1);
        relax_pair(5, 7, ux + uy, w5);
        relax_pair(8, 6, ux - uy, w5);
        mass = r;
    }
};

__global__ __launch_bounds__(256) void macro_kernel(MacroArgs<double> a) {
    const int x = blockIdx.x * 64 + threadIdx.x;
    const int y = blockIdx.y * 4 + threadIdx.y;
    if (x >= a.nx || y >= a.ny) return;
    const size_t n = (size_t)y * a.pitch + x;
    const size_t l = (size_t)y * a.nx + x;
    double r = 0.0, ux = 0.0, uy = 0.0;
    if (cell_type(a.cell[n]) != kSolid) Moments::at(a.f, a.plane, n, r, ux, uy);
    if (a.rho) {
        a.rho[l] = r;
        a.ux[l] = ux;
        a.uy[l] = uy;
    }
    if (a.uprev) {
        a.uprev[n] = ux;
        a.uprev[a.plane + n] = uy;
    }
}

__global__ __launch_bounds__(256) void mass_kernel(MacroArgs<double> a,
                                                   double *partials) {
    const int x = blockIdx.x * 64 + threadIdx.x;
    const int y = blockIdx.y * 4 + threadIdx.y;
    double v[1] = {0.0};
    if (x < a.nx && y < a.ny) {
        const size_t n = (size_t)y * a.pitch + x;
        if (cell_type(a.cell[n]) != kSolid) {
            double f[9], mx, my;
#pragma unroll
            for (int i = 0; i < 9; ++i) f[i] = a.f[(size_t)i * a.plane + n];
            moments(f, v[0], mx, my);
        }
    }
    const int tid = threadIdx.y * 64 + threadIdx.x;
    block_sum<1>(v, tid);
    if (tid == 0) partials[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = v[0];
}

// Boundary sums (lbm_boundary.h) of the stored state (a.fin) and of the state
// one step later; out: the stored state's 2 n_out + 5 sums, then the later's.
template <bool BC>
__global__ __launch_bounds__(kBoundaryThreads) void boundary_kernel(SweepArgs<double> a,
                                                                    const int32_t *out_y0,
                                                                    const int32_t *out_y1,
                                                                    int n_out, double *out) {
    if (blockIdx.y == 0)
        boundary_sums(a.cell, a.nx, a.ny, a.pitch, out_y0, out_y1, n_out, out,
                      [&](int x, int y, double &r, double &mx) {
                          const size_t n = (size_t)y * a.pitch + x;
                          double f[9], my;
#pragma unroll
                          for (int i = 0; i < 9; ++i) f[i] = a.fin[(size_t)i * a.plane + n];
                          moments(f, r, mx, my);
                      });
    else
        boundary_sums(a.cell, a.nx, a.ny, a.pitch, out_y0, out_y1, n_out, out + 2 * n_out + 5,
                      [&](int x, int y, double &r, double &mx) {
                          double f[9], m, ux, uy, my;
                          sweep::step_cell<Cell, BC>(a, x, y, a.cell[(size_t)y * a.pitch + x], f,
                                                     m, ux, uy);
                          moments(f, r, mx, my);
                      });
}

__global__ void rest_cells_kernel(double *f, size_t plane, const int32_t *cells,
                                  int count, int nx, int pitch) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= count) return;
    const int l = cells[k];
    const size_t n = (size_t)(l / nx) * pitch + (l % nx);
#pragma unroll
    for (int i = 0; i < 9; ++i) f[(size_t)i * plane + n] = weight(i);
}

__global__ void rest_all_kernel(double *f, size_t plane) {
    for (size_t j = (size_t)blockIdx.x * blockDim.x + threadIdx.x; j < plane;
         j += (size_t)gridDim.x * blockDim.x)
#pragma unroll
        for (int i = 0; i < 9; ++i) f[(size_t)i * plane + j] = weight(i);
}

__global__ __launch_bounds__(256) void export_plane_kernel(
    const double *f, const uint16_t *cell, double *out, int i, int nx, int ny,
    int pitch, size_t plane) {
    const int x = blockIdx.x * 64 + threadIdx.x;
    const int y = blockIdx.y * 4 + threadIdx.y;
    if (x >= nx || y >= ny) return;
    const size_t n = (size_t)y * pitch + x;
    out[(size_t)y * nx + x] = cell_type(cell[n]) == kSolid ? 0.0 : f[(size_t)i * plane + n];
}

__global__ __launch_bounds__(256) void import_plane_kernel(
    double *f, const uint16_t *cell, const double *in, int i, int nx, int ny,
    int pitch, size_t plane) {
    const int x = blockIdx.x * 64 + threadIdx.x;
    const int y = blockIdx.y * 4 + threadIdx.y;
    if (x >= nx || y >= ny) return;
    const size_t n = (size_t)y * pitch + x;
    f[(size_t)i * plane + n] = cell_type(cell[n]) == kSolid ? weight(i) : in[(size_t)y * nx + x];
}

}  // namespace f64

static inline dim3 grid_cells(int ncols, int ny) {
    return dim3((unsigned)((ncols + 63) / 64), (unsigned)((ny + 3) / 4));
}

template <>
hipError_t launch_sweep<double>(const SweepArgs<double> &a, bool check, hipStream_t s) {
    return sweep::launch_step<f64::Cell>(a, check, s);
}

template <>
hipError_t launch_tb<double>(const SweepArgs<double> &a, const int32_t *tiles, int n_tiles,
                             int steps, bool check, int variant, hipStream_t s) {
    return sweep::launch_tb_variant<f64::Cell>(a, tiles, n_tiles, steps, check, variant, s);
}

template <>
hipError_t launch_tb_batch<double>(const SweepArgs<double> *args, const int32_t *lat,
                                   const int32_t *tiles, int n_items, int steps, int variant,
                                   bool bc, hipStream_t s) {
    return sweep::launch_tb_batch_variant<f64::Cell>(args, lat, tiles, n_items, steps, variant,
                                                     bc, s);
}

template <>
hipError_t launch_step_batch<double>(const SweepArgs<double> *args, const int32_t *lat,
                                     const int32_t *blocks, int n_items, bool bc,
                                     hipStream_t s) {
    return sweep::launch_step_batch<f64::Cell>(args, lat, blocks, n_items, bc, s);
}

template <>
hipError_t launch_march<double>(const SweepArgs<double> &a, const MarchPlan &p, bool check,
                                hipStream_t s) {
    return sweep::launch_march<f64::Cell>(a, p, check, s);
}

template <>
hipError_t launch_macro<double>(const MacroArgs<double> &a, hipStream_t s) {
    hipLaunchKernelGGL(f64::macro_kernel, grid_cells(a.nx, a.ny), dim3(64, 4), 0, s, a);
    return hipGetLastError();
}

template <>
hipError_t launch_keys<double>(const KeysArgs &a, hipStream_t s) {
    return keys::launch_keys<f64::Moments>(a, s);
}

template <>
hipError_t launch_flip<double>(const FlipArgs &a, hipStream_t s) {
    return keys::launch_flip<f64::Moments>(a, s);
}

template <>
hipError_t launch_mass<double>(const MacroArgs<double> &a, double *partials,
                               hipStream_t s) {
    hipLaunchKernelGGL(f64::mass_kernel, grid_cells(a.nx, a.ny), dim3(64, 4), 0, s, a,
                       partials);
    return hipGetLastError();
}

template <>
hipError_t launch_boundary<double>(const SweepArgs<double> &a, const int32_t *y0,
                                   const int32_t *y1, int n_out, double *out, hipStream_t s) {
    const dim3 g((unsigned)(n_out + 1), 2), b(kBoundaryThreads);
    if (a.flags)
        hipLaunchKernelGGL(f64::boundary_kernel<true>, g, b, 0, s, a, y0, y1, n_out, out);
    else
        hipLaunchKernelGGL(f64::boundary_kernel<false>, g, b, 0, s, a, y0, y1, n_out, out);
    return hipGetLastError();
}

template <>
hipError_t launch_rest_cells<double>(double *f, size_t plane, const int32_t *cells,
                                     int count, int nx, int pitch, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(f64::rest_cells_kernel, dim3((count + 255) / 256), dim3(256), 0, s,
                       f, plane, cells, count, nx, pitch);
    return hipGetLastError();
}

template <>
hipError_t launch_rest_all<double>(double *f, size_t plane, hipStream_t s) {
    size_t blocks = (plane + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(f64::rest_all_kernel, dim3((unsigned)blocks), dim3(256), 0, s, f,
                       plane);
    return hipGetLastError();
}

template <>
hipError_t launch_export_plane<double>(const double *f, const uint16_t *cell, double *out,
                                       int i, int nx, int ny, int pitch, size_t plane,
                                       hipStream_t s) {
    hipLaunchKernelGGL(f64::export_plane_kernel, grid_cells(nx, ny), dim3(64, 4), 0, s, f,
                       cell, out, i, nx, ny, pitch, plane);
    return hipGetLastError();
}

template <>
hipError_t launch_import_plane<double>(double *f, const uint16_t *cell, const double *in,
                                       int i, int nx, int ny, int pitch, size_t plane,
                                       hipStream_t s) {
    hipLaunchKernelGGL(f64::import_plane_kernel, grid_cells(nx, ny), dim3(64, 4), 0, s, f,
                       cell, in, i, nx, ny, pitch, plane);
    return hipGetLastError();
}

}  // namespace lbm
