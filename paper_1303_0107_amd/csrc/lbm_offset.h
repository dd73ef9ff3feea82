// The offset forms' cell policy: one cell of one time step in single precision
// (or 16-bit storage with float arithmetic), shared by every sweep kernel.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lbm_internal.h"

namespace lbm {

// Reciprocal for the per-cell arithmetic: in float the hardware reciprocal
// refined by one Newton step, r + r (1 - x r) (the raw estimate's error has
// a sign bias that the flux split between outlets integrates); in double
// the division.  The same in every kernel.
__device__ __forceinline__ float recip(float x) {
    const float r = __builtin_amdgcn_rcpf(x);
    return __builtin_fmaf(__builtin_fmaf(-x, r, 1.0f), r, r);
}
__device__ __forceinline__ double recip(double x) { return 1.0 / x; }

// One cell of one time step on offsets d_i = f_i - w_i stored as T (float,
// or 16-bit for the reduced-storage forms), arithmetic in CT (all
// forms: float).  The relaxation restores exact mass
// and momentum conservation after rounding (see update); without that, the
// rounded weights bias every step the same way and float arithmetic, not
// the storage, dominated the error of steady fields.  Zou-He closure on inlet
// (velocity u_in, unknowns 1, 5, 8) and outlet cells (density rho_out, zero
// transverse velocity, unknowns 3, 6, 7), moments (Eq. 2), BGK relaxation
// (Eq. 1) to the equilibrium of Sec. 2.1 written for offsets:
// feq_i - w_i = w_i (drho + rho (3 c.u + 4.5 (c.u)^2 - 1.5 u.u)).  Every sum
// pairs the populations that a reflection y -> -y exchanges (2<->4, 5<->8,
// 6<->7) and every product maps to itself or its exact negative under it, so
// on a mirror-symmetric lattice the computed flow is mirror-symmetric bit for
// bit.  Multiply-adds are fused only inside one expression, as written, so
// every kernel that inlines this function rounds identically.
template <typename Storage, typename Arith>
struct OffsetCell {
    using T = Storage;
    using CT = Arith;
    static constexpr bool kOffsets = true;
    __device__ static __forceinline__ CT load(T v) { return (CT)Sto<T>::to_d(v); }
    __device__ static __forceinline__ CT load_f(T v) { return (CT)Sto<T>::to_f(v); }
    __device__ static __forceinline__ T store(CT v) {
        if constexpr (sizeof(CT) == 8)
            return Sto<T>::from_d((double)v);
        else
            return Sto<T>::from_f((float)v);
    }
    // Velocity (Eq. 2) of a stored offset set, with the update's pairing.
    __device__ static __forceinline__ void velocity(const CT (&d)[9], CT &ux, CT &uy) {
        const CT dr = ((d[0] + (d[1] + d[3])) + (d[2] + d[4])) + ((d[5] + d[8]) + (d[6] + d[7]));
        const CT jx = (d[1] + (d[5] + d[8])) - (d[3] + (d[6] + d[7]));
        const CT jy = (d[2] + (d[5] + d[6])) - (d[4] + (d[8] + d[7]));
        const CT ir = recip(CT(1) + dr);
        ux = jx * ir;
        uy = jy * ir;
    }
    __device__ static __forceinline__ void update(CT (&d)[9], uint32_t type, CT bx, CT by,
                                                  const SweepArgs<T> &a, double &mass,
                                                  double &ux_out, double &uy_out) {
        closure(d, type, bx, by, a);
        relax(d, a, mass, ux_out, uy_out);
    }
    // Zou-He closures: the three unknown populations, 1, 5, 8 of an inlet
    // cell (velocity bx) and 3, 7, 6 of an outlet cell (fixed density, or the
    // velocity (bx, by) of its x-1 neighbour's stored state).
    __device__ static __forceinline__ void inlet(const CT (&d)[9], CT bx, CT &k1, CT &k5, CT &k8) {
#pragma clang fp contract(on)
        const CT s = (d[0] + (d[2] + d[4])) + CT(2) * (d[3] + (d[6] + d[7]));
        const CT dr = (s + bx) * recip(CT(1) - bx);
        const CT ru = (CT(1) + dr) * bx;
        const CT h = CT(0.5) * (d[2] - d[4]);
        k1 = d[3] + (CT(2) / CT(3)) * ru;
        k5 = d[7] - h + (CT(1) / CT(6)) * ru;
        k8 = d[6] + h + (CT(1) / CT(6)) * ru;
    }
    __device__ static __forceinline__ void outlet(const CT (&d)[9], const SweepArgs<T> &a, CT &k3,
                                                  CT &k7, CT &k6) {
#pragma clang fp contract(on)
        const CT s = (d[0] + (d[2] + d[4])) + CT(2) * (d[1] + (d[5] + d[8]));
        const CT uo = (s + (CT)a.one_minus_rho_out) * recip((CT)a.rho_out);
        const CT ru = (CT)a.rho_out * uo;
        const CT h = CT(0.5) * (d[2] - d[4]);
        k3 = d[1] - (CT(2) / CT(3)) * ru;
        k7 = d[5] + h - (CT(1) / CT(6)) * ru;
        k6 = d[8] - h - (CT(1) / CT(6)) * ru;
    }
    __device__ static __forceinline__ void neumann(const CT (&d)[9], CT bx, CT by, CT &k3, CT &k7,
                                                   CT &k6) {
#pragma clang fp contract(on)
        // rho = (1 + s) / (1 + ux): offsets of the Zou-He velocity closure
        const CT s = (d[0] + (d[2] + d[4])) + CT(2) * (d[1] + (d[5] + d[8]));
        const CT dr = (s - bx) * recip(CT(1) + bx);
        const CT ru = (CT(1) + dr) * bx, rv = (CT(1) + dr) * by;
        const CT h = CT(0.5) * (d[2] - d[4]);
        k3 = d[1] - (CT(2) / CT(3)) * ru;
        k7 = d[5] + h - (CT(1) / CT(6)) * ru - CT(0.5) * rv;
        k6 = d[8] - h - (CT(1) / CT(6)) * ru + CT(0.5) * rv;
    }
    __device__ static __forceinline__ void closure(CT (&d)[9], uint32_t type, CT bx, CT by,
                                                   const SweepArgs<T> &a) {
        if (type == kFluid) {
            // no closure (the common case, tested first)
        } else if (type == kInlet) {
            inlet(d, bx, d[1], d[5], d[8]);
        } else if (type == kOutlet) {
            outlet(d, a, d[3], d[7], d[6]);
        } else if (type == kOutletNeumann) {
            neumann(d, bx, by, d[3], d[7], d[6]);
        }
    }
    __device__ static __forceinline__ void relax(CT (&d)[9], const SweepArgs<T> &a, double &mass,
                                                 double &ux_out, double &uy_out) {
#pragma clang fp contract(on)
        const CT dr = ((d[0] + (d[1] + d[3])) + (d[2] + d[4])) + ((d[5] + d[8]) + (d[6] + d[7]));
        const CT rho = CT(1) + dr;
        const CT jx = (d[1] + (d[5] + d[8])) - (d[3] + (d[6] + d[7]));
        const CT jy = (d[2] + (d[5] + d[6])) - (d[4] + (d[8] + d[7]));
        const CT ir = recip(rho);
        const CT ux = jx * ir, uy = jy * ir;
        const CT om = (CT)a.omega;
        // Opposite directions i, opp(i) have c.u = +-cu: their equilibrium
        // offsets share the even part A = 4.5 cu^2 - 1.5 u.u and differ in the
        // sign of the odd part B = 3 cu.
        const CT pux = ux, puy = uy;
        const CT puu15 = CT(1.5) * (pux * pux + puy * puy);
        // With the weights rounded (to float), the equilibrium's mass and
        // momentum differ from dr and (jx, jy) by ~1e-8 relative, every step,
        // with a fixed sign: a bias that the flow's slowest mode accumulates
        // over thousands of steps (a steady-state error ~1e-4).  So the
        // increments t_i = e_i - d_i toward equilibrium are corrected to
        // conserve exactly before the relaxation: the (1,3) and (2,4) pairs
        // take the momentum defects, t_0 the mass defect.  Each population
        // then relaxes as d_i + om t_i in one multiply-add.  Every sum is in
        // mirror-symmetric order, so a y-reflection maps each increment onto
        // its mirror image bit for bit.
        CT t[9];
        // A + B = (4.5 cu + 3) cu - 1.5 u.u and A - B = (4.5 cu - 3) cu - 1.5 u.u,
        // two multiply-adds each.
        auto incr_pair = [&](int i, int j, CT cu, CT w) {
            const CT hp = CT(4.5) * cu + CT(3), hm = CT(4.5) * cu - CT(3);
            const CT ApB = hp * cu - puu15, AmB = hm * cu - puu15;
            t[i] = w * (dr + rho * ApB) - d[i];
            t[j] = w * (dr + rho * AmB) - d[j];
        };
        const CT w1 = CT(1) / CT(9), w5 = CT(1) / CT(36);
        incr_pair(1, 3, pux, w1);
        incr_pair(2, 4, puy, w1);
        incr_pair(5, 7, pux + puy, w5);
        incr_pair(6, 8, puy - pux, w5);
        const CT mx = (t[1] - t[3]) + ((t[5] - t[7]) + (t[8] - t[6]));
        const CT my = (t[2] - t[4]) + ((t[5] - t[8]) + (t[6] - t[7]));
        t[1] = t[1] - CT(0.5) * mx;
        t[3] = t[3] + CT(0.5) * mx;
        t[2] = t[2] - CT(0.5) * my;
        t[4] = t[4] + CT(0.5) * my;
        t[0] = -(((t[1] + t[3]) + (t[2] + t[4])) + ((t[5] + t[8]) + (t[6] + t[7])));
#pragma unroll
        for (int i = 0; i < 9; ++i) d[i] = d[i] + om * t[i];
        mass = 1.0 + (double)dr;
        ux_out = (double)ux;
        uy_out = (double)uy;
    }
};

using F32Cell = OffsetCell<float, ArithT<float>>;
using H16Cell = OffsetCell<h16, ArithT<h16>>;
using BF16Cell = OffsetCell<bf16, ArithT<bf16>>;

}  // namespace lbm
