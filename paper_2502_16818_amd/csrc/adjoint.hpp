// Reverse-mode (transpose) arithmetic of one Runge-Kutta stage of the CDBM.
//
// A stage is E(g) = g + dt L(g) with L(g)_i = c_x D_x(g_i) + c_y D_y(g_i)
// - (g_i - g_i^eq) / tau (c = -dt v_ir / dr, D the NND flux difference of
// Eqs. (12)-(20)).  Its transpose applied to a vector a at cell y is
//   a_i + dt (J_adv^T a)_i - (dt/tau) (a_i - [(d g^eq / d g)^T a]_i).
//
// NND transpose.  With the minmod selections fixed, D is linear.  The
// selection at a cell is (alpha, beta): mm(x) = alpha d(x+1/2) + beta d(x-1/2)
// (branch order of Eq. (16): neither if the differences do not share a strict
// sign, else the first argument when |X| <= |Y|).  For v > 0
//   D(x) = d(x-1/2) + (mm(x) - mm(x-1)) / 2,
// so with a the adjoint of D the adjoint of mm(x) is (a(x) - a(x+1)) / 2 and
// that of the face difference d(x+1/2)
//   G(x+1/2) = a(x+1) + alpha(x) (a(x) - a(x+1)) / 2
//                     + beta(x+1) (a(x+1) - a(x+2)) / 2;
// for v < 0, D(x) = d(x+1/2) - (mm(x+1) - mm(x)) / 2 gives
//   G(x+1/2) = a(x) + alpha(x) (a(x) - a(x-1)) / 2 + beta(x+1) (a(x+1) - a(x)) / 2.
// As d(x+1/2) = f(x+1) - f(x), the transpose at x is G(x-1/2) - G(x+1/2).
// Periodic positions wrap.  At a zero-gradient side a is zero at the ghosts,
// and the ghosts' own contributions belong to the edge cell, whose values they
// repeat: their sum telescopes to minus G of the grid's edge face, so that
// face simply drops out.
//
// Equilibrium transpose.  f^eq = P h with h = rho B mhat(u, T) (P: unpacking
// of parity combinations, B: scaled block inverses).  P^T is the parity
// transform itself, so with w = B^T P^T a:
//   g_rho = w . mhat,  g_q = rho w . d mhat / d q  (q = u_x, u_y, T),
// and [(d f^eq/d g)^T a]_k = g_rho + (g_ux (v_kx - u_x) + g_uy (v_ky - u_y)
//   + g_T (|v_k - u|^2 + eta_k^2 - (D+I) T) / (D+I)) / rho.
#pragma once

#include <hip/hip_runtime.h>

#include "cell.hpp"

namespace cdbm {

struct Quad {
    double rho, ux, uy, T;
};

// (d f^eq / d q)^T a for q = (rho, u_x, u_y, T) at the state m, from the
// parity transform hb = P^T a of a: w = B^T hb and its products with the
// raw moments and their derivatives, one parity block at a time (ee, then oe
// and eo, then oo) with the scheduler kept from interleaving the blocks, so
// that only one block's weights and tables are live at once.
__device__ __forceinline__ Quad equilibrium_vjp_q_parity(const Macro& m, const KParams& K,
                                                        double a, const Parity& hb) {
    const double ux = m.ux, uy = m.uy, T = m.T;
    const double ux2 = ux * ux, uy2 = uy * uy, u2 = ux2 + uy2, uxy = ux * uy;
    const double A2 = u2 + (a + 2.0) * T, A4 = u2 + (a + 4.0) * T;
    double gr = 0.0, gx = 0.0, gy = 0.0, gT = 0.0;
    {
        double wee[6];
#pragma unroll
        for (int c = 0; c < 6; ++c) {
            double s = 0.0;
#pragma unroll
            for (int r = 0; r < 6; ++r) s = fma(K.iee[r][c], hb.ee[r], s);
            wee[c] = s;
        }
        const double mee[6] = {1.0, u2 + a * T, ux2 + T, uy2 + T, ux2 * A4 + T * A2,
                               uy2 * A4 + T * A2};
        const double ee_x[6] = {0.0, 2.0 * ux, 2.0 * ux, 0.0, 2.0 * ux * (A4 + ux2 + T),
                                2.0 * ux * (uy2 + T)};
        const double ee_y[6] = {0.0, 2.0 * uy, 0.0, 2.0 * uy, 2.0 * uy * (ux2 + T),
                                2.0 * uy * (A4 + uy2 + T)};
        const double ee_T[6] = {0.0, a, 1.0, 1.0, ux2 * (a + 4.0) + A2 + T * (a + 2.0),
                                uy2 * (a + 4.0) + A2 + T * (a + 2.0)};
#pragma unroll
        for (int c = 0; c < 6; ++c) {
            gr = fma(wee[c], mee[c], gr);
            gx = fma(wee[c], ee_x[c], gx);
            gy = fma(wee[c], ee_y[c], gy);
            gT = fma(wee[c], ee_T[c], gT);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    {
        double woe[4], weo[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            double so = 0.0, se = 0.0;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                so = fma(K.ioe[r][c], hb.oe[r], so);
                se = fma(K.ieo[r][c], hb.eo[r], se);
            }
            woe[c] = so;
            weo[c] = se;
        }
        const double moe[4] = {ux, ux * A2, ux * (ux2 + 3.0 * T), ux * (uy2 + T)};
        const double meo[4] = {uy, uy * A2, uy * (ux2 + T), uy * (uy2 + 3.0 * T)};
        const double oe_x[4] = {1.0, A2 + 2.0 * ux2, 3.0 * (ux2 + T), uy2 + T};
        const double oe_y[4] = {0.0, 2.0 * uxy, 0.0, 2.0 * uxy};
        const double oe_T[4] = {0.0, ux * (a + 2.0), 3.0 * ux, ux};
        const double eo_x[4] = {0.0, 2.0 * uxy, 2.0 * uxy, 0.0};
        const double eo_y[4] = {1.0, A2 + 2.0 * uy2, ux2 + T, 3.0 * (uy2 + T)};
        const double eo_T[4] = {0.0, uy * (a + 2.0), uy, 3.0 * uy};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            gr = fma(woe[c], moe[c], fma(weo[c], meo[c], gr));
            gx = fma(woe[c], oe_x[c], fma(weo[c], eo_x[c], gx));
            gy = fma(woe[c], oe_y[c], fma(weo[c], eo_y[c], gy));
            gT = fma(woe[c], oe_T[c], fma(weo[c], eo_T[c], gT));
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    {
        double woo[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) woo[c] = fma(K.ioo[0][c], hb.oo[0], K.ioo[1][c] * hb.oo[1]);
        const double moo[2] = {uxy, uxy * A4};
        const double oo_x[2] = {uy, uy * (A4 + 2.0 * ux2)};
        const double oo_y[2] = {ux, ux * (A4 + 2.0 * uy2)};
        const double oo_T[2] = {0.0, uxy * (a + 4.0)};
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            gr = fma(woo[c], moo[c], gr);
            gx = fma(woo[c], oo_x[c], gx);
            gy = fma(woo[c], oo_y[c], gy);
            gT = fma(woo[c], oo_T[c], gT);
        }
    }
    return Quad{gr, m.rho * gx, m.rho * gy, m.rho * gT};
}

// (d f^eq / d q)^T a for q = (rho, u_x, u_y, T) at the state m.
__device__ __forceinline__ Quad equilibrium_vjp_q(const Macro& m, const KParams& K, double a,
                                                 const double adj[NV]) {
    Parity hb;
    to_parity(adj, hb);   // P^T a
    return equilibrium_vjp_q_parity(m, K, a, hb);
}

// (d q / d f)^T g at the state m, velocity k: q = (rho, u_x, u_y, T).
__device__ __forceinline__ double moments_vjp_k(const Macro& m, const KParams& K, double a,
                                                const Quad& g, int k) {
    const double cx = K.vx[k] - m.ux, cy = K.vy[k] - m.uy;
    const double e = cx * cx + cy * cy + K.eta2[k];
    return g.rho + (g.ux * cx + g.uy * cy + g.T * (e - a * m.T) / a) / m.rho;
}

// Parity form h of f^eq (f^eq = unpacking of h, see equilibrium()), from the
// whole block inverses, the products in one fixed order of rounding: dL/dtau
// sums a . (g - f^eq), where nearly all of a . g cancels when a is close to a
// moment (conserved), so the form must round like its own earlier values.
template <typename Table>
__device__ __forceinline__ void equilibrium_parity(const Macro& m, Table& K, double a, Parity& h) {
    const double ux = m.ux, uy = m.uy, T = m.T;
    const double ux2 = ux * ux, uy2 = uy * uy, u2 = fma(ux, ux, uy2), uxy = ux * uy;
    const double E = fma(a, T, u2), A2 = fma(2.0, T, E), A4 = fma(2.0, T, A2);
    const double xx = fma(ux, ux, T), yy = fma(uy, uy, T), TA2 = T * A2;
    const double mee[6] = {1.0, E, xx, yy, fma(ux2, A4, TA2), fma(uy2, A4, TA2)};
    const double moe[4] = {ux, ux * A2, ux * fma(3.0, T, ux2), ux * yy};
    const double meo[4] = {uy, uy * A2, uy * xx, uy * fma(3.0, T, uy2)};
    const double moo[2] = {uxy, uxy * A4};
#pragma unroll
    for (int r = 0; r < 6; ++r) {
        double s = K.iee[r][0];
#pragma unroll
        for (int c = 1; c < 6; ++c) s = fma(K.iee[r][c], mee[c], s);
        h.ee[r] = m.rho * s;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        double so = 0.0, se = 0.0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            so = fma(K.ioe[r][c], moe[c], so);
            se = fma(K.ieo[r][c], meo[c], se);
        }
        h.oe[r] = m.rho * so;
        h.eo[r] = m.rho * se;
    }
#pragma unroll
    for (int r = 0; r < 2; ++r) h.oo[r] = m.rho * fma(K.ioo[r][0], moo[0], K.ioo[r][1] * moo[1]);
}

// Half the minmod selections at a cell, from the differences X on its far side
// and Y on its near side (the branch order of Eq. (16)): alpha / 2 (X is
// taken: the signs agree and 0 < |X| <= |Y|) and beta / 2 (Y is taken:
// 0 < |Y| < |X|).  With Ys = Y times the sign of X these are 0 < |X| <= Ys and
// 0 < Ys < |X|; a NaN selects neither.
__device__ __forceinline__ float times_sign(float y, float x) {
    return __int_as_float(__float_as_int(y) ^ (__float_as_int(x) & (int)0x80000000));
}
__device__ __forceinline__ double times_sign(double y, double x) {
    const uint64_t b = __builtin_bit_cast(uint64_t, y);
    const uint32_t s = (uint32_t)(__builtin_bit_cast(uint64_t, x) >> 32) & 0x80000000u;
    return __builtin_bit_cast(double, b ^ ((uint64_t)s << 32));
}
// 0.5 or 0.0 (the low word of both is zero: one select).
__device__ __forceinline__ double half_if(bool c) {
    return __builtin_bit_cast(double, (uint64_t)(c ? 0x3fe00000u : 0u) << 32);
}
template <typename S>
__device__ __forceinline__ double half_alpha(S X, S Y) {
    const S ax = fabs(X), ys = times_sign(Y, X);
    return half_if(ax > S(0) && ax <= ys);
}
template <typename S>
__device__ __forceinline__ double half_beta(S X, S Y) {
    const S ax = fabs(X), ys = times_sign(Y, X);
    return half_if(ys > S(0) && ys < ax);
}

// Transpose of the flux difference along a line at cell x (without its
// coefficient), from the state f(x-2 .. x+2) and the adjoint of the
// differences at x-2 .. x+2 (those not needed are not read), through the
// adjoints G of the face differences d (see the header): km and kp are 0 where
// the face on that side is the edge of a zero-gradient side, else 1.
template <bool POS, typename S>
__device__ __forceinline__ double nnd_transpose(const S f[5], const double A[5], double km,
                                                double kp) {
    const S d0 = f[1] - f[0], d1 = f[2] - f[1], d2 = f[3] - f[2], d3 = f[4] - f[3];
    const double am = half_alpha(d1, d0);                           // cell x - 1
    const double ac = half_alpha(d2, d1), bc = half_beta(d2, d1);   // cell x
    const double bp = half_beta(d3, d2);                            // cell x + 1
    double gm, gp;   // faces x - 1/2, x + 1/2
    if (POS) {
        const double e = A[1] - A[2], h = A[2] - A[3], k = A[3] - A[4];
        gm = fma(am, e, fma(bc, h, A[2]));
        gp = fma(ac, h, fma(bp, k, A[3]));
    } else {
        const double e = A[1] - A[0], h = A[2] - A[1], k = A[3] - A[2];
        gm = fma(am, e, fma(bc, h, A[1]));
        gp = fma(ac, h, fma(bp, k, A[2]));
    }
    return fma(-kp, gp, km * gm);
}

}  // namespace cdbm
