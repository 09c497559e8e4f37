// Runge-Kutta stages with four lanes per cell, for grids too small to fill
// the chip with one cell per lane.
//
// With one lane per cell a stage is a chain of about 900 instructions in a
// single wave (5-7 us however small the grid).  Here lane q of a quad takes
// the q-th velocity of each of the four groups (axis groups a and c: +x, +y,
// -x, -y; diagonal groups b and d), so the NND differences and the rows of the
// inverse moment matrix spread over the quad; only the moments of the cell
// (about 70 instructions) are formed by all four lanes.  The chain drops to
// about 300 instructions, and both stages (and, on a line of cells, several
// steps) run in one launch on a tile held in LDS.
//
// A tile's buffer is laid out [group][cell][q]: a wave's 16 cells x 4 lanes
// read 64 consecutive elements, lanes of different q never share a bank
// (their element index is q mod 4), and a cell's four values of a group are
// one 16- or 32-byte read.
//
// The operations and their order are those of stage_cell_k, so the results are
// bitwise the same, next to infinities and NaN too.
// A velocity that moves towards smaller indices is treated as the mirror image of
// one that moves towards larger ones: its values are held with the opposite sign,
// in LDS and in registers, and its stencil is read backwards, so that its
// differences are those of the other kernels and its coefficient is that of its
// mirror image.  (A diagonal velocity is held with the sign of its x component.)
// A change of sign is exact, and so is a sign per lane (+-1 by fma) that selects
// between the sums and the differences of the unpacking.
#pragma once

#include "cell.hpp"

namespace cdbm {

// A lane's position in its quad: axis groups: lanes 0, 2 move along x, lanes
// 1, 3 along y; sa, sx, sy: direction signs of its axis velocity and, along x
// and y, of its diagonal ones.
struct QuadLane {
    int q;
    bool isx;
    int sa, sx, sy;
};

// Is velocity k of a group (diagonal: 0 or 1) held with the opposite sign?
__device__ __forceinline__ constexpr bool quad_negated(int diagonal, int k) {
    return diagonal ? k == 1 || k == 2 : k >= 2;
}

// Parity combinations (to_parity) of 16 distributions as they are held.
__device__ __forceinline__ void quad_parity(const double f[NV], Parity& g) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int a = 8 * q, d = 8 * q + 4;
        g.ee[3 * q + 0] = f[a + 0] - f[a + 2];
        g.ee[3 * q + 1] = f[a + 1] - f[a + 3];
        g.oe[2 * q + 0] = f[a + 0] + f[a + 2];
        g.eo[2 * q + 0] = f[a + 1] + f[a + 3];
        const double s01 = f[d + 0] - f[d + 1], s23 = f[d + 3] - f[d + 2];
        const double d01 = f[d + 0] + f[d + 1], d32 = f[d + 2] + f[d + 3];
        g.ee[3 * q + 2] = s01 + s23;
        g.oe[2 * q + 1] = d01 + d32;
        g.eo[2 * q + 1] = s01 - s23;
        g.oo[q] = d01 - d32;
    }
}

__device__ __forceinline__ QuadLane quad_lane(int q) {
    return QuadLane{q, (q & 1) == 0, q < 2 ? 1 : -1, (q == 0 || q == 3) ? 1 : -1, q < 2 ? 1 : -1};
}

// The run's constants, loaded once per kernel while the first loads of f are
// on their way: those that are the same for every lane in scalar registers
// (76 of them), the lane's own in vector registers.  The scalar cache starts
// cold in a kernel of a few microseconds, and loads spread over the stage
// came as a chain of misses; so every line is touched first, all at once.
// (Kept in LDS, the 16-byte reads of every lane took more of the LDS's time
// than the stencils; fetched per lane from global memory, they took longer
// than f itself.)
template <typename S>
struct QuadConst {
    double eep[2][6];     // the part odd in x <-> y negated for the lanes along y
    double odd[2][4];     // row of the axis pair odd along the lane's axis
    S a[2], x[2], y[2], nz[2];   // first stage; half of them in the second
    QuadParams::Shared s;
};

template <typename S>
__device__ __forceinline__ QuadConst<S> quad_const(const QuadParams* __restrict__ Qd,
                                                   const QuadLane& L) {
    {
        int t;   // whichever line comes last; the loads are complete when the block ends
        asm volatile(
            "s_load_dword %0, %1, 0x0\n\ts_load_dword %0, %1, 0x40\n\t"
            "s_load_dword %0, %1, 0x80\n\ts_load_dword %0, %1, 0xc0\n\t"
            "s_load_dword %0, %1, 0x100\n\ts_load_dword %0, %1, 0x140\n\t"
            "s_load_dword %0, %1, 0x180\n\ts_load_dword %0, %1, 0x1c0\n\t"
            "s_load_dword %0, %1, 0x200\n\ts_load_dword %0, %1, 0x240\n\t"
            "s_waitcnt lgkmcnt(0)"
            : "=&s"(t)
            : "s"(Qd));
        asm volatile("" ::"v"(t));
    }
    // constant address space: scalar loads, also behind the statement above
    typedef const __attribute__((address_space(4))) double* Table;
    const Table l = (Table)(uintptr_t)&Qd->lane, u = (Table)(uintptr_t)&Qd->s;
    QuadConst<S> c;
    double v[38];   // QuadParams::Lane
#pragma unroll
    for (int k = 0; k < 38; ++k) v[k] = l[k];
#pragma unroll
    for (int k = 0; k < 38; ++k) asm volatile("" : "+s"(v[k]));   // loaded, not selected by address
#pragma unroll
    for (int p = 0; p < 2; ++p) {
#pragma unroll
        for (int k = 0; k < 6; ++k)
            c.eep[p][k] = (k >= 4 && !L.isx) ? -v[6 * p + k] : v[6 * p + k];
#pragma unroll
        for (int k = 0; k < 4; ++k) c.odd[p][k] = L.isx ? v[12 + 4 * p + k] : v[20 + 4 * p + k];
        c.a[p] = (S)(L.isx ? v[28 + p] : v[30 + p]);
        c.x[p] = (S)v[32 + p];
        c.y[p] = (S)v[34 + p];
        c.nz[p] = (S)v[36 + p];
    }
#pragma unroll
    for (int p = 0; p < 2; ++p) {
#pragma unroll
        for (int k = 0; k < 6; ++k) asm volatile("" : "+v"(c.eep[p][k]));
#pragma unroll
        for (int k = 0; k < 4; ++k) asm volatile("" : "+v"(c.odd[p][k]));
        asm volatile("" : "+v"(c.a[p]), "+v"(c.x[p]), "+v"(c.y[p]), "+v"(c.nz[p]));
    }
    double* s = (double*)&c.s;
#pragma unroll
    for (int k = 0; k < 38; ++k) s[k] = u[k];
#pragma unroll
    for (int k = 0; k < 38; ++k) asm volatile("" : "+s"(s[k]));
    return c;
}

// macro_from_parity() from the shared constants.
__device__ __forceinline__ Macro quad_macro(const Parity& g, const QuadParams::Shared& K) {
    const double rho = ((g.ee[0] + g.ee[1]) + (g.ee[2] + g.ee[3])) + (g.ee[4] + g.ee[5]);
    const double en[6] = {K.en_a, K.en_a, K.en_b, K.en_c, K.en_c, K.en_d};
    double jx = 0.0, jy = 0.0, e2 = 0.0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        jx = fma(K.jv[c], g.oe[c], jx);
        jy = fma(K.jv[c], g.eo[c], jy);
    }
#pragma unroll
    for (int c = 0; c < 6; ++c) e2 = fma(en[c], g.ee[c], e2);
    return macro_of(rho, jx, jy, e2, K.inv_a);
}

// k (f - f^eq) of the lane's four velocities (groups a, b, c, d), k = 2 for
// the axis groups and 4 for the diagonal ones, as they are held: nonequilibrium()
// of the cell, the lane's rows only.
__device__ __forceinline__ void quad_nonequilibrium(const Parity& g, const Macro& m,
                                                    const QuadLane& L,
                                                    const double eep[2][6],
                                                    const double odd[2][4],
                                                    const QuadParams::Shared& K, double out[4]) {
    const double a = K.a;
    const double ux = m.ux, uy = m.uy, T = m.T;
    const double ux2 = ux * ux, uy2 = uy * uy, u2 = fma(ux, ux, uy2), uxy = ux * uy;
    const double E = fma(a, T, u2);        // u^2 + (D+I) T
    const double A2 = fma(2.0, T, E);
    const double A4 = fma(2.0, T, A2);
    const double xx = fma(ux, ux, T), yy = fma(uy, uy, T), TA2 = T * A2;
    const double mee[6] = {1.0, E, xx, yy, fma(ux2, A4, TA2), fma(uy2, A4, TA2)};
    const double moe[4] = {ux, ux * A2, ux * fma(3.0, T, ux2), ux * yy};
    const double meo[4] = {uy, uy * A2, uy * xx, uy * fma(3.0, T, uy2)};
    const double moo[2] = {uxy, uxy * A4};
    const double n2 = -2.0 * m.rho, n4 = -4.0 * m.rho;
    const double s23 = mee[2] + mee[3], d23 = mee[2] - mee[3];
    const double s45 = mee[4] + mee[5], d45 = mee[4] - mee[5];
    double mo[4];   // odd moments along the lane's axis
#pragma unroll
    for (int c = 0; c < 4; ++c) mo[c] = L.isx ? moe[c] : meo[c];
    const double sa = L.sa, sx = L.sx, sy = L.sy;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const double ge = L.isx ? g.ee[3 * p] : g.ee[3 * p + 1];
        const double go = L.isx ? g.oe[2 * p] : g.eo[2 * p];
        const double* ee = eep[p];
        const double P = fma(ee[3], s45, fma(ee[2], s23, ee[1] * mee[1]));
        const double Q = fma(ee[5], d45, ee[4] * d23);
        const double te = fma(n2, P + Q, fma(n2, ee[0], ge));
        double s = 0.0;
#pragma unroll
        for (int c = 0; c < 4; ++c) s = fma(odd[p][c], mo[c], s);
        out[2 * p] = fma(sa, te, fma(n2, s, go));

        const int r = 2 * p + 1;
        const double D =
            fma(K.diag[p].ees[3], s45, fma(K.diag[p].ees[2], s23, K.diag[p].ees[1] * mee[1]));
        const double td = fma(n4, D, fma(n4, K.diag[p].ees[0], g.ee[3 * p + 2]));
        double so = 0.0, se = 0.0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            so = fma(K.diag[p].ioe[c], moe[c], so);
            se = fma(K.diag[p].ieo[c], meo[c], se);
        }
        const double to = fma(n4, so, g.oe[r]);
        const double tv = fma(n4, se, g.eo[r]);
        const double tt =
            fma(n4, fma(K.diag[p].ioo[0], moo[0], K.diag[p].ioo[1] * moo[1]), g.oo[p]);
        out[r] = fma(sx, fma(sy, tv, td), fma(sy, tt, to));
    }
}

// Stencil cells of a lane in a tile: the cells 2 and 1 upwind and 1 downwind
// of its cell, along its axis velocity's direction and, for the diagonal
// velocities, along x and along y.
struct QuadStencil {
    int a[3], x[3], y[3];
};

// LINE: the grid is one row of cells; nothing changes along y.
// (lx, ly): the cell in the tile, w: the tile's row length; (lo, hi): the
// range of tile columns and rows that stencils are clamped to (the grid's
// edge cells on a zero-gradient side).
template <bool LINE>
__device__ __forceinline__ QuadStencil quad_stencil(const QuadLane& L, int lx, int ly, int w,
                                                    int xlo, int xhi, int ylo, int yhi) {
    QuadStencil s;
    const int here = ly * w + lx;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int o = k == 2 ? 1 : k - 2;   // -2, -1, 1 downwind
        s.x[k] = ly * w + min(max(lx + o * L.sx, xlo), xhi);
        const int ax = ly * w + min(max(lx + o * L.sa, xlo), xhi);
        if constexpr (LINE) {
            s.y[k] = here;
            s.a[k] = L.isx ? ax : here;
        } else {
            s.y[k] = min(max(ly + o * L.sy, ylo), yhi) * w + lx;
            const int ay = min(max(ly + o * L.sa, ylo), yhi) * w + lx;
            s.a[k] = L.isx ? ax : ay;
        }
    }
    return s;
}

// A cell's four values of a group.
template <typename S>
struct Quad4 {
    typedef S type __attribute__((ext_vector_type(4)));
};

// The sign with which the lane's velocity of a group is held.
__device__ __forceinline__ int quad_sign(const QuadLane& L, int gr) { return gr & 1 ? L.sx : L.sa; }

// The 16 distributions of cell `here` of a tile of NC cells, as they are held.
template <typename S, int NC>
__device__ __forceinline__ void quad_cell(const S* F, int here, double fd[NV]) {
    typedef typename Quad4<S>::type V4;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const V4 v = *(const V4*)(F + (g * NC + here) * 4);
#pragma unroll
        for (int k = 0; k < 4; ++k) fd[4 * g + k] = (double)v[k];
    }
}

// Advection term of the lane's velocity of group gr, as it is held: A is the
// arithmetic type of the differences, ca / cxd / cyd the coefficients of the
// velocities towards larger indices.
template <typename A, typename S, int NC, bool LINE>
__device__ __forceinline__ A quad_advection(const S* F, int gr, const QuadLane& L,
                                            const QuadStencil& st, A f, A ca, A cxd, A cyd) {
    auto at = [&](int cell) { return (A)F[(gr * NC + cell) * 4 + L.q]; };
    if ((gr & 1) == 0) return ca * nnd_pos<A>(at(st.a[0]), at(st.a[1]), f, at(st.a[2]));
    const A dx = nnd_pos<A>(at(st.x[0]), at(st.x[1]), f, at(st.x[2]));
    if constexpr (LINE) {
        return cxd * dx;
    } else if constexpr (sizeof(A) == 8) {
        return fma(cxd, dx, cyd * nnd_pos<A>(at(st.y[0]), at(st.y[1]), f, at(st.y[2])));
    } else {
        // minmod of a NaN and Y is min(Y, 0) in FP32 (Y in FP64): the differences
        // along y need the sign of the y component
        const A s = (A)(L.sx * L.sy), m2 = at(st.y[0]), m1 = at(st.y[1]), p1 = at(st.y[2]);
        const A d0 = s * (f - m1);
        const A dy = plus_half(d0, minmod(s * (p1 - f), d0) - minmod(d0, s * (m1 - m2)));
        return fma(cxd, dx, s * cyd * dy);
    }
}

// One stage of the lane's four velocities (groups a .. d) at cell `here`:
// stage_cell_k of the cell, fc the cell's own values of these velocities (all as held).
template <typename S, int NC, bool HALF, bool LINE>
__device__ __forceinline__ void quad_stage(const S* F, int here, const QuadStencil& st,
                                           const S fc[4], const QuadLane& L,
                                           const QuadConst<S>& C, S out[4]) {
    double fd[NV];
    quad_cell<S, NC>(F, here, fd);
    Parity g;
    quad_parity(fd, g);
    const Macro m = quad_macro(g, C.s);
    double neq[4];
    quad_nonequilibrium(g, m, L, C.eep, C.odd, C.s, neq);
    const S h = HALF ? S(0.5) : S(1);
#pragma unroll
    for (int gr = 0; gr < 4; ++gr) {
        const int p = gr >> 1;
        const S adv = quad_advection<S, S, NC, LINE>(F, gr, L, st, fc[gr], h * C.a[p], h * C.x[p], h * C.y[p]);
        const S d = fma(h * C.nz[gr & 1], (S)neq[gr], adv);
        out[gr] = HALF ? fma(S(0.5), fc[gr], d) : fc[gr] + d;
    }
}

}  // namespace cdbm
