// Fused two-stage Runge-Kutta step with FP64 storage, two waves per strip,
// marching in y with everything a row needs from the rows before it in
// registers.
//
// A strip is 56 output columns: lane l holds column x0 - 4 + l, stage 1 is
// valid on lanes 2 .. 61 and stage 2 on lanes 4 .. 59.  Each of the block's two
// waves has eight velocities (part 0: groups a and b, part 1: c and d), by
// offsets alone: both run the same instructions.  Once per stage they exchange
// the parity combinations of their centres through LDS, and each forms the
// moments.  Along x the NND takes the neighbouring values and minmod terms from
// the neighbouring lanes.  Along y the marching keeps, per velocity, the last
// difference and the last minmod term, so that a new row costs one difference
// and one minmod:
//   v_y > 0, cell j:  D = d(j-1/2) + (mm(j) - mm(j-1)) / 2,     new row j + 1
//   v_y < 0, cell j:  D = d(j+1/2) - (mm(j+1) - mm(j)) / 2,     new row j + 2
// with mm(j) = minmod(d(j+1/2), d(j-1/2)).  Iteration a takes row a of the
// velocities with v_y < 0, row a - 1 of those with v_y > 0 and row a - 2 of
// the others, which completes stage 1 of row a - 2; its f^(1) goes the same
// way into stage 2, two rows behind (the velocities that need it one or two
// rows later wait in registers).  Only the f^n of the two rows between the
// stages (the Heun term) go through LDS, each lane reading what it wrote.  The
// operations are those of the single-stage kernels term by term, and the
// result is bitwise the same.
//
// Bound by memory: 2047 x 1531 (401 MB in, 401 MB out) 205 us, 192 with the
// arithmetic left out (the rows at the ends of the pieces and the columns at
// the sides of the strips are read again), 166 without the stores; the strip
// with rings of rows in LDS (step_fused.hpp; one block of six waves per CU and
// two barriers per six rows, its stencils read from LDS) took 263.
#pragma once

#include "march_order.hpp"
#include "row_block.hpp"
#include "step_fused.hpp"

namespace cdbm {

constexpr int MARCH_TX = 56;   // output columns of a strip

// Local index of a part's velocities (one axis group, one diagonal group) by
// the sign of v_y.
constexpr int MARCH_POS[3] = {1, 4, 5};
constexpr int MARCH_NEG[3] = {3, 6, 7};
constexpr int MARCH_FLAT[2] = {0, 2};
constexpr int march_slot(int j) { return j < 4 ? 0 : 1 + (j & 1); }
static_assert(march_slot(1) == 0 && march_slot(4) == 1 && march_slot(5) == 2 && march_slot(3) == 0 &&
                  march_slot(6) == 1 && march_slot(7) == 2,
              "position among those of the same sign");

typedef const __attribute__((address_space(4))) StageParams* MarchTable;

typedef unsigned MarchBits __attribute__((ext_vector_type(2)));
typedef double MarchPair __attribute__((ext_vector_type(2)));

struct MarchLds {
    // by buffer and part: parity combinations.  march_buffer() gives the buffer of
    // an exchange; between a wave's reads of one and the other wave's next write
    // to it lies the barrier of the exchange between them
    double half[2][2][7][64];
    // by part and row parity: f^n between the stages; a lane reads what it wrote
    MarchPair heun[2][2][4][64];
};

// minmod() of values that are results of arithmetic: fmin and fmax of double
// would quiet each operand again, an instruction each.
__device__ __forceinline__ double march_minmod(double X, double Y) {
    double lo, hi;
    asm("v_min_f64 %0, %1, %2" : "=v"(lo) : "v"(X), "v"(Y));
    asm("v_max_f64 %0, %1, %2" : "=v"(hi) : "v"(X), "v"(Y));
    asm("v_min_f64 %0, %1, 0" : "=v"(hi) : "v"(hi));
    asm("v_max_f64 %0, %1, %2" : "=v"(lo) : "v"(lo), "v"(hi));
    return lo;
}

// What the marching keeps of the rows before (see the header).
struct MarchState {
    double pf[3], pd[3], pm[3];           // v_y > 0: the next centre, d, mm
    double nf1[3], nf0[3], nd[3], nm[3];  // v_y < 0: the last row, the next centre, d, mm
};

// k (f - f^eq) of a part's eight velocities; own: the part's parity
// combinations in the order of half_parity (nonequilibrium() with q = part).
__device__ __forceinline__ void nonequilibrium_own(const double own[8], const Macro& m,
                                                   MarchTable K, int q, double out[8]) {
    const double a = K->a;
    const double ux = m.ux, uy = m.uy, T = m.T;
    const double ux2 = ux * ux, uy2 = uy * uy, u2 = fma(ux, ux, uy2), uxy = ux * uy;
    const double E = fma(a, T, u2);
    const double A2 = fma(2.0, T, E);
    const double A4 = fma(2.0, T, A2);
    const double xx = fma(ux, ux, T), yy = fma(uy, uy, T), TA2 = T * A2;
    const double m4 = fma(ux2, A4, TA2), m5 = fma(uy2, A4, TA2);
    const double moe[4] = {ux, ux * A2, ux * fma(3.0, T, ux2), ux * yy};
    const double meo[4] = {uy, uy * A2, uy * xx, uy * fma(3.0, T, uy2)};
    const double n2 = -2.0 * m.rho, n4 = -4.0 * m.rho;
    const double s23 = xx + yy, d23 = xx - yy, s45 = m4 + m5, d45 = m4 - m5;
    const double P = fma(K->eep[q][3], s45, fma(K->eep[q][2], s23, K->eep[q][1] * E));
    const double Q = fma(K->eep[q][5], d45, K->eep[q][4] * d23);
    const double e0 = fma(n2, P + Q, fma(n2, K->eep[q][0], own[0]));
    const double e1 = fma(n2, P - Q, fma(n2, K->eep[q][0], own[1]));
    const double D = fma(K->ees[q][3], s45, fma(K->ees[q][2], s23, K->ees[q][1] * E));
    const double e2 = fma(n4, D, fma(n4, K->ees[q][0], own[4]));
    double o[2], e[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        double so = 0.0, se = 0.0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            so = fma(K->ioe[2 * q + r][c], moe[c], so);
            se = fma(K->ioe[2 * q + r][c < 2 ? c : 5 - c], meo[c], se);
        }
        const double n = r ? n4 : n2;
        o[r] = fma(n, so, own[r ? 5 : 2]);
        e[r] = fma(n, se, own[r ? 6 : 3]);
    }
    const double oo = fma(n4, fma(K->ioo[q][0], uxy, K->ioo[q][1] * (uxy * A4)), own[7]);
    out[0] = e0 + o[0];
    out[2] = e0 - o[0];
    out[1] = e1 + e[0];
    out[3] = e1 - e[0];
    const double p = e2 + e[1], n = e2 - e[1], r = o[1] + oo, s = o[1] - oo;
    out[4] = p + r;
    out[5] = p - r;
    out[6] = n - s;
    out[7] = n + s;
}

// One stage of a part (q): centres from the state and, for the velocities
// without y component, from v; then, velocity by velocity, the new row v[j]
// (one past the centre for v_y > 0, two for v_y < 0) gives the difference along
// y and moves into the state.  fc: the centres.
template <bool HALF>
__device__ __forceinline__ void march_stage(MarchState& s, const double v[8], MarchTable K0, int q,
                                            double (*half)[7][64], double fc[8], double out[8]) {
    const int lane = threadIdx.x & 63;
    const MarchTable K = K0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        fc[MARCH_POS[k]] = s.pf[k];
        fc[MARCH_NEG[k]] = s.nf0[k];
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) fc[MARCH_FLAT[k]] = v[MARCH_FLAT[k]];
    double neq[8];
    {
        double fd[8], own[8], g0[7], g1[7];
#pragma unroll
        for (int j = 0; j < 8; ++j) fd[j] = (double)fc[j];
        half_parity(fd, own);
#pragma unroll
        for (int j = 0; j < 7; ++j) half[q][j][lane] = own[j];
        lds_barrier();
#pragma unroll
        for (int j = 0; j < 7; ++j) {
            g0[j] = half[0][j][lane];
            g1[j] = half[1][j][lane];
        }
        // the order of half_parity: ee, ee, oe, eo, ee (diagonal), oe, eo
        const double rho = ((g0[0] + g0[1]) + (g0[4] + g1[0])) + (g1[1] + g1[4]);
        double jx = 0.0, jy = 0.0, e2 = 0.0;
        jx = fma(K->jv[0], g0[2], jx);
        jx = fma(K->jv[1], g0[5], jx);
        jx = fma(K->jv[2], g1[2], jx);
        jx = fma(K->jv[3], g1[5], jx);
        jy = fma(K->jv[0], g0[3], jy);
        jy = fma(K->jv[1], g0[6], jy);
        jy = fma(K->jv[2], g1[3], jy);
        jy = fma(K->jv[3], g1[6], jy);
        e2 = fma(K->en[0], g0[0], e2);
        e2 = fma(K->en[0], g0[1], e2);
        e2 = fma(K->en[1], g0[4], e2);
        e2 = fma(K->en[2], g1[0], e2);
        e2 = fma(K->en[2], g1[1], e2);
        e2 = fma(K->en[3], g1[4], e2);
        const Macro m = macro_of(rho, jx, jy, e2, K->inv_a);
        nonequilibrium_own(own, m, K, q, neq);
    }
    const MarchTable C = (MarchTable)((uintptr_t)K0 + (uint32_t)opaque_zero());
    double cx[2], cy[2], nz[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        cx[k] = C->cd[HALF][2 * q + k];
        cy[k] = C->cd[HALF][4 + 2 * q + k];
        nz[k] = C->cd[HALF][8 + k];
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const double f = fc[j];
        double adv = 0.0;
        if (SY[j] > 0) {
            const int k = march_slot(j);
            const double dn = v[j] - s.pf[k], mn = march_minmod(dn, s.pd[k]);
            adv = cy[j / 4] * fma(0.5, mn - s.pm[k], s.pd[k]);
            s.pf[k] = v[j];
            s.pd[k] = dn;
            s.pm[k] = mn;
        } else if (SY[j] < 0) {
            const int k = march_slot(j);
            const double dn = v[j] - s.nf1[k], mn = march_minmod(dn, s.nd[k]);
            adv = -cy[j / 4] * fma(-0.5, mn - s.nm[k], s.nd[k]);
            s.nf0[k] = s.nf1[k];
            s.nf1[k] = v[j];
            s.nd[k] = dn;
            s.nm[k] = mn;
        }
        if (SX[j] != 0) {
            const double dl = f - from_left(f), dr = from_right(f) - f;
            const double M = march_minmod(dr, dl);
            if (SX[j] > 0) adv = fma(cx[j / 4], fma(0.5, M - from_left(M), dl), adv);
            else adv = fma(-cx[j / 4], fma(-0.5, from_right(M) - M, dr), adv);
        }
        const double d = fma(nz[j / 4], neq[j], adv);
        out[j] = HALF ? fma(0.5, f, d) : f + d;
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) materialize(out[j]);
}

// The first rows of a piece: only the state moves.
__device__ __forceinline__ void march_take(MarchState& s, const double v[8]) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double x = v[MARCH_POS[k]], dn = x - s.pf[k];
        s.pm[k] = march_minmod(dn, s.pd[k]);
        s.pf[k] = x;
        s.pd[k] = dn;
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double x = v[MARCH_NEG[k]], dn = x - s.nf1[k];
        s.nm[k] = march_minmod(dn, s.nd[k]);
        s.nf0[k] = s.nf1[k];
        s.nf1[k] = x;
        s.nd[k] = dn;
    }
}

// A part's strip.  EDGE: the strip touches a zero-gradient side of the grid.
template <bool EDGE>
struct March {
    MarchTable K;
    MarchLds& lds;
    int q, nx, ny, bcy, lane;
    int from;                 // 4 * the lane whose f^(1) stage 2 reads in this place
    const char* in;           // the part's first plane
    char* out;
    int64_t plane;            // bytes of a plane (at most 2^31)
    uint32_t lo, so;          // byte offsets in a row: of the column read, and written
    int r0, r1, r2;           // source rows a, a - 1, a - 2 of the next iteration
    double pre[8];                 // the next rows' values
    double ps[3], fl[2][2];        // f^(1) on its way to stage 2: v_y > 0 (one row), v_y = 0 (two)
    MarchState s1, s2;

    __device__ __forceinline__ March(const double* fin, double* fout, MarchTable k, int nx_, int ny_, int bcx,
                                     int bcy_, int x0, int ya, int part, MarchLds& l)
        : K(k), lds(l), ps{}, fl{}, s1{}, s2{} {
        lane = threadIdx.x & 63;
        q = part;
        nx = nx_;
        ny = ny_;
        bcy = bcy_;
        plane = (int64_t)nx * ny * 8;
        in = (const char*)fin + 8 * q * plane;
        out = (char*)fout + 8 * q * plane;
        const int x = x0 - 4 + lane;
        lo = (uint32_t)map_index(x, nx, bcx) * 8u;
        // a column that is not this strip's to write gets an offset out of bounds
        so = lane >= 4 && lane < 60 && x < nx ? (uint32_t)x * 8u : 0x80000000u;
        const int cx = bcx == CDBM_ZERO_GRADIENT ? min(max(x, 0), nx - 1) : x;
        from = 4 * (cx - x0 + 4);
        r1 = source_row(ya - 6, ny, bcy);
        r0 = source_row(ya - 5, ny, bcy);
        load(ya - 4);
    }

    // Starts the loads of iteration a (one more than the last time).
    __device__ __forceinline__ void load(int a) {
        r2 = r1;
        r1 = r0;
        const int n = r0 + 1 == ny ? 0 : r0 + 1, c = min(max(a, 0), ny - 1);
        r0 = bcy == CDBM_PERIODIC ? n : c;
        const uint32_t pitch = (uint32_t)nx * 8u;
        const char* p = in + (uint32_t)opaque_zero();
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t row = (uint32_t)(SY[j] < 0 ? r0 : (SY[j] > 0 ? r1 : r2)) * pitch;
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<char*>(p) + j * plane, 0, (int)(uint32_t)plane, 0x00020000);
            const MarchBits w = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)lo, (int)row, 0);
            pre[j] = __builtin_bit_cast(double, w);
        }
    }

    __device__ __forceinline__ void store(int row, const double v[8]) {
        const uint32_t at = (uint32_t)row * (uint32_t)nx * 8u;
        char* p = out + (uint32_t)opaque_zero();
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                p + j * plane, 0, (int)(uint32_t)plane, 0x00020000);
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(MarchBits, v[j]), rs, (int)so,
                                                  (int)at, 0);
        }
    }

    // Iteration a; STAGES: how many of the two stages run; first: the buffer of
    // stage 1's exchange.
    template <int STAGES>
    __device__ __forceinline__ void iterate(int a, int yb, int first) {
        if constexpr (STAGES == 0) {
            march_take(s1, pre);
            load(a + 1);
            return;
        }
        // stage 1 at row c1
        const int c1 = a - 2, c2 = c1 - 2;
        double f1[8], fn[8], v2[8];
        MarchPair(*hs)[64] = lds.heun[q][c1 & 1];
        {
            double fc[8];
            march_stage<false>(s1, pre, K, q, lds.half[first], fc, f1);
            // the Heun term of row c2 comes out of LDS, that of row c1 goes in
            if constexpr (STAGES == 2) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const MarchPair v = hs[g][lane];
                    fn[2 * g] = v[0];
                    fn[2 * g + 1] = v[1];
                }
            }
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                hs[g][lane] = MarchPair{fc[2 * g], fc[2 * g + 1]};
            }
        }
        load(a + 1);
        if constexpr (EDGE) ghosts(c1, f1);
        // f^(1) of row c1 (v_y < 0), c1 - 1 (v_y > 0) and c1 - 2 into stage 2
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            v2[MARCH_NEG[k]] = f1[MARCH_NEG[k]];
            v2[MARCH_POS[k]] = ps[k];
            ps[k] = f1[MARCH_POS[k]];
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            v2[MARCH_FLAT[k]] = fl[0][k];
            fl[0][k] = fl[1][k];
            fl[1][k] = f1[MARCH_FLAT[k]];
        }
        if constexpr (STAGES < 2) {
            march_take(s2, v2);
            return;
        }
        if (c2 < yb) {
            double r[8];
            {
                double fc[8];
                march_stage<true>(s2, v2, K, q, lds.half[march_buffer(MARCH_TAKE + MARCH_ONE, 1)], fc, r);
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                r[j] = fma(0.5, fn[j], r[j]);
                materialize(r[j]);
            }
            // the next row's loads are waited for here: in the next iteration
            // they would wait behind these stores
#pragma unroll
            for (int j = 0; j < 8; ++j) materialize(pre[j]);
            store(c2, r);
        }
    }

    // f^(1) at ghost cells of zero-gradient sides repeats the edge cell's.
    __device__ __forceinline__ void ghosts(int c1, double f1[8]) {
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (SX[j] != 0) {
                typedef int i32x2 __attribute__((ext_vector_type(2)));
                const i32x2 w = __builtin_bit_cast(i32x2, f1[j]);
                const i32x2 t = {__builtin_amdgcn_ds_bpermute(from, w[0]),
                                 __builtin_amdgcn_ds_bpermute(from, w[1])};
                f1[j] = __builtin_bit_cast(double, t);
            }
        if (bcy != CDBM_ZERO_GRADIENT) return;
        if (c1 >= ny) {   // row ny - 1 again
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                f1[MARCH_NEG[k]] = s2.nf1[k];
                f1[MARCH_POS[k]] = ps[k];
            }
        } else if (c1 <= 0) {   // no difference before row 0
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                ps[k] = f1[MARCH_POS[k]];
                s2.nf1[k] = f1[MARCH_NEG[k]];
                s2.pf[k] = f1[MARCH_POS[k]];
                s2.pd[k] = s2.pm[k] = s2.nd[k] = s2.nm[k] = 0.0;
            }
        }
    }
};

// Advance rows [ya, yb) of the strip starting at column x0; one part.
template <bool EDGE>
__device__ __forceinline__ void march_strip(const double* __restrict__ fin, double* __restrict__ fout,
                                            MarchTable K, int nx, int ny, int bcx, int bcy, int x0,
                                            int ya, int yb, int part, MarchLds& lds) {
    March<EDGE> m(fin, fout, K, nx, ny, bcx, bcy, x0, ya, part, lds);
    const int a0 = ya - 4;
    int a = a0;
#pragma unroll 1
    for (; a < a0 + MARCH_TAKE; ++a) m.template iterate<0>(a, yb, 0);
#pragma unroll 1
    for (; a < a0 + MARCH_TAKE + MARCH_ONE; ++a)
        m.template iterate<1>(a, yb, march_buffer(a - a0, 0));
    constexpr int first = march_buffer(MARCH_TAKE + MARCH_ONE, 0);
#pragma unroll 1
    for (; a < yb + 4; a += 2) {
        m.template iterate<2>(a, yb, first);
        m.template iterate<2>(a + 1, yb, first);
    }
}

}  // namespace cdbm
