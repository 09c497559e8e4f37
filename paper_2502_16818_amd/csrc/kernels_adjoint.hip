// Reverse-mode kernels: transpose of one Runge-Kutta stage, of the initial
// equilibrium and of the macroscopic moments (see adjoint.hpp).
#include <hip/hip_runtime.h>

#include "adjoint.hpp"
#include "launch.hpp"
#include "row_block.hpp"

namespace cdbm {

namespace {

typedef const __attribute__((address_space(4))) StageParams* AdjointTable;
typedef const __attribute__((address_space(4))) KParams* BlockTable;

// Reads of one vector at the lane's column: rows y - 2 .. y + 2 are scalar byte
// offsets in a plane, the column a vector one.  Reads out of a plane's bounds
// give 0: a column offset of OUTSIDE is the adjoint at a zero-gradient ghost.
constexpr uint32_t OUTSIDE = 0x80000000u;
template <typename T>
struct ColumnLd {
    const char* p;
    int64_t plane;       // bytes of a plane (at most 2^31)
    uint32_t row[5];
    uint32_t col[5];     // the lane's column in those rows (OUTSIDE for a ghost)
    __device__ __forceinline__ T operator()(int i, int o) const {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<char*>(p) + i * plane, 0, (int)(uint32_t)plane, 0x00020000);
        const int v = (int)col[o + 2], s = (int)row[o + 2];
        if constexpr (sizeof(T) == 4) {
            return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, v, s, 0));
        } else {
            typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
            const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(rs, v, s, 0);
            return __builtin_bit_cast(double, w);
        }
    }
};

// GHOSTS_ZERO: ghosts of zero-gradient sides read 0 (else the edge cell).
template <bool GHOSTS_ZERO, typename T>
__device__ __forceinline__ void column_offsets(ColumnLd<T>& ld, const void* f, int x, int y,
                                               int nx, int ny, int bc) {
    ld.p = (const char*)f;
    ld.plane = (int64_t)nx * ny * (int64_t)sizeof(T);
    const bool px = !(bc & 1), py = !(bc & 2);
    const int cx = block_column(x, nx, px);
    const bool gx = GHOSTS_ZERO && !px && x >= nx;
#pragma unroll
    for (int o = -2; o <= 2; ++o) {
        const int cy = wrap_by_two(y + o, ny, py);
        const bool gy = GHOSTS_ZERO && !py && cy != y + o;
        ld.row[o + 2] = (uint32_t)cy * (uint32_t)nx * (uint32_t)sizeof(T);
        ld.col[o + 2] = gx || gy ? OUTSIDE : (uint32_t)cx * (uint32_t)sizeof(T);
    }
}

// One velocity's y stencils without the centres: the state at offsets -2 .. 2
// and the adjoint at the three of them its transpose reads.
template <typename S>
struct AdjointStencil {
    S f[5];
    double a[5];
};
template <typename S>
__device__ __forceinline__ void load_adjoint_stencil(ColumnLd<S> g, ColumnLd<double> a, int i,
                                                     AdjointStencil<S>& s) {
    if (SY[i] == 0) return;
    // descriptors formed anew: kept from the loads of the centres, those of 16
    // planes of both vectors would fill the scalar registers
    const uint32_t z0 = (uint32_t)opaque_zero();
    g.p += z0;
    a.p += z0;
#pragma unroll
    for (int o = -2; o <= 2; ++o) {
        if (o == 0) continue;
        s.f[o + 2] = g(i, o);
        // v > 0 reads the adjoint at -1, 1, 2 and v < 0 at -2, -1, 1
        s.a[o + 2] = (o != (SY[i] > 0 ? -2 : 2)) ? a(i, o) : 0.0;
    }
}

// The equilibrium transpose of a cell as a polynomial in the velocity:
// [(d g^eq / d g)^T a]_i = c0 + cx v_ix + cy v_iy + ce (|v_i|^2 + eta_i^2).
struct EqTranspose {
    double c0, cx, cy, ce;
};

// From the state m and pa = P^T a: w = B^T pa (the even-even block in mirror
// form, see nonequilibrium()) and its products with the raw moments and their
// derivatives.
__device__ __forceinline__ EqTranspose eq_transpose(const Macro& m, const Parity& pa,
                                                    AdjointTable K) {
    const double ux = m.ux, uy = m.uy, T = m.T, a = K->a;
    const double ux2 = ux * ux, uy2 = uy * uy, u2 = ux2 + uy2, uxy = ux * uy, D = ux2 - uy2;
    const double E = fma(a, T, u2), A2 = fma(2.0, T, E), A4 = fma(2.0, T, A2);
    const double xx = ux2 + T, yy = uy2 + T, a2 = a + 2.0, a4 = a + 4.0;
    double gr, gx, gy, gT;
    {
        const double sa = pa.ee[0] + pa.ee[1], da = pa.ee[0] - pa.ee[1];
        const double sc = pa.ee[3] + pa.ee[4], dc = pa.ee[3] - pa.ee[4];
        double w[4];   // of 1, E and the sums of the mirrored pairs
#pragma unroll
        for (int c = 0; c < 4; ++c)
            w[c] = fma(K->eep[0][c], sa,
                       fma(K->eep[1][c], sc,
                           fma(K->ees[0][c], pa.ee[2], K->ees[1][c] * pa.ee[5])));
        const double v2 = fma(K->eep[0][4], da, K->eep[1][4] * dc);   // of their differences
        const double v4 = fma(K->eep[0][5], da, K->eep[1][5] * dc);
        // sums: u^2 + 2 T and u^2 A4 + 2 T A2; differences: D and D A4
        const double s4 = fma(u2, A4, 2.0 * T * A2);
        gr = fma(w[1], E, w[0]) + fma(w[2], fma(2.0, T, u2), w[3] * s4) + D * fma(v4, A4, v2);
        const double t = fma(w[3], A4 + u2 + 2.0 * T, w[1] + w[2]);
        gx = 2.0 * ux * (t + fma(v4, A4 + D, v2));
        gy = 2.0 * uy * (t - fma(v4, A4 - D, v2));
        gT = fma(w[1], a, 2.0 * w[2]) + w[3] * fma(u2, a4, 2.0 * fma(T, a2, A2)) + v4 * (D * a4);
    }
    {
        double wo[4], we[4];   // of the moments odd in x and odd in y
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            double so = 0.0, se = 0.0;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                so = fma(K->ioe[r][c], pa.oe[r], so);
                se = fma(K->ioe[r][c < 2 ? c : 5 - c], pa.eo[r], se);
            }
            wo[c] = so;
            we[c] = se;
        }
        // moments ux {1, A2, ux^2 + 3T, yy} and uy {1, A2, xx, uy^2 + 3T}
        const double px = fma(wo[1], A2, wo[0]) + fma(wo[2], fma(3.0, T, ux2), wo[3] * yy);
        const double py = fma(we[1], A2, we[0]) + fma(we[2], xx, we[3] * fma(3.0, T, uy2));
        gr += fma(ux, px, uy * py);
        gx += px + 2.0 * ux * fma(ux, wo[1] + wo[2], uy * (we[1] + we[2]));
        gy += py + 2.0 * uy * fma(ux, wo[1] + wo[3], uy * (we[1] + we[3]));
        gT += fma(ux, fma(a2, wo[1], fma(3.0, wo[2], wo[3])),
                  uy * fma(a2, we[1], fma(3.0, we[3], we[2])));
    }
    {
        const double w0 = fma(K->ioo[0][0], pa.oo[0], K->ioo[1][0] * pa.oo[1]);
        const double w1 = fma(K->ioo[0][1], pa.oo[0], K->ioo[1][1] * pa.oo[1]);
        const double p = fma(w1, A4, w0);   // moments uxy {1, A4}
        gr = fma(uxy, p, gr);
        gx += uy * fma(2.0 * ux2, w1, p);
        gy += ux * fma(2.0 * uy2, w1, p);
        gT = fma(uxy * a4, w1, gT);
    }
    // through (rho, u, T) of g: (d q / d g)^T with the factors of rho cancelled
    EqTranspose t;
    t.ce = gT * K->inv_a;
    t.cx = fma(-2.0 * t.ce, ux, gx);
    t.cy = fma(-2.0 * t.ce, uy, gy);
    t.c0 = gr - fma(gx, ux, gy * uy) + t.ce * fma(-a, T, u2);
    return t;
}

// out = w_add * add + w_in * E'(g)^T a, and per 64 cells of a row the sum of
// w_in * sum_i a_i dE_i/dtau = w_in * sum_i a_i dt (g_i - g_i^eq) / tau^2
// written to tau_part (acc = 0) or added to it (acc = 1).
// The state g is in the storage precision S; adjoint vectors are double.
//
// A block is 64 cells of one row, one per lane, and two waves that each take
// the flux transposes of half of the velocities (PART = 0: groups a and b,
// PART = 1: c and d); of the pointwise part wave 0 forms the equilibrium
// transpose, handed to the other through LDS, and wave 1 the tau term.
//
// Bound by the return path of the vector loads (a 64-bit load of a wave takes
// 16 cycles of a CU whether it hits or not; with every stencil offset loaded
// that path was 86 % busy) and, on grids of a few waves per SIMD, by latencies.
// Therefore the x offsets come from the waves' own centres in LDS, with one
// load for the columns on either side; what a wave reads once (add, the tau
// slot) is requested with the centres, and the y offsets of four velocities
// ahead; the fluxes are formed before the waves meet for the equilibrium
// transpose.  The blocks are numbered in bands (row_band_index), so that the rows
// y +- 2 are in the block's own L2.  Time of a step's two stages (the four-wave
// block with both lines loaded / one wave per row, loaded / two waves, loaded /
// x through LDS and bands / this):
//   256^2 mixed 31.6 / 29.9 / 22.9 / 21.2 / 18.5 us, FP64 35.0 / 33.4 / 27.3 / 23.5 / 21.8,
//   1000 x 777 mixed 297 / 207 / 200 / 206 / 179, FP64 338 / 254 / 289 / 227 / 204,
//   1800^2 FP64 1474 / 1194 / 1282 / 912 / 835, and 816 with bands of eight rows.
// Two rows per block (four waves) cost up to 16 % more on large grids and gain
// at most 2 % on small ones; without the bands 256^2 FP64 took 10 % more; y
// offsets 2 / 4 / 8 velocities ahead: 1000 x 777 FP64 211 / 204 / 206 us,
// 256^2 mixed 18.8 / 18.5 / 19.8.
struct AdjointArgs {
    int nx, ny, bc;
    uint32_t band;
    double w_in, w_add, z, dt_tau2;
};

// LDS of a block: the x rows of its waves, and what they exchange.
template <typename S>
struct AdjointRow {
    S g[2][NVX / 2][68];           // six velocities with a component along x each,
    double a[2][NVX / 2][68];      // two halo columns on either side
    double parity[2][16][64];   // halves of P g, then of P a
    double eq[4][64];
};

template <typename S, int PART>
__device__ __forceinline__ void stage_adjoint_part(const S* __restrict__ g,
                                                   const double* __restrict__ a,
                                                   const double* __restrict__ add,
                                                   double* __restrict__ out, AdjointTable K, BlockTable I,
                                                   const AdjointArgs& p, int x0, int y,
                                                   double* __restrict__ tau_slot, int acc,
                                                   AdjointRow<S>& sh) {
    constexpr int NI = NV / 2, I0 = PART * NI, I1 = I0 + NI, AHEAD = 4, NX = NVX / 2, K0 = PART * NX;
    const int nx = p.nx, ny = p.ny, bc = p.bc, lane = threadIdx.x & 63, x = x0 + lane;
    ColumnLd<S> lg;
    ColumnLd<double> la;
    column_offsets<false>(lg, g, x, y, nx, ny, bc);
    column_offsets<true>(la, a, x, y, nx, ny, bc);
    S gc[NI];
    double ac[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        gc[i] = lg(I0 + i, 0);
        ac[i] = la(I0 + i, 0);
    }
    const S hg = halo_value<S>(g, K0, NX, x0, y, nx, ny, !(bc & 1), false);
    const double ha = halo_value<double>(a, K0, NX, x0, y, nx, ny, !(bc & 1), true);
    AdjointStencil<S> st[AHEAD + 1];
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) load_adjoint_stencil(lg, la, I0 + i, st[i]);
    const bool inside = x < nx;
    const int64_t at = (int64_t)y * nx + min(x, nx - 1), cells = (int64_t)nx * ny;
    double prior[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) prior[i] = 0.0;
    if (p.w_add != 0.0) {
#pragma unroll
        for (int i = 0; i < NI; ++i) prior[i] = add[(I0 + i) * cells + at];
    }
    double tau_before = 0.0;
    if (PART == 1 && acc) tau_before = *tau_slot;
    __builtin_amdgcn_sched_barrier(0);

    S (&tg)[NX][68] = sh.g[PART];
    double (&ta)[NX][68] = sh.a[PART];
#pragma unroll
    for (int i = 0; i < NI; ++i)
        if (SX[I0 + i] != 0) {
            tg[x_slot(I0 + i) - K0][2 + lane] = gc[i];
            ta[x_slot(I0 + i) - K0][2 + lane] = ac[i];
        }
    if (lane < 4 * NX) {
        const int c = halo_place();
        tg[lane >> 2][c] = hg;
        ta[lane >> 2][c] = ha;
    }
    EqTranspose eq;
    {
        Parity pg, pa;
        double v[8], c[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = (double)gc[i];
        half_parity(v, c);
        set_half(pg, PART, c);
#pragma unroll
        for (int i = 0; i < 8; ++i) sh.parity[PART][i][lane] = c[i];
        half_parity(ac, c);
        set_half(pa, PART, c);
#pragma unroll
        for (int i = 0; i < 8; ++i) sh.parity[PART][8 + i][lane] = c[i];
        __syncthreads();   // also orders the x rows, which a wave reads only of its own
#pragma unroll
        for (int i = 0; i < 8; ++i) c[i] = sh.parity[1 - PART][i][lane];
        set_half(pg, 1 - PART, c);
#pragma unroll
        for (int i = 0; i < 8; ++i) c[i] = sh.parity[1 - PART][8 + i][lane];
        set_half(pa, 1 - PART, c);
        const double rho = ((pg.ee[0] + pg.ee[1]) + (pg.ee[2] + pg.ee[3])) + (pg.ee[4] + pg.ee[5]);
        double jx = 0.0, jy = 0.0, e2 = 0.0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            jx = fma(K->jv[c], pg.oe[c], jx);
            jy = fma(K->jv[c], pg.eo[c], jy);
        }
        constexpr int group[6] = {0, 0, 1, 2, 2, 3};
#pragma unroll
        for (int c = 0; c < 6; ++c) e2 = fma(K->en[group[c]], pg.ee[c], e2);
        const Macro m = macro_of(rho, jx, jy, e2, K->inv_a);
        if constexpr (PART == 0) {
            eq = eq_transpose(m, pa, K);
            sh.eq[0][lane] = eq.c0;
            sh.eq[1][lane] = eq.cx;
            sh.eq[2][lane] = eq.cy;
            sh.eq[3][lane] = eq.ce;
        } else {
            // a . (g - f^eq) = pa . (pg / k - h), P P^T = k I per group (2 for the
            // axis pairs, 4 for the rest)
            Parity h;
            equilibrium_parity(m, *I, I->a, h);
            double d = 0.0;
#pragma unroll
            for (int r = 0; r < 6; ++r)
                d = fma(pa.ee[r], fma((r == 2 || r == 5) ? 0.25 : 0.5, pg.ee[r], -h.ee[r]), d);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const double k = (r & 1) ? 0.25 : 0.5;
                d = fma(pa.oe[r], fma(k, pg.oe[r], -h.oe[r]), d);
                d = fma(pa.eo[r], fma(k, pg.eo[r], -h.eo[r]), d);
            }
#pragma unroll
            for (int r = 0; r < 2; ++r) d = fma(pa.oo[r], fma(0.25, pg.oo[r], -h.oo[r]), d);
            // the partial of the 64 cells, summed in a fixed order
            double v = x < nx ? p.dt_tau2 * d * p.w_in : 0.0;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
            if (lane == 0) *tau_slot = acc ? tau_before + v : v;
        }
    }
    // 0 where a face of the cell is the edge of a zero-gradient side
    const double kxm = (bc & 1) && x == 0 ? 0.0 : 1.0, kxp = (bc & 1) && x == nx - 1 ? 0.0 : 1.0;
    const double kym = (bc & 2) && y == 0 ? 0.0 : 1.0, kyp = (bc & 2) && y == ny - 1 ? 0.0 : 1.0;
    const double w1 = p.w_in * (1.0 - p.z), w2 = p.w_in * p.z;
    double cx[2], cy[2], flux[NI];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int gr = 2 * PART + k;
        cx[k] = K->cd[0][gr];
        cy[k] = K->cd[0][4 + gr];
    }
#pragma unroll
    for (int i = I0; i < I1; ++i) {
        if (i + AHEAD < I1) load_adjoint_stencil(lg, la, i + AHEAD, st[(i + AHEAD - I0) % (AHEAD + 1)]);
        __builtin_amdgcn_sched_barrier(0);
        const int k = (i - I0) / 4;
        const double aci = ac[i - I0];
        double adv = 0.0;
        if (SX[i] != 0) {
            S f[5];
            double A[5];
#pragma unroll
            for (int o = -2; o <= 2; ++o) {
                const bool need = o != (SX[i] > 0 ? -2 : 2);
                f[o + 2] = o == 0 ? gc[i - I0] : tg[x_slot(i) - K0][2 + lane + o];
                A[o + 2] = o == 0 ? aci : (need ? ta[x_slot(i) - K0][2 + lane + o] : 0.0);
            }
            if (SX[i] > 0) adv = cx[k] * nnd_transpose<true, S>(f, A, kxm, kxp);
            else adv = -cx[k] * nnd_transpose<false, S>(f, A, kxm, kxp);
        }
        AdjointStencil<S>& s = st[(i - I0) % (AHEAD + 1)];
        s.f[2] = gc[i - I0];
        s.a[2] = aci;
        if (SY[i] > 0) adv = fma(cy[k], nnd_transpose<true, S>(s.f, s.a, kym, kyp), adv);
        else if (SY[i] < 0) adv = fma(-cy[k], nnd_transpose<false, S>(s.f, s.a, kym, kyp), adv);
        flux[i - I0] = adv;
        __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    if constexpr (PART == 1)
        eq = EqTranspose{sh.eq[0][lane], sh.eq[1][lane], sh.eq[2][lane], sh.eq[3][lane]};
#pragma unroll
    for (int i = I0; i < I1; ++i) {
        const double vg = K->jv[i / 4];
        double ceq = fma(eq.ce, K->en[i / 4], eq.c0);
        if (SX[i] != 0) ceq = fma(SX[i] > 0 ? vg : -vg, eq.cx, ceq);
        if (SY[i] != 0) ceq = fma(SY[i] > 0 ? vg : -vg, eq.cy, ceq);
        double r = fma(p.w_in, flux[i - I0], fma(w1, ac[i - I0], w2 * ceq));
        r = fma(p.w_add, prior[i - I0], r);
        if (inside) out[i * cells + at] = r;
    }
}

template <typename S>
__global__ void __launch_bounds__(128) k_stage_adjoint(
    const S* __restrict__ g, const double* __restrict__ a, const double* __restrict__ add,
    double* __restrict__ out, const StageParams* __restrict__ Kd, const KParams* __restrict__ Bd,
    AdjointArgs p,
    double* __restrict__ tau_part, int acc) {
    __shared__ AdjointRow<S> row;
    const uint32_t per_row = (uint32_t)(p.nx + 63) / 64;
    const uint32_t b = row_band_index(blockIdx.x, gridDim.x, p.band);
    const int y = (int)(b / per_row), x0 = (int)(b - (uint32_t)y * per_row) * 64;
    const AdjointTable K = (AdjointTable)(uintptr_t)Kd;
    const BlockTable I = (BlockTable)(uintptr_t)Bd;
    if (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) == 0)
        stage_adjoint_part<S, 0>(g, a, add, out, K, I, p, x0, y, tau_part + b, acc, row);
    else
        stage_adjoint_part<S, 1>(g, a, add, out, K, I, p, x0, y, tau_part + b, acc, row);
}

// Sum of part[i], part[i + step], ... (i < n) over the 1024 threads of a
// block, thread t starting at its own i, in a fixed order: up to four loads
// in flight per thread, each wave's 64 sums by shuffles, then the 16 wave
// sums by the first wave.  The result is valid in thread 0.  With clear,
// every element read is set to zero.
__device__ __forceinline__ double block_sum_1024(double* __restrict__ part, int64_t i,
                                                 int64_t step, int64_t n, bool clear) {
    __shared__ double red[16];
    double s = 0.0;
    for (; i + 3 * step < n; i += 4 * step) {
        double v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = part[i + k * step];
        if (clear) {
#pragma unroll
            for (int k = 0; k < 4; ++k) part[i + k * step] = 0.0;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) s += v[k];
    }
    for (; i < n; i += step) {
        s += part[i];
        if (clear) part[i] = 0.0;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x < 64) {
        t = threadIdx.x < 16 ? red[threadIdx.x] : 0.0;
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) t += __shfl_xor(t, o);
    }
    return t;
}

// dst[0] += scale * sum_b part[b] by one block (part cleared with clear).
__global__ void __launch_bounds__(1024) k_accumulate(double* __restrict__ part, int64_t n,
                                                     double scale, double* __restrict__ dst,
                                                     int clear) {
    const double t = block_sum_1024(part, threadIdx.x, 1024, n, clear != 0);
    if (threadIdx.x == 0) dst[0] += scale * t;
}

// out[k] = sum of part[b] over b = 1024 k + t + j 1024 gridDim.x: the first
// pass of a two-pass sum of many partials.
__global__ void __launch_bounds__(1024) k_partial_sum(double* __restrict__ part, int64_t n,
                                                      double* __restrict__ out, int clear) {
    const double t = block_sum_1024(part, (int64_t)blockIdx.x * 1024 + threadIdx.x,
                                    (int64_t)gridDim.x * 1024, n, clear != 0);
    if (threadIdx.x == 0) out[blockIdx.x] = t;
}

// g_q = (d f^eq(q) / d q)^T lam per cell.
template <typename S>
__global__ void __launch_bounds__(256) k_init_adjoint(const double* __restrict__ rho,
                                                      const double* __restrict__ ux,
                                                      const double* __restrict__ uy,
                                                      const double* __restrict__ T,
                                                      const double* __restrict__ lam,
                                                      double* __restrict__ g_rho,
                                                      double* __restrict__ g_ux,
                                                      double* __restrict__ g_uy,
                                                      double* __restrict__ g_T, KParams K,
                                                      int64_t cells) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= cells) return;
    double ad[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) ad[i] = lam[i * cells + c];
    const Macro m{rho[c], ux[c], uy[c], T[c]};
    const Quad q = equilibrium_vjp_q(m, K, K.a, ad);
    g_rho[c] = q.rho;
    g_ux[c] = q.ux;
    g_uy[c] = q.uy;
    g_T[c] = q.T;
}

// lam_f = (d (rho, u, T) / d f)^T g per cell.
template <typename S>
__global__ void __launch_bounds__(256) k_moments_adjoint(const S* __restrict__ f,
                                                         const double* __restrict__ g_rho,
                                                         const double* __restrict__ g_ux,
                                                         const double* __restrict__ g_uy,
                                                         const double* __restrict__ g_T,
                                                         double* __restrict__ lam, KParams K,
                                                         int64_t cells) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= cells) return;
    double fd[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) fd[i] = (double)f[i * cells + c];
    Parity pg;
    to_parity(fd, pg);
    const Macro m = macro_from_parity(pg, K, K.inv_a);
    const Quad q{g_rho[c], g_ux[c], g_uy[c], g_T[c]};
#pragma unroll
    for (int i = 0; i < NV; ++i) lam[i * cells + c] = moments_vjp_k(m, K, K.a, q, i);
}

inline unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

}  // namespace

int stage_adjoint_blocks(const KParams& K) {
    return (int)(blocks_for(K.nx, 64) * (unsigned)K.ny);
}

template <typename S>
hipError_t launch_stage_adjoint(const void* g, const void* a, const void* add, void* out,
                                double* tau_part, bool tau_add, double w_in, double w_add,
                                const KParams& K, const StageParams* Kd, const KParams* Bd,
                                hipStream_t st) {
    const AdjointArgs p{K.nx, K.ny, K.bcx | K.bcy << 1, row_band(K.nx, K.ny), w_in, w_add, K.z, K.dt / (K.tau * K.tau)};
    hipLaunchKernelGGL(k_stage_adjoint<S>, dim3(stage_adjoint_blocks(K)), dim3(128), 0, st,
                       (const S*)g, (const double*)a, (const double*)add, (double*)out, Kd, Bd, p,
                       tau_part, tau_add ? 1 : 0);
    return hipGetLastError();
}

template <typename S>
hipError_t launch_init_adjoint(const double* rho, const double* ux, const double* uy,
                               const double* T, const void* lam, double* g_rho, double* g_ux,
                               double* g_uy, double* g_T, const KParams& K, hipStream_t st) {
    const int64_t cells = (int64_t)K.nx * K.ny;
    hipLaunchKernelGGL(k_init_adjoint<S>, dim3(blocks_for(cells, 256)), dim3(256), 0, st, rho, ux,
                       uy, T, (const double*)lam, g_rho, g_ux, g_uy, g_T, K, cells);
    return hipGetLastError();
}

template <typename S>
hipError_t launch_moments_adjoint(const void* f, const double* g_rho, const double* g_ux,
                                  const double* g_uy, const double* g_T, void* lam,
                                  const KParams& K, hipStream_t st) {
    const int64_t cells = (int64_t)K.nx * K.ny;
    hipLaunchKernelGGL(k_moments_adjoint<S>, dim3(blocks_for(cells, 256)), dim3(256), 0, st,
                       (const S*)f, g_rho, g_ux, g_uy, g_T, (double*)lam, K, cells);
    return hipGetLastError();
}

hipError_t launch_accumulate_scalar(double* part, int n, double* scratch, double scale,
                                    double* dst, bool clear, hipStream_t st) {
    if (n > ACCUMULATE_ONE_PASS) {
        hipLaunchKernelGGL(k_partial_sum, dim3(ACCUMULATE_BLOCKS), dim3(1024), 0, st, part,
                           (int64_t)n, scratch, clear ? 1 : 0);
        part = scratch;
        n = ACCUMULATE_BLOCKS;
        clear = false;
    }
    hipLaunchKernelGGL(k_accumulate, dim3(1), dim3(1024), 0, st, part, (int64_t)n, scale, dst,
                       clear ? 1 : 0);
    return hipGetLastError();
}

#define CDBM_INSTANTIATE(S)                                                                      \
    template hipError_t launch_stage_adjoint<S>(const void*, const void*, const void*, void*,   \
                                                double*, bool, double, double, const KParams&,  \
                                                const StageParams*, const KParams*, hipStream_t); \
    template hipError_t launch_init_adjoint<S>(const double*, const double*, const double*,     \
                                               const double*, const void*, double*, double*,    \
                                               double*, double*, const KParams&, hipStream_t);  \
    template hipError_t launch_moments_adjoint<S>(const void*, const double*, const double*,    \
                                                  const double*, const double*, void*,          \
                                                  const KParams&, hipStream_t);
CDBM_INSTANTIATE(float)
CDBM_INSTANTIATE(double)
#undef CDBM_INSTANTIATE

}  // namespace cdbm
