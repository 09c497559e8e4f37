// Single Runge-Kutta stages, one cell per lane: steps of mid-size grids, the
// compensated form, and the recomputation of stages in reverse passes.
#include <hip/hip_runtime.h>

#include "launch.hpp"
#include "row_block.hpp"
#include "step_fused.hpp"

namespace cdbm {

namespace {

typedef const __attribute__((address_space(4))) StageParams* StageTable;

// Reads of a block's planes at the lane's column.  A block is 64 cells of one
// row, so the rows' offsets are scalar and only the column is a vector operand:
// a load takes one scalar addition for its plane and nothing on the vector unit.
template <typename S>
struct StageLd {
    const char* f;
    int64_t plane;       // bytes of a plane (at most 2^31)
    uint32_t row[5];     // byte offsets in a plane of the rows at offset -2 .. 2
    uint32_t col;        // byte offset in a row of the lane's column
    __device__ __forceinline__ S operator()(int i, int oy) const {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<char*>(f) + i * plane, 0, (int)(uint32_t)plane, 0x00020000);
        const int v = (int)col, s = (int)row[oy + 2];
        if constexpr (sizeof(S) == 4) {
            return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, v, s, 0));
        } else {
            typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
            const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(rs, v, s, 0);
            return __builtin_bit_cast(double, w);
        }
    }
};

// The stencil of a velocity without its centre, upwind first: s[0..2] along x
// (from r, the block's row of this velocity, the cell at r[2 + lane]), s[3..5]
// along y.
template <typename S>
__device__ __forceinline__ void load_stencil_y(const StageLd<S>& ld, int i, S s[6]) {
    if (SY[i] > 0) {
        s[3] = ld(i, -2); s[4] = ld(i, -1); s[5] = ld(i, 1);
    } else if (SY[i] < 0) {
        s[3] = ld(i, -1); s[4] = ld(i, 1); s[5] = ld(i, 2);
    }
}
template <typename S>
__device__ __forceinline__ void read_stencil_x(const S* r, int lane, int i, S s[6]) {
    if (SX[i] > 0) {
        s[0] = r[lane]; s[1] = r[lane + 1]; s[2] = r[lane + 3];
    } else if (SX[i] < 0) {
        s[0] = r[lane + 1]; s[1] = r[lane + 3]; s[2] = r[lane + 4];
    }
}

// cx D_x + cy D_y of a velocity (coefficients of velocities towards larger indices).
template <typename A, typename S>
__device__ __forceinline__ A stencil_advection(int i, const S s[6], A f, A cx, A cy) {
    A adv = A(0);
    if (SY[i] > 0) adv = cy * nnd_pos<A>(s[3], s[4], f, s[5]);
    else if (SY[i] < 0) adv = -cy * nnd_neg<A>(s[3], f, s[4], s[5]);
    if (SX[i] > 0) adv = fma(cx, nnd_pos<A>(s[0], s[1], f, s[2]), adv);
    else if (SX[i] < 0) adv = fma(-cx, nnd_neg<A>(s[0], f, s[1], s[2]), adv);
    return adv;
}

// (rho, j_x, j_y, 2E) of the distributions whose parity combinations are g.
__device__ __forceinline__ void stage_conserved(const Parity& g, StageTable K, double q[4]) {
    q[0] = ((g.ee[0] + g.ee[1]) + (g.ee[2] + g.ee[3])) + (g.ee[4] + g.ee[5]);
    double jx = 0.0, jy = 0.0, e2 = 0.0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        jx = fma(K->jv[c], g.oe[c], jx);
        jy = fma(K->jv[c], g.eo[c], jy);
    }
    constexpr int group[6] = {0, 0, 1, 2, 2, 3};
#pragma unroll
    for (int c = 0; c < 6; ++c) e2 = fma(K->en[group[c]], g.ee[c], e2);
    q[1] = jx;
    q[2] = jy;
    q[3] = e2;
}

// Adds the (rho, j_x, j_y, 2E) of a group's four values to q.
__device__ __forceinline__ void group_conserved(const double v[4], int group, StageTable K,
                                                double q[4]) {
    double sum, x, y;
    if (group % 2 == 0) {
        sum = (v[0] + v[2]) + (v[1] + v[3]);
        x = v[0] - v[2];
        y = v[1] - v[3];
    } else {
        const double s01 = v[0] + v[1], s23 = v[2] + v[3];
        sum = s01 + s23;
        x = (v[0] - v[1]) - (v[2] - v[3]);
        y = s01 - s23;
    }
    q[0] += sum;
    q[1] = fma(K->jv[group], x, q[1]);
    q[2] = fma(K->jv[group], y, q[2]);
    q[3] = fma(K->en[group], sum, q[3]);
}

// One stage with the per-cell arithmetic of the fused step:
//   STAGE2 == false:  out = f + dt L(f)
//   STAGE2 == true:   out = base / 2 + (f + dt L(f)) / 2
// COMP, the compensated form: f is read from float storage and every term is
// formed in double, as in the FP64 form:
//   STAGE2 == false:  y = f + A,              out = round(y + C),
//                     r_out = r + m(y - out)
//   STAGE2 == true:   y = base/2 + f/2 + A,   out = round(y + C),
//                     r_out = r_base/2 + r/2 + m(y - out)
// where A is the stage's advection term dt (-v . grad f) of Eqs. (12)-(20)
// and C its relaxation term -dt (f - f^eq)/tau of Eq. (1) (both halved in
// the second stage), f^eq is that of the compensated moments m(f) + r, and
// m(.) is (rho, j_x, j_y, 2E) of a set of 16 values.  The conserved moments
// m(f) + r of the output are those of the stage's combination without C
// (the advection flux changes them, the relaxation does not); C itself
// carries dt/tau of r into f.  The differences of the NND stencil are exact
// in double (two floats of like size), so the advection terms of
// neighbouring cells cancel in the grid sums to FP64 rounding.
//
// A block is 64 cells of a row and PARTS waves, each with the fluxes of 16 / PARTS
// velocities; two waves exchange the parity halves of their values through LDS
// and each form the moments.  The y stencils are requested together with the
// cell's own values (of one wave: those of half of its velocities, the rest and
// the Heun terms right after the moment arithmetic), so that they arrive during
// that arithmetic; in the compensated form three velocities ahead instead, the
// residual summed group by group and f and r converted twice, which takes the
// kernel from 183 to 127 registers and four waves a SIMD (512^2 27.5 -> 26.5 us
// a step).  Bound by latencies up to about 384 x 384, above by the return
// path of the vector loads (8 cycles of a CU for a 32-bit load of a wave, 16 for
// a 64-bit one) and by the FP64 arithmetic.  With x offsets loaded too, blocks of
// four rows and blocks in the grid's own order, a step of two stages took:
//   256^2 mixed 13.2 -> 8.8 us, FP64 17.7 -> 12.1, compensated 14.3 -> 11.7,
//   512^2 mixed 24.3 -> 18.4, FP64 38.7 -> 34.8, compensated 31.7 -> 28.7,
//   724^2 mixed 48.6 -> 35.6, FP64 79.1 -> 63.3, compensated 63.8 -> 51.9
// (one row per block 512^2 mixed 22.1 against four 22.9, eight 24.7; the band
// order of blocks: 256^2 mixed 13.2 -> 10.6, FP64 17.7 -> 13.6).
// LDS of a block of PARTS waves: their x rows and the parity halves they exchange.
template <typename S, bool COMP, int PARTS>
struct StageRow {
    S x[PARTS][NVX / PARTS][68];
    double half[PARTS][PARTS > 1 ? 8 : 1][64];
    double lost[PARTS][PARTS > 1 && COMP ? 4 : 1][64];
};

template <int PART, typename Row>
__device__ __forceinline__ void exchange_half(Row& half, const double v[8], Parity& g) {
    const int lane = threadIdx.x & 63;
    double c[8];
    half_parity(v, c);
    set_half(g, PART, c);
#pragma unroll
    for (int i = 0; i < 8; ++i) half[PART][i][lane] = c[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) c[i] = half[1 - PART][i][lane];
    set_half(g, 1 - PART, c);
}

template <typename S, bool STAGE2, bool COMP, int PART, int PARTS>
__device__ __forceinline__ void stage_part(const S* __restrict__ fin, const S* __restrict__ base,
                                           S* __restrict__ fout, StageTable K, int nx, int ny,
                                           int bc, int x0, int y, StageRow<S, COMP, PARTS>& sh) {
    using A = typename std::conditional<COMP, double, S>::type;
    constexpr int NI = NV / PARTS, I0 = PART * NI, NX = NVX / PARTS, K0 = PART * NX;
    // velocities whose y stencils are requested with the centres and, by the end
    // of the moments, with the Heun terms; those beyond that many ahead
    constexpr int FIRST = PARTS > 1 ? NI : COMP ? 3 : NI / 2;
    constexpr int AHEAD = COMP && PARTS == 1 ? FIRST : NI;
    const int lane = threadIdx.x & 63, x = x0 + lane;
    const bool px = !(bc & 1), py = !(bc & 2);
    StageLd<S> ld;
    ld.f = (const char*)fin;
    ld.plane = (int64_t)nx * ny * (int64_t)sizeof(S);
    const uint32_t pitch = (uint32_t)nx * (uint32_t)sizeof(S);
    ld.col = (uint32_t)block_column(x, nx, px) * (uint32_t)sizeof(S);
#pragma unroll
    for (int o = -2; o <= 2; ++o) ld.row[o + 2] = (uint32_t)wrap_by_two(y + o, ny, py) * pitch;
    StageLd<S> lb = ld;
    lb.f = (const char*)base;
    S f[NI], st[NI][6], rf[4], hb[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) f[i] = ld(I0 + i, 0);
    if constexpr (COMP) {
#pragma unroll
        for (int k = 0; k < 4; ++k) rf[k] = ld(NV + k, 0);
    }
    const S halo = halo_value<S>(fin, K0, NX, x0, y, nx, ny, px, false);
#pragma unroll
    for (int i = 0; i < FIRST; ++i) load_stencil_y(ld, I0 + i, st[i]);
    __builtin_amdgcn_sched_barrier(0);

    S (&row)[NX][68] = sh.x[PART];
#pragma unroll
    for (int i = 0; i < NI; ++i)
        if (SX[I0 + i] != 0) row[x_slot(I0 + i) - K0][2 + lane] = f[i];
    double neq[NI], r[4];
    {
        double fd[NI];
#pragma unroll
        for (int i = 0; i < NI; ++i) fd[i] = (double)f[i];
        Parity g;
        if constexpr (PARTS == 1) to_parity(fd, g);
        else exchange_half<PART>(sh.half, fd, g);
        double q[4];
        stage_conserved(g, K, q);
        Macro m;
        if constexpr (COMP) {
#pragma unroll
            for (int k = 0; k < 4; ++k) r[k] = (double)rf[k];
            const double rho = q[0] + r[0];
            m.rho = rho;
            m.ux = (q[1] + r[1]) / rho;
            m.uy = (q[2] + r[2]) / rho;
            m.T = ((q[3] + r[3]) / rho - (m.ux * m.ux + m.uy * m.uy)) * K->inv_a;
        } else {
            m = macro_of(q[0], q[1], q[2], q[3], K->inv_a);
        }
        nonequilibrium<PARTS == 1 ? 0 : PART, PARTS == 1 ? 2 : PART + 1>(g, m, *K, K->a, neq);
    }
    if constexpr (COMP) {
        // converted again below: kept in double over the moments, they and r
        // would take 40 registers
#pragma unroll
        for (int i = 0; i < NI; ++i) materialize(f[i]);
#pragma unroll
        for (int k = 0; k < 4; ++k) materialize(rf[k]);
    }
    if (lane < 4 * NX) row[lane >> 2][halo_place()] = halo;
    __builtin_amdgcn_sched_barrier(0);
    // the row is read by the wave that wrote it, whose LDS operations are in order
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
#pragma unroll
    for (int i = FIRST; i < AHEAD; ++i) load_stencil_y(ld, I0 + i, st[i]);
    if constexpr (STAGE2) {
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) hb[i] = lb(I0 + i, 0);
    }
    __builtin_amdgcn_sched_barrier(0);

    const bool inside = x < nx;
    char* const o = (char*)fout + (int64_t)y * pitch + (int64_t)x * (int64_t)sizeof(S);
    double lost[4], dm[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int j = 0; j < NI; ++j) {
        if (j + AHEAD < NI) {
            load_stencil_y(ld, I0 + j + AHEAD, st[j + AHEAD]);
            if (STAGE2) hb[j + AHEAD] = lb(I0 + j + AHEAD, 0);
        }
        const int i = I0 + j;
        A cx, cy, nz;
        if constexpr (sizeof(A) == 4) {
            cx = K->cf[STAGE2][i / 4];
            cy = K->cf[STAGE2][4 + i / 4];
            nz = K->cf[STAGE2][8 + (i / 4) % 2];
        } else {
            cx = K->cd[STAGE2][i / 4];
            cy = K->cd[STAGE2][4 + i / 4];
            nz = K->cd[STAGE2][8 + (i / 4) % 2];
        }
        const A fi = (A)f[j];
        if (SX[i] != 0) read_stencil_x(row[x_slot(i) - K0], lane, i, st[j]);
        const A adv = stencil_advection<A, S>(i, st[j], fi, cx, cy);
        S v;
        if constexpr (COMP) {
            double yv = adv;
            if (STAGE2) yv += 0.5 * fi + 0.5 * (double)hb[j];
            else yv += fi;
            v = (S)fma(nz, neq[j], yv);
            lost[j % 4] = yv - (double)v;
            if (j % 4 == 3) group_conserved(lost, i / 4, K, dm);
        } else {
            const A d = fma(nz, (A)neq[j], adv);
            v = STAGE2 ? fma(A(0.5), fi, d) : fi + d;
            if (STAGE2) v = fma(A(0.5), hb[j], v);
        }
        if (inside) *(S*)(o + i * ld.plane) = v;
    }
    if constexpr (COMP) {
        if constexpr (PARTS > 1) {
#pragma unroll
            for (int k = 0; k < 4; ++k) sh.lost[PART][k][lane] = dm[k];
            __syncthreads();
#pragma unroll
            for (int k = 0; k < 4; ++k) dm[k] = sh.lost[0][k][lane] + sh.lost[1][k][lane];
        }
#pragma unroll
        for (int k = 4 / PARTS * PART; k < 4 / PARTS * (PART + 1); ++k) {
            double rk = (double)rf[k];
            if (STAGE2) rk = 0.5 * (double)lb(NV + k, 0) + 0.5 * rk;
            if (inside) *(S*)(o + (NV + k) * ld.plane) = (S)(rk + dm[k]);
        }
    }
}

// COLUMNS: the blocks' bands are columns (COLUMN_BAND_ROWS), else rows in bands of
// `band` (row_band).
template <typename S, bool STAGE2, bool COMP, int PARTS, bool COLUMNS>
__global__ void __launch_bounds__(64 * PARTS) k_stage(const S* __restrict__ fin,
                                                      const S* __restrict__ base,
                                                      S* __restrict__ fout,
                                                      const StageParams* __restrict__ Kd, int nx,
                                                      int ny, int bc, uint32_t band) {
    __shared__ StageRow<S, COMP, PARTS> row;
    int x0, y;
    if constexpr (COLUMNS) {
        const uint32_t b = band_index(blockIdx.x, gridDim.x), column = b / (uint32_t)ny;
        x0 = (int)column * 64;
        y = (int)(b - column * (uint32_t)ny);
    } else {
        const uint32_t per_row = (uint32_t)(nx + 63) / 64;
        const uint32_t b = row_band_index(blockIdx.x, gridDim.x, band);
        y = (int)(b / per_row);
        x0 = (int)(b - (uint32_t)y * per_row) * 64;
    }
    const StageTable K = (StageTable)(uintptr_t)Kd;
    if (PARTS == 1 || __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) == 0)
        stage_part<S, STAGE2, COMP, 0, PARTS>(fin, base, fout, K, nx, ny, bc, x0, y, row);
    else
        stage_part<S, STAGE2, COMP, PARTS - 1, PARTS>(fin, base, fout, K, nx, ny, bc, x0, y, row);
}

template <typename S, bool COMP, int PARTS, bool COLUMNS>
hipError_t stage_launch_parts(const void* fin, const void* base, void* fout, bool stage2,
                              const KParams& K, const StageParams* Kd, hipStream_t st) {
    const dim3 grid((unsigned)((K.nx + 63) / 64) * (unsigned)K.ny), block(64 * PARTS);
    const int bc = K.bcx | K.bcy << 1;
    const uint32_t band = row_band(K.nx, K.ny);
    if (stage2)
        hipLaunchKernelGGL((k_stage<S, true, COMP, PARTS, COLUMNS>), grid, block, 0, st, (const S*)fin,
                           (const S*)base, (S*)fout, Kd, K.nx, K.ny, bc, band);
    else
        hipLaunchKernelGGL((k_stage<S, false, COMP, PARTS, COLUMNS>), grid, block, 0, st, (const S*)fin,
                           (const S*)base, (S*)fout, Kd, K.nx, K.ny, bc, band);
    return hipGetLastError();
}

// Two waves per block up to 3 * 2^15 cells (1.5 one-wave blocks per SIMD): below
// that a SIMD has one wave, which issues an instruction every five cycles and
// waits alone, above it the second wave's copy of the moments costs more.  Step
// of two stages with one / two waves per block:
//   100^2 mixed 8.3 / 6.8 us, FP64 9.2 / 7.4, compensated 9.8 / 8.3,
//   256^2 mixed 9.6 / 8.8, FP64 13.1 / 12.1, compensated 11.6 / 11.7,
//   400^2 mixed 14.2 / 15.3, FP64 23.3 / 24.2, compensated 21.4 / 23.5.
constexpr int64_t TWO_WAVE_CELLS = 3 << 15;

// Larger grids of up to this many rows: an eighth of them is four at most, the rows
// y +- 2 of such a band are mostly other XCDs', and the bands are an eighth of the
// columns each instead (kept-stage step in the mixed form, rows / columns: 65536 x
// 11 64.3 / 44.8 us, 65536 x 32 180 / 176, 4096 x 32 12.7 / 12.2; 4096 x 48 15.1 /
// 15.3, 8192 x 128 61.9 / 65.9; with rows 65536 x 8 .. 31 took 3 to 7 % more than
// with blocks in the grid's own order).
constexpr int COLUMN_BAND_ROWS = 32;

template <typename S, bool COMP>
hipError_t stage_launch(const void* fin, const void* base, void* fout, bool stage2,
                        const KParams& K, const StageParams* Kd, hipStream_t st) {
    if ((int64_t)K.nx * K.ny <= TWO_WAVE_CELLS)
        return stage_launch_parts<S, COMP, 2, false>(fin, base, fout, stage2, K, Kd, st);
    return K.ny <= COLUMN_BAND_ROWS
               ? stage_launch_parts<S, COMP, 1, true>(fin, base, fout, stage2, K, Kd, st)
               : stage_launch_parts<S, COMP, 1, false>(fin, base, fout, stage2, K, Kd, st);
}

}  // namespace

template <typename S>
hipError_t launch_stage(const void* fin, const void* base, void* fout, bool stage2,
                        const KParams& K, const StageParams* Kd, hipStream_t st) {
    return stage_launch<S, false>(fin, base, fout, stage2, K, Kd, st);
}

hipError_t launch_stage_comp(const void* fin, const void* base, void* fout, bool stage2,
                             const KParams& K, const StageParams* Kd, hipStream_t st) {
    return stage_launch<float, true>(fin, base, fout, stage2, K, Kd, st);
}

template hipError_t launch_stage<float>(const void*, const void*, void*, bool, const KParams&,
                                        const StageParams*, hipStream_t);
template hipError_t launch_stage<double>(const void*, const void*, void*, bool, const KParams&,
                                         const StageParams*, hipStream_t);

}  // namespace cdbm
