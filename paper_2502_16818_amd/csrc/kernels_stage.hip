// Single Runge-Kutta stages, one cell per lane: steps of mid-size grids, the
// compensated form, and the recomputation of stages in reverse passes.
#include <hip/hip_runtime.h>

#include "launch.hpp"
#include "step_fused.hpp"

namespace cdbm {

namespace {

typedef const __attribute__((address_space(4))) StageParams* StageTable;

// Neighbour reads of one cell.  A wave is 64 cells of one row, so the rows'
// offsets are scalar and only the five columns are vector operands: a load
// takes one scalar addition for its plane and nothing on the vector unit
// (with 64-bit addresses and the wrap's divisions these were a third of the
// stage's vector instructions).
template <typename S>
struct StageLd {
    const char* f;
    int64_t plane;       // bytes of a plane (at most 2^31)
    uint32_t row[5];     // byte offsets in a plane of the rows at offset -2 .. 2
    uint32_t col[5];     // byte offsets in a row of the columns at offset -2 .. 2
    __device__ __forceinline__ S operator()(int i, int ox, int oy) const {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<char*>(f) + i * plane, 0, (int)(uint32_t)plane, 0x00020000);
        const int v = (int)col[ox + 2], s = (int)row[oy + 2];
        if constexpr (sizeof(S) == 4) {
            return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, v, s, 0));
        } else {
            typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
            const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(rs, v, s, 0);
            return __builtin_bit_cast(double, w);
        }
    }
};

// The stencil of a velocity without its centre, upwind first: s[0..2] along x,
// s[3..5] along y.
template <typename S>
__device__ __forceinline__ void load_stencil(const StageLd<S>& ld, int i, S s[6]) {
    if (SX[i] > 0) {
        s[0] = ld(i, -2, 0); s[1] = ld(i, -1, 0); s[2] = ld(i, 1, 0);
    } else if (SX[i] < 0) {
        s[0] = ld(i, -1, 0); s[1] = ld(i, 1, 0); s[2] = ld(i, 2, 0);
    }
    if (SY[i] > 0) {
        s[3] = ld(i, 0, -2); s[4] = ld(i, 0, -1); s[5] = ld(i, 0, 1);
    } else if (SY[i] < 0) {
        s[3] = ld(i, 0, -1); s[4] = ld(i, 0, 1); s[5] = ld(i, 0, 2);
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
// The stencils of groups a and b are requested together with the cell's own
// values, so that they arrive during the moment arithmetic, and those of c
// and d (and the Heun terms) right after it; left to itself the compiler
// fetched values where it needed them, a wait each.  Bound by latencies up to
// about 384 x 384 and by the cache traffic of the stencils above; against 64-bit
// addresses and wraps by division (926 vector instructions in the mixed first
// stage, now 515): 256 x 256 mixed 6.9 -> 5.7 us, 512 x 512 compensated
// 17.4 -> 15.9 us, FP64 21.9 -> 19.3 us a stage.
template <typename S, bool STAGE2, bool COMP>
__global__ void __launch_bounds__(256) k_stage(const S* __restrict__ fin,
                                               const S* __restrict__ base, S* __restrict__ fout,
                                               const StageParams* __restrict__ Kd, int nx, int ny,
                                               int bc) {
    using A = typename std::conditional<COMP, double, S>::type;
    const int lane = threadIdx.x & 63;
    const int x = blockIdx.x * 64 + lane;
    const int y = blockIdx.y * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (y >= ny) return;
    StageLd<S> ld;
    ld.f = (const char*)fin;
    ld.plane = (int64_t)nx * ny * (int64_t)sizeof(S);
    const uint32_t pitch = (uint32_t)nx * (uint32_t)sizeof(S);
#pragma unroll
    for (int o = -2; o <= 2; ++o) {
        ld.col[o + 2] = (uint32_t)wrap_by_two(min(x, nx - 1) + o, nx, !(bc & 1)) * (uint32_t)sizeof(S);
        ld.row[o + 2] = (uint32_t)wrap_by_two(y + o, ny, !(bc & 2)) * pitch;
    }
    StageLd<S> lb = ld;
    lb.f = (const char*)base;
    S f[NV], st[NV][6], rf[4], hb[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) f[i] = ld(i, 0, 0);
    if constexpr (COMP) {
#pragma unroll
        for (int k = 0; k < 4; ++k) rf[k] = ld(NV + k, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < NV / 2; ++i) load_stencil(ld, i, st[i]);
    const StageTable K = (StageTable)(uintptr_t)Kd;
    __builtin_amdgcn_sched_barrier(0);

    double neq[NV], r[4];
    {
        double fd[NV];
#pragma unroll
        for (int i = 0; i < NV; ++i) fd[i] = (double)f[i];
        Parity g;
        to_parity(fd, g);
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
        nonequilibrium(g, m, *K, K->a, neq);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = NV / 2; i < NV; ++i) load_stencil(ld, i, st[i]);
    if constexpr (STAGE2) {
#pragma unroll
        for (int i = 0; i < NV; ++i) hb[i] = lb(i, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);

    const bool inside = x < nx;
    char* const o = (char*)fout + (int64_t)y * pitch + (int64_t)x * (int64_t)sizeof(S);
    double lost[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
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
        const A fi = (A)f[i];
        const A adv = stencil_advection<A, S>(i, st[i], fi, cx, cy);
        S v;
        if constexpr (COMP) {
            double yv = adv;
            if (STAGE2) yv += 0.5 * fi + 0.5 * (double)hb[i];
            else yv += fi;
            v = (S)fma(nz, neq[i], yv);
            lost[i] = yv - (double)v;
        } else {
            const A d = fma(nz, (A)neq[i], adv);
            v = STAGE2 ? fma(A(0.5), fi, d) : fi + d;
            if (STAGE2) v = fma(A(0.5), hb[i], v);
        }
        if (inside) *(S*)(o + i * ld.plane) = v;
    }
    if constexpr (COMP) {
        Parity gl;
        to_parity(lost, gl);
        double dm[4];
        stage_conserved(gl, K, dm);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            double rk = r[k];
            if (STAGE2) rk = 0.5 * (double)lb(NV + k, 0, 0) + 0.5 * rk;
            if (inside) *(S*)(o + (NV + k) * ld.plane) = (S)(rk + dm[k]);
        }
    }
}

template <typename S, bool COMP>
hipError_t stage_launch(const void* fin, const void* base, void* fout, bool stage2,
                        const KParams& K, const StageParams* Kd, hipStream_t st) {
    const dim3 grid((K.nx + 63) / 64, (K.ny + 3) / 4);
    const int bc = K.bcx | K.bcy << 1;
    if (stage2)
        hipLaunchKernelGGL((k_stage<S, true, COMP>), grid, dim3(256), 0, st, (const S*)fin,
                           (const S*)base, (S*)fout, Kd, K.nx, K.ny, bc);
    else
        hipLaunchKernelGGL((k_stage<S, false, COMP>), grid, dim3(256), 0, st, (const S*)fin,
                           (const S*)base, (S*)fout, Kd, K.nx, K.ny, bc);
    return hipGetLastError();
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
