// Point-wise kernels of the CDBM library: initial
// equilibrium, field checks, macroscopic moments, nonequilibrium measures and
// conserved totals.
#include <hip/hip_runtime.h>

#include "cell.hpp"
#include "launch.hpp"

namespace cdbm {

namespace {

// f = f^eq(rho, u, T) per cell (the initial condition of Sec. 3).
template <typename S>
__global__ void __launch_bounds__(256) k_init(const double* __restrict__ rho,
                                              const double* __restrict__ ux,
                                              const double* __restrict__ uy,
                                              const double* __restrict__ T, S* __restrict__ f,
                                              KParams K, int64_t cells) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= cells) return;
    Macro m{rho[c], ux[c], uy[c], T[c]};
    double feq[NV];
    equilibrium(m, K, K.a, feq);
#pragma unroll
    for (int i = 0; i < NV; ++i) f[i * cells + c] = (S)feq[i];
}

// bad |= 1 if rho <= 0, T <= 0 or any field value is not finite.
__global__ void __launch_bounds__(256) k_check_fields(const double* __restrict__ rho,
                                                      const double* __restrict__ ux,
                                                      const double* __restrict__ uy,
                                                      const double* __restrict__ T,
                                                      int64_t cells, int* __restrict__ bad) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= cells) return;
    const double r = rho[c], a = ux[c], b = uy[c], t = T[c];
    const bool ok = isfinite(r) && isfinite(a) && isfinite(b) && isfinite(t) && r > 0.0 && t > 0.0;
    if (!ok) atomicOr(bad, 1);
}

template <typename S>
__device__ __forceinline__ void load_cell(const S* __restrict__ f, int64_t cells, int64_t c,
                                          double fd[NV]) {
#pragma unroll
    for (int i = 0; i < NV; ++i) fd[i] = (double)f[i * cells + c];
}

// The compensated mixed form (CDBM_MIXED_COMP): a state holds the 16 planes
// of f in float and then the four planes of r, the part of the cell's
// (rho, j_x, j_y, 2E) that float storage of f rounded off.

// (rho, j_x, j_y, 2E) of the distributions whose parity combinations are g.
__device__ __forceinline__ void conserved_of(const Parity& g, const KParams& K, double out[4]) {
    out[0] = ((g.ee[0] + g.ee[1]) + (g.ee[2] + g.ee[3])) + (g.ee[4] + g.ee[5]);
    double jx = 0.0, jy = 0.0, e2 = 0.0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        jx = fma(K.jx[c], g.oe[c], jx);
        jy = fma(K.jy[c], g.eo[c], jy);
    }
#pragma unroll
    for (int c = 0; c < 6; ++c) e2 = fma(K.en[c], g.ee[c], e2);
    out[1] = jx;
    out[2] = jy;
    out[3] = e2;
}

// Macroscopic fields of a compensated cell: the conserved moments of its
// stored f plus its residual r.
__device__ __forceinline__ Macro macro_compensated(const Parity& g, const double r[4],
                                                   const KParams& K) {
    double q[4];
    conserved_of(g, K, q);
    const double rho = q[0] + r[0];
    Macro m;
    m.rho = rho;
    m.ux = (q[1] + r[1]) / rho;
    m.uy = (q[2] + r[2]) / rho;
    m.T = ((q[3] + r[3]) / rho - (m.ux * m.ux + m.uy * m.uy)) * K.inv_a;
    return m;
}

__device__ __forceinline__ void load_residual(const float* __restrict__ f, int64_t cells,
                                              int64_t c, double r[4]) {
#pragma unroll
    for (int k = 0; k < 4; ++k) r[k] = (double)f[(NV + k) * cells + c];
}

// Compensated initial state: f = f^eq rounded to float, r = the conserved
// moments of what the rounding removed.
__global__ void __launch_bounds__(256) k_init_comp(const double* __restrict__ rho,
                                                   const double* __restrict__ ux,
                                                   const double* __restrict__ uy,
                                                   const double* __restrict__ T,
                                                   float* __restrict__ f, KParams K,
                                                   int64_t cells) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= cells) return;
    Macro m{rho[c], ux[c], uy[c], T[c]};
    double feq[NV], lost[NV];
    equilibrium(m, K, K.a, feq);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const float v = (float)feq[i];
        f[i * cells + c] = v;
        lost[i] = feq[i] - (double)v;
    }
    Parity g;
    to_parity(lost, g);
    double r[4];
    conserved_of(g, K, r);
#pragma unroll
    for (int k = 0; k < 4; ++k) f[(NV + k) * cells + c] = (float)r[k];
}

template <typename S, bool COMP = false>
__global__ void __launch_bounds__(256) k_moments(const S* __restrict__ f, double* __restrict__ rho,
                                                 double* __restrict__ ux, double* __restrict__ uy,
                                                 double* __restrict__ T, KParams K, int64_t cells) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= cells) return;
    double fd[NV];
    load_cell(f, cells, c, fd);
    Parity g;
    to_parity(fd, g);
    Macro m;
    if constexpr (COMP) {
        double r[4];
        load_residual(f, cells, c, r);
        m = macro_compensated(g, r, K);
    } else {
        m = macro_from_parity(g, K, K.inv_a);
    }
    rho[c] = m.rho;
    ux[c] = m.ux;
    uy[c] = m.uy;
    T[c] = m.T;
}

// Eqs. (8)-(11): sum_i (f_i - f_i^eq) Psi_r(v_i - u), rows r = 5..16.
// RAW: the measures of the raw-moment construction, Psi_r(v_i) at the raw
// velocities (same f^eq).
// COMP: f^eq of the compensated moments, f the stored float distributions.
template <typename S, bool RAW, bool COMP = false>
__global__ void __launch_bounds__(256) k_tne(const S* __restrict__ f, double* __restrict__ out,
                                             KParams K, int64_t cells) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= cells) return;
    double fd[NV];
    load_cell(f, cells, c, fd);
    Parity g;
    to_parity(fd, g);
    Macro m;
    if constexpr (COMP) {
        double r[4];
        load_residual(f, cells, c, r);
        m = macro_compensated(g, r, K);
    } else {
        m = macro_from_parity(g, K, K.inv_a);
    }
    double feq[NV];
    equilibrium(m, K, K.a, feq);
    double acc[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) acc[k] = 0.0;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const double d = fd[i] - feq[i];
        const double cx = RAW ? K.vx[i] : K.vx[i] - m.ux, cy = RAW ? K.vy[i] : K.vy[i] - m.uy;
        const double e = cx * cx + cy * cy + K.eta2[i];
        const double xx = cx * cx, xy = cx * cy, yy = cy * cy;
        acc[0] = fma(d, xx, acc[0]);
        acc[1] = fma(d, xy, acc[1]);
        acc[2] = fma(d, yy, acc[2]);
        acc[3] = fma(d, e * cx, acc[3]);
        acc[4] = fma(d, e * cy, acc[4]);
        acc[5] = fma(d, xx * cx, acc[5]);
        acc[6] = fma(d, xx * cy, acc[6]);
        acc[7] = fma(d, xy * cy, acc[7]);
        acc[8] = fma(d, yy * cy, acc[8]);
        acc[9] = fma(d, e * xx, acc[9]);
        acc[10] = fma(d, e * xy, acc[10]);
        acc[11] = fma(d, e * yy, acc[11]);
    }
#pragma unroll
    for (int k = 0; k < 12; ++k) out[k * cells + c] = acc[k];
}

// Per-block partial sums of (rho, j_x, j_y, 2E); block count is fixed.  A cell's
// values are formed from its parity combinations (sums and differences of
// opposite velocities first) and its successor's are requested before that.
// Bound by memory, the write-back of what the kernel before it left in the
// last-level cache included; that kernel went through the state front to back,
// so this one starts at the end, of which a part is still there.  After the
// twelve non-equilibrium measures of 2048^2 mixed (268 MB of state, 402 MB of
// results): front to back 84 us, from the end 73 us (the measures themselves
// read from the end did not gain: 118 us both ways).
template <typename S, bool COMP = false>
__global__ void __launch_bounds__(256) k_totals_partial(const S* __restrict__ f, KParams K,
                                                        int64_t cells, double* __restrict__ part) {
    constexpr int PLANES = COMP ? NV + 4 : NV;
    __shared__ double red[4][4];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    int64_t c = (cells - 1) / step * step + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= cells) c -= step;
    S next[PLANES];
    if (c >= 0) {
#pragma unroll
        for (int i = 0; i < PLANES; ++i) next[i] = f[i * cells + c];
    }
    for (; c >= 0; c -= step) {
        S v[PLANES];
#pragma unroll
        for (int i = 0; i < PLANES; ++i) v[i] = next[i];
        if (c >= step) {
#pragma unroll
            for (int i = 0; i < PLANES; ++i) next[i] = f[i * cells + c - step];
        }
        double fd[NV], q[4];
#pragma unroll
        for (int i = 0; i < NV; ++i) fd[i] = (double)v[i];
        Parity g;
        to_parity(fd, g);
        conserved_of(g, K, q);
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[k] += COMP ? q[k] + (double)v[NV + (COMP ? k : -1)] : q[k];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) acc[k] += __shfl_xor(acc[k], o);
        if (lane == 0) red[k][w] = acc[k];
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        const double* r = red[threadIdx.x];
        part[blockIdx.x * 4 + threadIdx.x] = (r[0] + r[1]) + (r[2] + r[3]);
    }
}

// out[k] = sum over blocks of part[4 b + k], in a fixed order: wave k of the one
// block, four loads in flight per lane.
__global__ void __launch_bounds__(256) k_sum_partials(const double* __restrict__ part, int nblocks,
                                                      double* __restrict__ out) {
    const int lane = threadIdx.x & 63, k = threadIdx.x >> 6;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    for (int b = lane; b < nblocks; b += 256) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (b + 64 * j < nblocks) s[j] += part[(b + 64 * j) * 4 + k];
    }
    double t = (s[0] + s[1]) + (s[2] + s[3]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o);
    if (lane == 0) out[k] = t;
}

inline unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

}  // namespace

template <typename S>
hipError_t launch_init(const double* rho, const double* ux, const double* uy, const double* T,
                       void* f, const KParams& K, hipStream_t st) {
    const int64_t cells = (int64_t)K.nx * K.ny;
    hipLaunchKernelGGL(k_init<S>, dim3(blocks_for(cells, 256)), dim3(256), 0, st, rho, ux, uy, T,
                       (S*)f, K, cells);
    return hipGetLastError();
}

hipError_t launch_check_fields(const double* rho, const double* ux, const double* uy,
                               const double* T, int64_t cells, int* bad, hipStream_t st) {
    hipLaunchKernelGGL(k_check_fields, dim3(blocks_for(cells, 256)), dim3(256), 0, st, rho, ux, uy,
                       T, cells, bad);
    return hipGetLastError();
}

template <typename S>
hipError_t launch_moments(const void* f, double* rho, double* ux, double* uy, double* T,
                          const KParams& K, hipStream_t st) {
    const int64_t cells = (int64_t)K.nx * K.ny;
    hipLaunchKernelGGL(k_moments<S>, dim3(blocks_for(cells, 256)), dim3(256), 0, st,
                       (const S*)f, rho, ux, uy, T, K, cells);
    return hipGetLastError();
}

template <typename S>
hipError_t launch_tne(const void* f, double* out12, bool raw, const KParams& K, hipStream_t st) {
    const int64_t cells = (int64_t)K.nx * K.ny;
    if (raw)
        hipLaunchKernelGGL((k_tne<S, true>), dim3(blocks_for(cells, 256)), dim3(256), 0, st,
                           (const S*)f, out12, K, cells);
    else
        hipLaunchKernelGGL((k_tne<S, false>), dim3(blocks_for(cells, 256)), dim3(256), 0, st,
                           (const S*)f, out12, K, cells);
    return hipGetLastError();
}

template <typename S>
hipError_t launch_totals(const void* f, double* partials, int nblocks, double* out4,
                         const KParams& K, hipStream_t st) {
    const int64_t cells = (int64_t)K.nx * K.ny;
    hipLaunchKernelGGL(k_totals_partial<S>, dim3(nblocks), dim3(256), 0, st, (const S*)f, K,
                       cells, partials);
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(256), 0, st, partials, nblocks, out4);
    return hipGetLastError();
}

hipError_t launch_init_comp(const double* rho, const double* ux, const double* uy,
                            const double* T, void* f, const KParams& K, hipStream_t st) {
    const int64_t cells = (int64_t)K.nx * K.ny;
    hipLaunchKernelGGL(k_init_comp, dim3(blocks_for(cells, 256)), dim3(256), 0, st, rho, ux, uy,
                       T, (float*)f, K, cells);
    return hipGetLastError();
}

hipError_t launch_moments_comp(const void* f, double* rho, double* ux, double* uy, double* T,
                               const KParams& K, hipStream_t st) {
    const int64_t cells = (int64_t)K.nx * K.ny;
    hipLaunchKernelGGL((k_moments<float, true>), dim3(blocks_for(cells, 256)), dim3(256), 0, st,
                       (const float*)f, rho, ux, uy, T, K, cells);
    return hipGetLastError();
}

hipError_t launch_tne_comp(const void* f, double* out12, bool raw, const KParams& K,
                           hipStream_t st) {
    const int64_t cells = (int64_t)K.nx * K.ny;
    if (raw)
        hipLaunchKernelGGL((k_tne<float, true, true>), dim3(blocks_for(cells, 256)), dim3(256), 0,
                           st, (const float*)f, out12, K, cells);
    else
        hipLaunchKernelGGL((k_tne<float, false, true>), dim3(blocks_for(cells, 256)), dim3(256), 0,
                           st, (const float*)f, out12, K, cells);
    return hipGetLastError();
}

hipError_t launch_totals_comp(const void* f, double* partials, int nblocks, double* out4,
                              const KParams& K, hipStream_t st) {
    const int64_t cells = (int64_t)K.nx * K.ny;
    hipLaunchKernelGGL((k_totals_partial<float, true>), dim3(nblocks), dim3(256), 0, st,
                       (const float*)f, K, cells, partials);
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(256), 0, st, partials, nblocks, out4);
    return hipGetLastError();
}

#define CDBM_INSTANTIATE(S)                                                                     \
    template hipError_t launch_init<S>(const double*, const double*, const double*,            \
                                       const double*, void*, const KParams&, hipStream_t);     \
    template hipError_t launch_moments<S>(const void*, double*, double*, double*, double*,     \
                                          const KParams&, hipStream_t);                        \
    template hipError_t launch_tne<S>(const void*, double*, bool, const KParams&, hipStream_t);      \
    template hipError_t launch_totals<S>(const void*, double*, int, double*, const KParams&,   \
                                         hipStream_t);
CDBM_INSTANTIATE(float)
CDBM_INSTANTIATE(double)
#undef CDBM_INSTANTIATE

}  // namespace cdbm
