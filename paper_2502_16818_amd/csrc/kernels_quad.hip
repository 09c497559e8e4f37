// Steps of small grids: both Runge-Kutta stages in one launch, four lanes per
// cell (step_quad.hpp).
#include <hip/hip_runtime.h>

#include "launch.hpp"
#include "row_block.hpp"
#include "step_quad.hpp"

namespace cdbm {

namespace {

// The arguments are plain integers and pointers, which reach the wave in
// registers (the build asks for preloaded arguments); only the constants are
// behind a pointer.  `bc` holds the boundary kinds, x in bit 0, y in bit 1.
__device__ __forceinline__ int bc_x(int bc) { return bc & 1; }
__device__ __forceinline__ int bc_y(int bc) { return bc >> 1; }
static_assert(CDBM_PERIODIC == 0 && CDBM_ZERO_GRADIENT == 1, "one bit each");

// One step of a two-dimensional grid.  A block takes a tile of 8 x TY cells (TY =
// 8 or 4): f^n of the 16 x (TY + 8) cells around it goes to LDS, stage 1 runs on
// the tile and the 2-cell strips beside its four sides (128 cells for TY = 8, one
// quad each), stage 2 on the tile's own.  The corners of the halo are not needed:
// the stencils are crosses.  Bound by latencies: of about 6.2 us from launch to launch at
// 100 x 100 in FP64, 1.6 are stage 1 (two waves per SIMD), 0.8 stage 2, the
// rest until f^n is in LDS and between the launches.  Tiles are numbered in
// bands (band_index): 100 x 100 FP64 7.6 -> 6.2 us, 128 x 128 mixed 6.5 -> 5.0.
// (The signs of the mirrored velocities, step_quad.hpp: 128 x 128 mixed 5.1 -> 5.2
// us, FP64 6.25 -> 6.28.)
// One step of 100 x 100 in FP64 14.7 -> 6.2 us against the two launches of one
// cell per lane; a call of one step on 32 x 32 (mixed) 11.3 -> 8.3 us.
constexpr int TILE = 8, TW0 = TILE + 8, TW1 = TILE + 4;   // columns of the tile, F0 and F1
template <int TY>
struct TileRows {
    static constexpr int H0 = TY + 8, N0 = TW0 * H0, H1 = TY + 4, N1 = TW1 * H1;
    static constexpr int QUADS = TILE * TY + 4 * TY + 4 * TILE;   // stage 1
    static constexpr int GROUPS = 2;   // of four velocities, that a thread loads of a cell
    static constexpr int THREADS = N0 * 4 / GROUPS;
    static_assert(GROUPS % 2 == 0 && 4 * QUADS <= THREADS && QUADS % 16 == 0 && N0 % 64 == 0, "whole waves");
};

template <typename S, int TY>
__global__ void __launch_bounds__(TileRows<TY>::THREADS) k_tile_step(const S* __restrict__ fin,
                                                            const QuadParams* __restrict__ Qd,
                                                            int nx, int ny, int bc,
                                                            S* __restrict__ fout,
                                                            S* __restrict__ f1out) {
    constexpr int TN0 = TileRows<TY>::N0, TN1 = TileRows<TY>::N1, H0 = TileRows<TY>::H0;
    __shared__ __attribute__((aligned(32))) S F0[NV * TN0];
    __shared__ __attribute__((aligned(32))) S F1[NV * TN1];
    const int64_t cells = (int64_t)nx * ny;
    const uint32_t per_row = (uint32_t)(nx + TILE - 1) / TILE;
    const uint32_t b = band_index(blockIdx.x, gridDim.x), ty = b / per_row;
    const int x0 = (int)(b - ty * per_row) * TILE, y0 = (int)ty * TY;
    const int tid = threadIdx.x, q = tid & 3;
    const QuadLane L = quad_lane(q);
    QuadConst<S> Q;
    {
        const int cell = tid % TN0;
        const int gx = wrap_near(x0 - 4 + (cell & (TW0 - 1)), nx, bc_x(bc), TW0);
        const int gy = wrap_near(y0 - 4 + cell / TW0, ny, bc_y(bc), H0);
        // a thread takes whole groups of its cell, so that each goes to LDS in
        // one piece; the planes' starts are scalar, the offset within one 32 bits
        constexpr int GRP = TileRows<TY>::GROUPS;
        const int g0 = __builtin_amdgcn_readfirstlane(tid / TN0) * GRP;
        const uint32_t off = (uint32_t)(gy * nx + gx) * (uint32_t)sizeof(S);
        typename Quad4<S>::type v[GRP];
#pragma unroll
        for (int g = 0; g < GRP; ++g)
#pragma unroll
            for (int k = 0; k < 4; ++k)
                v[g][k] = *(const S*)((const char*)(fin + (int64_t)(4 * (g0 + g) + k) * cells) + off);
        Q = quad_const<S>(Qd, L);
#pragma unroll
        for (int g = 0; g < GRP; ++g) {   // g0 is even
#pragma unroll
            for (int k = 0; k < 4; ++k) v[g][k] = quad_negated(g & 1, k) ? -v[g][k] : v[g][k];
            *(typename Quad4<S>::type*)(F0 + ((g0 + g) * TN0 + cell) * 4) = v[g];
        }
    }
    // the quad's cell: the tile row by row, then the strips left, right, above, below
    const int t = tid >> 2;
    int lx, ly;   // in the 16 x 16 cells
    if (t < TILE * TY) {
        lx = 4 + t % TILE;
        ly = 4 + t / TILE;
    } else if (t < TILE * TY + 4 * TY) {
        const int u = t - TILE * TY, v = u % (2 * TY);
        lx = (u < 2 * TY ? 2 : TILE + 4) + v % 2;
        ly = 4 + v / 2;
    } else {
        const int u = t - TILE * TY - 4 * TY, v = u % (2 * TILE);
        lx = 4 + v % TILE;
        ly = (u < 2 * TILE ? 2 : TY + 4) + v / TILE;
    }
    const bool zx = bc_x(bc) == CDBM_ZERO_GRADIENT, zy = bc_y(bc) == CDBM_ZERO_GRADIENT;
    const int xlo = zx ? max(0, 4 - x0) : 0, xhi = zx ? min(TW0 - 1, nx - 1 - x0 + 4) : TW0 - 1;
    const int ylo = zy ? max(0, 4 - y0) : 0, yhi = zy ? min(H0 - 1, ny - 1 - y0 + 4) : H0 - 1;
    const int here = ly * TW0 + lx;
    const QuadStencil st0 = quad_stencil<false>(L, lx, ly, TW0, xlo, xhi, ylo, yhi);
    __syncthreads();
    const int here1 = (ly - 2) * TW1 + lx - 2;
    S fc[4], f1[4];
    if (t < TileRows<TY>::QUADS) {   // whole waves
#pragma unroll
        for (int g = 0; g < 4; ++g) fc[g] = F0[(g * TN0 + here) * 4 + q];
        quad_stage<S, TN0, false, false>(F0, here, st0, fc, L, Q, f1);
#pragma unroll
        for (int g = 0; g < 4; ++g) F1[(g * TN1 + here1) * 4 + q] = f1[g];
    }
    __syncthreads();
    const int x = x0 + lx - 4, y = y0 + ly - 4;
    if (t >= TILE * TY) return;   // whole waves
    const bool inside = x < nx && y < ny;
    // byte offset of the cell in the plane of the lane's velocity, from group a's
    const uint32_t at = ((uint32_t)q * (uint32_t)cells + (uint32_t)(y * nx + x)) * (uint32_t)sizeof(S);
    if (f1out != nullptr && inside) {
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *(S*)((char*)(f1out + (int64_t)(4 * g) * cells) + at) = S(quad_sign(L, g)) * f1[g];
    }
    S out[4];
    {
        const QuadStencil st =
            quad_stencil<false>(L, lx - 2, ly - 2, TW1, max(xlo - 2, 0), min(xhi - 2, TW1 - 1),
                                max(ylo - 2, 0), min(yhi - 2, TileRows<TY>::H1 - 1));
        quad_stage<S, TN1, true, false>(F1, here1, st, f1, L, Q, out);
    }
    if (inside) {
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *(S*)((char*)(fout + (int64_t)(4 * g) * cells) + at) =
                S(quad_sign(L, g)) * fma(S(0.5), fc[g], out[g]);
    }
}

// `steps` steps of a grid of one row (a tube).  A block holds LINE_CELLS
// consecutive cells in LDS, one quad each; a step makes the outer four on
// either side stale, and the LINE_CELLS - 8 steps cells in the middle are
// written.  Bound by the instructions of one wave per SIMD (about 235 a
// stage, 0.55 us).  Per step, FP64, 500 cells: 10.1 -> 1.8 us against the two
// single-stage launches; mixed, 10000 cells: 9.4 -> 2.2 us.
constexpr int LINE_CELLS = 64;

template <typename S>
__global__ void __launch_bounds__(4 * LINE_CELLS) k_line_steps(const S* __restrict__ fin,
                                                               const QuadParams* __restrict__ Qd,
                                                               int nx, int bc, int steps,
                                                               S* __restrict__ fout) {
    constexpr int W = LINE_CELLS;
    __shared__ __attribute__((aligned(32))) S F0[NV * W];
    __shared__ __attribute__((aligned(32))) S F1[NV * W];
    const int x0 = (int)band_index(blockIdx.x, gridDim.x) * (W - 8 * steps) - 4 * steps;
    const int tid = threadIdx.x, q = tid & 3, lx = tid >> 2;
    const QuadLane L = quad_lane(q);
    QuadConst<S> Q;
    {
        const int cell = tid & (W - 1), g = __builtin_amdgcn_readfirstlane(tid / W);
        const uint32_t off =
            (uint32_t)wrap_near(x0 + cell, nx, bc_x(bc), W) * (uint32_t)sizeof(S);
        typename Quad4<S>::type v;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            v[k] = *(const S*)((const char*)(fin + (int64_t)(4 * g + k) * nx) + off);
        Q = quad_const<S>(Qd, L);
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = quad_negated(g & 1, k) ? -v[k] : v[k];
        *(typename Quad4<S>::type*)(F0 + (g * W + cell) * 4) = v;
    }
    const bool zx = bc_x(bc) == CDBM_ZERO_GRADIENT;
    const int xlo = zx ? min(max(0, -x0), W - 1) : 0;
    const int xhi = zx ? min(W - 1, nx - 1 - x0) : W - 1;
    const QuadStencil st = quad_stencil<true>(L, lx, 0, W, xlo, xhi, 0, 0);
    __syncthreads();
    S fc[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) fc[g] = F0[(g * W + lx) * 4 + q];
    for (int s = 0; s < steps; ++s) {
        S f1[4], out[4];
        quad_stage<S, W, false, true>(F0, lx, st, fc, L, Q, f1);
#pragma unroll
        for (int g = 0; g < 4; ++g) F1[(g * W + lx) * 4 + q] = f1[g];
        __syncthreads();
        quad_stage<S, W, true, true>(F1, lx, st, f1, L, Q, out);
#pragma unroll
        for (int g = 0; g < 4; ++g) fc[g] = fma(S(0.5), fc[g], out[g]);
        if (s + 1 < steps) {
#pragma unroll
            for (int g = 0; g < 4; ++g) F0[(g * W + lx) * 4 + q] = fc[g];
            __syncthreads();
        }
    }
    const int x = x0 + lx;
    if (lx >= 4 * steps && lx < W - 4 * steps && x < nx) {
        const uint32_t at = (uint32_t)(q * nx + x) * (uint32_t)sizeof(S);
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *(S*)((char*)(fout + (int64_t)(4 * g) * nx) + at) = S(quad_sign(L, g)) * fc[g];
    }
}

}  // namespace

// One block per compute unit at most: a block's stages are bound by the
// latency of two waves per SIMD, and with a second round of blocks the two
// launches of the single-stage kernels are faster (mixed / FP64: 128 x 128,
// 256 blocks, 5.2 / 6.3 us against 6.3 / 7.1; 144 x 144, 324 blocks, 7.9 / 9.9
// against 7.3 / 8.8; 160 x 160 7.8 / 9.7 against 7.3 / 9.0).
bool tile_step_fits(const KParams& K) {
    return (int64_t)((K.nx + TILE - 1) / TILE) * ((K.ny + TILE - 1) / TILE) <= device_cus();
}

// Time of a launch of k steps, in us: about 3 + 1.3 k with at most one block per
// compute unit, whose waves are bound by their own latency, and 3 + r (k + 0.3) with
// r of them on the fullest one, which share its SIMDs (FP64; mixed about 0.85 of the
// part after the 3, which moves no choice).  More steps per launch mean fewer
// cells written per block.  Measured per step for k = 1 .. 7 (FP64), at 500 cells
// 4.5 2.8 2.3 2.1 1.9 1.8 1.7, 10000 cells 4.7 2.9 2.4 2.9 2.7 3.5 5.3, 12000 cells
// 4.7 3.0 3.2 2.9 2.8 3.6 6.2, 20000 cells 5.7 3.8 3.3 3.8 4.6 5.4 9.9, 65536 cells
// 9.9 8.4 8.4 8.9 11.3 15.7 30.4; mixed 12000 cells 4.1 2.6 2.8 2.6 2.4 3.0 5.3, 65536
// cells 8.2 6.9 7.1 7.4 9.4 13.0 25.0.  At 16 lengths from 64 to 65536 the choice is the
// fastest of the seven in both precisions.
int line_steps_per_launch(const KParams& K) {
    if (K.ny != 1) return 0;
    const int cus = device_cus();
    int best = 1;
    double cost = 0.0;
    for (int k = 1; 8 * k < LINE_CELLS; ++k) {
        const int out = LINE_CELLS - 8 * k;
        const int blocks = (K.nx + out - 1) / out, rounds = (blocks + cus - 1) / cus;
        const double c = (3.0 + (rounds == 1 ? 1.3 * k : rounds * (k + 0.3))) / k;
        if (k == 1 || c < cost) {
            cost = c;
            best = k;
        }
    }
    return best;
}

template <typename S, int TY>
hipError_t launch_tile_rows(const void* fin, void* f1out, void* fout, const KParams& K,
                            const QuadParams* Qd, hipStream_t st) {
    const dim3 grid(((K.nx + TILE - 1) / TILE) * ((K.ny + TY - 1) / TY));
    hipLaunchKernelGGL((k_tile_step<S, TY>), grid, dim3(TileRows<TY>::THREADS), 0, st,
                       (const S*)fin, Qd, K.nx, K.ny, K.bcx | K.bcy << 1, (S*)fout, (S*)f1out);
    return hipGetLastError();
}

template <typename S>
hipError_t launch_tile_step(const void* fin, void* f1out, void* fout, const KParams& K,
                            const QuadParams* Qd, hipStream_t st) {
    // Tiles of four rows while there is at most one per compute unit: a tile of
    // eight has two waves per SIMD in stage 1, one of four little more than one
    // (32 x 32 mixed 4.59 -> 4.45 us, FP64 5.42 -> 4.91; 88 x 88 FP64 5.85 -> 5.38);
    // a second round costs more (96 x 96 mixed 7.0 against 4.9).
    if ((int64_t)((K.nx + TILE - 1) / TILE) * ((K.ny + 3) / 4) <= device_cus())
        return launch_tile_rows<S, 4>(fin, f1out, fout, K, Qd, st);
    return launch_tile_rows<S, TILE>(fin, f1out, fout, K, Qd, st);
}

template <typename S>
hipError_t launch_line_steps(const void* fin, void* fout, int steps, const KParams& K,
                             const QuadParams* Qd, hipStream_t st) {
    const int out = LINE_CELLS - 8 * steps;
    hipLaunchKernelGGL(k_line_steps<S>, dim3((K.nx + out - 1) / out), dim3(4 * LINE_CELLS), 0, st,
                       (const S*)fin, Qd, K.nx, K.bcx, steps, (S*)fout);
    return hipGetLastError();
}

#define CDBM_INSTANTIATE(S)                                                                       \
    template hipError_t launch_tile_step<S>(const void*, void*, void*, const KParams&,           \
                                            const QuadParams*, hipStream_t);                        \
    template hipError_t launch_line_steps<S>(const void*, void*, int, const KParams&,            \
                                             const QuadParams*, hipStream_t);
CDBM_INSTANTIATE(float)
CDBM_INSTANTIATE(double)
#undef CDBM_INSTANTIATE

}  // namespace cdbm
