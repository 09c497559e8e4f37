// Steps of grids of about 129 x 129 to 176 x 176 (tiles of 16 x 8 cells) and 182 x
// 182 to 256 x 256 cells (16 x 16): both Runge-Kutta stages in one launch, one cell
// per lane.
#include <hip/hip_runtime.h>

#include "launch.hpp"
#include "row_block.hpp"
#include "step_fused.hpp"

namespace cdbm {

namespace {

// Reads of a tile around one cell, N cells per velocity.
template <typename S, int N>
struct TileLd {
    const S* tile;
    int here, left[2], right[2], below[2], above[2];   // cells at distance 1, 2
    __device__ __forceinline__ S operator()(int i, int ox, int oy) const {
        const int c = ox < 0 ? left[-ox - 1] : ox > 0 ? right[ox - 1]
                    : oy < 0 ? below[-oy - 1] : oy > 0 ? above[oy - 1] : here;
        return tile[i * N + c];
    }
};

constexpr int CT = 16, CW0 = CT + 8, CW1 = CT + 4;   // columns of the tile, f^n, f^(1)
template <int TY>
struct CellTile {
    static constexpr int H0 = TY + 8, N0 = CW0 * H0, N1 = CW1 * (TY + 4);
    static constexpr int CELLS1 = CT * TY + 4 * TY + 4 * CT;   // with the 2-cell strips at its sides
    static constexpr int THREADS = TY == 16 ? 512 : 384, EXTRA = N0 - THREADS;
    static_assert(CELLS1 <= THREADS && (EXTRA == 0 || (EXTRA == 64 && THREADS == 512)),
                  "a cell a thread, and two velocities of one of 64 more");
};

// One step.  A block takes a tile of 16 x TY cells: f^n of the 24 x (TY + 8) cells
// around it goes to LDS, stage 1 runs on the tile and the 2-cell strips beside its
// four sides (384 cells for TY = 16, 224 for TY = 8), stage 2 on the tile's own.
// Bound by latencies (one block per compute unit, one or two waves per SIMD): the
// loads of f^n, then two stages of about 500 instructions each.
template <typename S, int TY>
__global__ void __launch_bounds__(CellTile<TY>::THREADS, 2) k_cell_tile_step(const S* __restrict__ fin,
                                                                  const KParams* __restrict__ Kd,
                                                                  int nx, int ny, int bc,
                                                                  S* __restrict__ fout,
                                                                  S* __restrict__ f1out) {
    using G = CellTile<TY>;
    constexpr int CN0 = G::N0, CN1 = G::N1;
    __shared__ S F0[NV * CN0];
    __shared__ S F1[NV * CN1];
    const int64_t cells = (int64_t)nx * ny;
    const uint32_t per_row = (uint32_t)(nx + CT - 1) / CT;
    const uint32_t b = band_index(blockIdx.x, gridDim.x), ty = b / per_row;
    const int x0 = (int)(b - ty * per_row) * CT, y0 = (int)ty * TY;
    const int tid = threadIdx.x;
    const bool zx = bc & 1, zy = bc & 2;
    {
        const int gx = wrap_near(x0 - 4 + tid % CW0, nx, bc & 1, CW0);
        const int gy = wrap_near(y0 - 4 + tid / CW0, ny, bc >> 1, G::H0);
        const uint32_t at = (uint32_t)(gy * nx + gx) * (uint32_t)sizeof(S);
        S v[NV], w[2];
#pragma unroll
        for (int i = 0; i < NV; ++i) v[i] = *(const S*)((const char*)(fin + i * cells) + at);
        const int e = G::THREADS + (tid & 63);
        const int i0 = 2 * __builtin_amdgcn_readfirstlane(tid >> 6);
        if constexpr (G::EXTRA > 0) {
            const int ex = wrap_near(x0 - 4 + e % CW0, nx, bc & 1, CW0);
            const int ey = wrap_near(y0 - 4 + e / CW0, ny, bc >> 1, G::H0);
            const uint32_t ae = (uint32_t)(ey * nx + ex) * (uint32_t)sizeof(S);
#pragma unroll
            for (int i = 0; i < 2; ++i)
                w[i] = *(const S*)((const char*)(fin + (i0 + i) * cells) + ae);
        }
#pragma unroll
        for (int i = 0; i < NV; ++i) F0[i * CN0 + tid] = v[i];
        if constexpr (G::EXTRA > 0) {
#pragma unroll
            for (int i = 0; i < 2; ++i) F0[(i0 + i) * CN0 + e] = w[i];
        }
    }
    // the lane's cell: the tile row by row, then the strips left, right, above, below
    const int t = tid;
    int lx, ly;   // in the cells of F0
    if (t < CT * TY) {
        lx = 4 + t % CT;
        ly = 4 + t / CT;
    } else if (t < CT * TY + 4 * TY) {
        const int u = t - CT * TY, v = u % (2 * TY);
        lx = (u < 2 * TY ? 2 : CT + 4) + v % 2;
        ly = 4 + v / 2;
    } else {
        const int u = t - CT * TY - 4 * TY, v = u % (2 * CT);
        lx = 4 + v % CT;
        ly = (u < 2 * CT ? 2 : TY + 4) + v / CT;
    }
    const KParams& K = *Kd;
    S fc[NV], f1[NV];
    __syncthreads();
    if (t < G::CELLS1) {
        const int c = ly * CW0 + lx;
        const TileLd<S, CN0> ld{F0, c, {c - 1, c - 2}, {c + 1, c + 2}, {c - CW0, c - 2 * CW0},
                                {c + CW0, c + 2 * CW0}};
        stage_cell_k<S, false>(ld, K, f1);
        const int c1 = (ly - 2) * CW1 + lx - 2;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            fc[i] = F0[i * CN0 + c];
            F1[i * CN1 + c1] = f1[i];
        }
    }
    __syncthreads();
    if (t >= CT * TY) return;
    const int x = x0 + lx - 4, y = y0 + ly - 4;
    const bool inside = x < nx && y < ny;
    const uint32_t at = (uint32_t)(y * nx + x) * (uint32_t)sizeof(S);
    if (f1out != nullptr && inside) {
#pragma unroll
        for (int i = 0; i < NV; ++i) *(S*)((char*)(f1out + i * cells) + at) = f1[i];
    }
    // f^(1) at a ghost of a zero-gradient side is the edge cell's
    const int xlo = zx ? max(-2, -x0) : -2, xhi = zx ? min(CT + 1, nx - 1 - x0) : CT + 1;
    const int ylo = zy ? max(-2, -y0) : -2, yhi = zy ? min(TY + 1, ny - 1 - y0) : TY + 1;
    auto cell1 = [&](int ox, int oy) {
        const int cx = min(max(lx - 4 + ox, xlo), xhi), cy = min(max(ly - 4 + oy, ylo), yhi);
        return (cy + 2) * CW1 + cx + 2;
    };
    const TileLd<S, CN1> ld{F1, cell1(0, 0), {cell1(-1, 0), cell1(-2, 0)}, {cell1(1, 0), cell1(2, 0)},
                            {cell1(0, -1), cell1(0, -2)}, {cell1(0, 1), cell1(0, 2)}};
    S out[NV];
    stage_cell_k<S, true>(ld, K, out);
    if (inside) {
#pragma unroll
        for (int i = 0; i < NV; ++i)
            *(S*)((char*)(fout + i * cells) + at) = fma(S(0.5), fc[i], out[i]);
    }
}

int64_t cell_tiles(const KParams& K, int rows) {
    return (int64_t)((K.nx + CT - 1) / CT) * ((K.ny + rows - 1) / rows);
}
bool half_tiles_fit(const KParams& K) { return cell_tiles(K, 8) <= device_cus(); }

}  // namespace

// One block per compute unit at most, as a block's time is its latency: tiles of
// eight rows as long as they fit (us a step, mixed / FP64, against the two
// single-stage launches: 136^2 6.8 / 8.2 against 7.1 / 8.7, 160^2 6.7 / 8.2 against
// 7.3 / 9.0, 176^2 6.8 / 8.4 against 7.6 / 9.7), then of sixteen (200^2 7.7 / 10.0
// against 8.4 / 14.8, 256^2 7.6 / 10.2 against 8.6 / 11.8).  A grid of up to 2^15 cells
// that only fits in the latter has less to do in two launches, unless it is very
// narrow (tiles of sixteen rows / split: 144^2 7.5 / 7.2 and 9.8 / 8.8, 17 x 1100 9.6 /
// 8.9 and 11.8 / 11.5, 181 x 170 7.9 / 7.9 and 10.1 / 9.7; the squares from 177^2 to
// 181^2, which run split, 7.7 / 8.0 and 10.0 / 10.3; 9 x 3000 7.6 / 13.6 and 9.4 / 19.6).
bool cell_tile_fits(const KParams& K) {
    return half_tiles_fit(K) || ((int64_t)K.nx * K.ny > 1 << 15 && cell_tiles(K, 16) <= device_cus());
}

template <typename S, int TY>
hipError_t launch_cell_tile(const void* fin, void* f1out, void* fout, const KParams& K,
                            const KParams* Kd, hipStream_t st) {
    hipLaunchKernelGGL((k_cell_tile_step<S, TY>), dim3((unsigned)cell_tiles(K, TY)),
                       dim3(CellTile<TY>::THREADS), 0, st, (const S*)fin, Kd, K.nx, K.ny,
                       K.bcx | K.bcy << 1, (S*)fout, (S*)f1out);
    return hipGetLastError();
}

template <typename S>
hipError_t launch_cell_tile_step(const void* fin, void* f1out, void* fout, const KParams& K,
                                 const KParams* Kd, hipStream_t st) {
    return half_tiles_fit(K) ? launch_cell_tile<S, 8>(fin, f1out, fout, K, Kd, st)
                             : launch_cell_tile<S, 16>(fin, f1out, fout, K, Kd, st);
}

template hipError_t launch_cell_tile_step<float>(const void*, void*, void*, const KParams&,
                                                 const KParams*, hipStream_t);
template hipError_t launch_cell_tile_step<double>(const void*, void*, void*, const KParams&,
                                                  const KParams*, hipStream_t);

}  // namespace cdbm
