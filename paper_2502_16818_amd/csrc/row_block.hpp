// Blocks of 64 cells of one row, one cell per lane: neighbours along x come
// from the lanes' own values through LDS, neighbours along y are loaded.
#pragma once

#include <hip/hip_runtime.h>

#include "cell.hpp"

namespace cdbm {

// Position of block b of n in a numbering whose consecutive blocks run on one
// XCD: the hardware hands blocks to the eight XCDs in turn, each with an L2 of
// its own, so blocks that share rows have to be eight apart to share a cache.
__device__ __forceinline__ uint32_t band_index(uint32_t b, uint32_t n) {
    const uint32_t per = n / 8;
    return b < 8 * per ? (b % 8) * per + b / 8 : b;
}

// The same for blocks of 64 cells of a row, in bands of row_band() blocks.  Up to
// 2^21 cells an XCD's blocks are one band of an eighth of the rows.  Above, where
// the grid outgrows the caches, eight fronts that far apart in every plane cost
// more than the shared rows give, and the bands are eight rows that follow each
// other (one band / bands of eight rows: compensated steps 1024^2 87 / 90 us,
// 2000^2 404 / 396, 4096^2 1766 / 1611; stage adjoints of an FP64 step 1024^2
// 286 / 307, 1800^2 836 / 816, 2048^2 1160 / 1076).
inline uint32_t row_band(int nx, int ny) {   // 0: one band per XCD
    return (int64_t)nx * ny <= 1 << 21 ? 0 : 8 * ((uint32_t)(nx + 63) / 64);
}
__device__ __forceinline__ uint32_t row_band_index(uint32_t b, uint32_t n, uint32_t band) {
    if (band == 0) return band_index(b, n);
    const uint32_t first = b / (8 * band) * (8 * band);
    if (first + 8 * band > n) return b;
    return first + (b - first) % 8 * band + (b - first) / 8;
}

// wrap_or_clamp for an index at most 2 off the grid.
__device__ __forceinline__ int wrap_by_two(int i, int n, bool periodic) {
    if (periodic) {
        if (n == 1) return 0;
        return i < 0 ? i + n : (i >= n ? i - n : i);
    }
    return min(max(i, 0), n - 1);
}

// The grid column of a block's column x >= -2: from two past the grid on a
// column is nobody's neighbour, and any will do.
__device__ __forceinline__ int block_column(int x, int nx, bool periodic) {
    return wrap_by_two(min(x, nx + 1), nx, periodic);
}

// Velocities with a component along x in order (three of every four: the axis
// groups have two, the diagonal ones four), and the position of velocity i
// among them.
constexpr int NVX = 12;
__device__ __forceinline__ constexpr int x_slot(int i) {
    return (i / 8) * 6 + ((i / 4) % 2 == 0 ? (i % 4) / 2 : 2 + i % 4);
}
__device__ __forceinline__ constexpr int x_velocity(int k) {
    return (k / 6) * 8 + (k % 6 < 2 ? 2 * (k % 6) : 2 + k % 6);
}
static_assert(x_slot(0) == 0 && x_slot(2) == 1 && x_slot(4) == 2 && x_slot(15) == 11 &&
                  x_velocity(1) == 2 && x_velocity(2) == 4 && x_velocity(11) == 15,
              "velocities 0, 2, 4 .. 7, 8, 10, 12 .. 15");

// The two columns on either side of the block, for n velocities in one load:
// lane 4 k + h takes column h (-2, -1, 64, 65) of the (k0 + k)-th velocity
// with a component along x.
template <typename T>
__device__ __forceinline__ T halo_value(const void* f, int k0, int n, int x0, int y, int nx,
                                        int ny, bool periodic, bool zero_ghosts) {
    const int lane = threadIdx.x & 63, h = lane & 3;
    const int i = x_velocity(k0 + min(lane >> 2, n - 1));
    const int x = x0 + (h < 2 ? h - 2 : 62 + h), cx = block_column(x, nx, periodic);
    const T v = ((const T*)f)[((int64_t)i * ny + y) * nx + cx];
    return zero_ghosts && !periodic && cx != x ? T(0) : v;
}
// Its place among the columns of a row of 2 + 64 + 2.
__device__ __forceinline__ int halo_place() {
    const int h = threadIdx.x & 3;
    return h < 2 ? h : 64 + h;
}

// Parity combinations of groups 2 q and 2 q + 1 (v: their eight values), as
// to_parity forms them.
__device__ __forceinline__ void half_parity(const double v[8], double c[8]) {
    c[0] = v[0] + v[2];
    c[1] = v[1] + v[3];
    c[2] = v[0] - v[2];
    c[3] = v[1] - v[3];
    const double s01 = v[4] + v[5], s23 = v[6] + v[7];
    const double d01 = v[4] - v[5], d23 = v[6] - v[7];
    c[4] = s01 + s23;
    c[5] = d01 - d23;
    c[6] = s01 - s23;
    c[7] = d01 + d23;
}
__device__ __forceinline__ void set_half(Parity& g, int q, const double c[8]) {
    g.ee[3 * q] = c[0];
    g.ee[3 * q + 1] = c[1];
    g.ee[3 * q + 2] = c[4];
    g.oe[2 * q] = c[2];
    g.oe[2 * q + 1] = c[5];
    g.eo[2 * q] = c[3];
    g.eo[2 * q + 1] = c[6];
    g.oo[q] = c[7];
}

}  // namespace cdbm
