// Fused FP64 step of large grids by marching strips (step_march.hpp).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "launch.hpp"
#include "step_march.hpp"

namespace cdbm {

namespace {

// Block b in band order takes strip b % nstrips of the (b / nstrips)-th piece of
// `len` rows, so neighbouring strips of a piece share an XCD's L2.
__global__ void __launch_bounds__(128, 2) k_step_march(const double* __restrict__ fin,
                                                       double* __restrict__ fout,
                                                       const StageParams* __restrict__ Kd, int nx,
                                                       int ny, int bc, int len) {
    __shared__ MarchLds lds;
    const uint32_t nstrips = (uint32_t)(nx + MARCH_TX - 1) / MARCH_TX;
    const uint32_t b = band_index(blockIdx.x, gridDim.x), p = b / nstrips;
    const int x0 = (int)(b - p * nstrips) * MARCH_TX, ya = (int)p * len, yb = min(ny, ya + len);
    const int part = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const MarchTable K = (MarchTable)(uintptr_t)Kd;
    const bool edge = ((bc & 1) && (x0 < 4 || x0 + MARCH_TX + 4 > nx)) ||
                      ((bc & 2) && (ya < 4 || yb + 4 > ny));
    if (edge)
        march_strip<true>(fin, fout, K, nx, ny, bc & 1, bc >> 1, x0, ya, yb, part, lds);
    else
        march_strip<false>(fin, fout, K, nx, ny, bc & 1, bc >> 1, x0, ya, yb, part, lds);
}

// Blocks a compute unit holds: two waves per SIMD at 256 registers.  More
// blocks than that in one round leave the rest a round of their own (2048 x
// 1536, blocks per unit 3 / 4 / 5 / 6: 220 / 200 / 239 / 241 us).
constexpr int MARCH_BLOCKS = 4;
// Rows of a piece that are read, and rows of stage 1, past its ends.
constexpr int MARCH_FILL = 8;

}  // namespace

hipError_t launch_step_march(const void* fin, void* fout, const KParams& K, const StageParams* Kd,
                             hipStream_t st) {
    const int nstrips = (K.nx + MARCH_TX - 1) / MARCH_TX;
    const int64_t resident = (int64_t)device_cus() * MARCH_BLOCKS;
    // the pieces per strip that fill one to four rounds: the cheapest
    int len = K.ny;
    int64_t cost = -1;
    for (int r = 1; r <= 4; ++r) {
        const int64_t p = std::min<int64_t>(r * resident / nstrips, (K.ny + 15) / 16);
        if (p < 1) continue;
        const int l = (int)((K.ny + p - 1) / p);
        const int64_t blocks = (int64_t)nstrips * ((K.ny + l - 1) / l);
        const int64_t c = (blocks + resident - 1) / resident * (l + MARCH_FILL);
        if (cost < 0 || c < cost) {
            cost = c;
            len = l;
        }
    }
    const unsigned pieces = (unsigned)((K.ny + len - 1) / len);
    hipLaunchKernelGGL(k_step_march, dim3((unsigned)nstrips * pieces), dim3(128), 0, st,
                       (const double*)fin, (double*)fout, Kd, K.nx, K.ny, K.bcx | K.bcy << 1, len);
    return hipGetLastError();
}

}  // namespace cdbm
