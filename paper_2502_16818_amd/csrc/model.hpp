// Host-side construction of the per-run constants of the CDBM step.
//
// The equilibrium of Eq. (7) is f^eq = M(u)^{-1} fbar^eq with M(u) the
// 16x16 matrix of Eq. (6) evaluated at the peculiar velocities v_i - u.
// Every row Psi_r(v - u) expands into rows of the same list with degree <= r
// (a binomial shift), so M(u) = S(u) M0 with S(u) unit lower triangular and
// M0 = M(0); then f^eq = M0^{-1} m^eq where m^eq = S(u)^{-1} fbar^eq is the
// vector of raw Maxwellian moments.  M0 depends only on the velocity set,
// so it is inverted once per run, here, and every cell applies the same
// inverse.
//
// The velocity set is symmetric under x -> -x and y -> -y.  In the basis of
// parity combinations of each group of four distributions, M0 is exactly
// block diagonal: a 6x6 block of rows even in both components
// (1, 4, 5, 7, 14, 16), two 4x4 blocks odd in one component
// (2, 8, 10, 12 and 3, 9, 11, 13) and a 2x2 block odd in both (6, 15).
// Those blocks are what the kernels contract with (72 multiply-adds per cell
// instead of 256).
#pragma once

#include <cstdint>
#include <string>

#include "../../include/cdbm.h"

namespace cdbm {

constexpr int NV = 16;

// Direction signs of the 16 discrete velocities (Eq. (2), axis groups a and
// c read as v(1,0), v(0,1), v(-1,0), v(0,-1); diagonal groups b and d as
// v(1,1), v(-1,1), v(-1,-1), v(1,-1)).
constexpr int SX[NV] = {1, 0, -1, 0, 1, -1, -1, 1, 1, 0, -1, 0, 1, -1, -1, 1};
constexpr int SY[NV] = {0, 1, 0, -1, 1, 1, -1, -1, 0, 1, 0, -1, 1, 1, -1, -1};

// The constants of a stage, packed
// in the order of use, so that they come in a few wide scalar loads: the
// groups' speeds (the rows of both momenta), the energy row, 1 / (D + I),
// D + I, then eep, ees, ioo and ioe (ieo is its mirror image); for the two
// Runge-Kutta stages the NND coefficients of velocities towards larger indices
// (groups a .. d along x, then along y) and the relaxation factors of the axis
// and the diagonal groups.
struct alignas(64) StageParams {
    double jv[4], en[4];
    double inv_a, a, eep[2][6], ees[2][4], ioo[2][2];
    double ioe[4][4];
    double cd[2][10];
    float cf[2][10];
};

// Constants handed by value to every kernel.
struct KParams {
    // Inverses of the parity blocks of M0.  Output rows are pre-multiplied by
    // 1/2 (axis groups) or 1/4 (diagonal groups), so that the unpacking of
    // parity combinations into the 16 distributions is additions only.  ieo is
    // ioe with columns 2 and 3 swapped (the x <-> y symmetry, exactly).
    double iee[6][6];
    double ioe[4][4];
    double ieo[4][4];
    double ioo[2][2];
    // The even-even block in mirror form.  The velocity set is symmetric under
    // x <-> y, which swaps unknowns 0 <-> 1 and 3 <-> 4 of the block (the
    // axis pairs of groups a and c), keeps 2 and 5 (the diagonal groups), and
    // swaps moments 2 <-> 3 and 4 <-> 5; so row 1 of iee is row 0 with those
    // columns swapped, row 4 likewise row 3, and rows 2 and 5 weigh each
    // swapped pair equally.  eep[p] (pairs p = 0: rows 0, 1; p = 1: rows 3, 4)
    // holds {B0, B1, (B2 + B3) / 2, (B4 + B5) / 2, (B2 - B3) / 2, (B4 - B5) / 2}
    // of the pair's first row B, and ees[p] (rows 2, 5) {B0, B1, B2, B4}.
    double eep[2][6];
    double ees[2][4];
    // Rows of M0 in the parity basis that give the conserved moments:
    // j_x = sum jx[k] g_oe[k], j_y = sum jy[k] g_eo[k], 2E = sum en[k] g_ee[k]
    // (rho = sum of the six even-even combinations).
    double jx[4], jy[4], en[6];
    double vx[NV], vy[NV], eta2[NV];
    double cx[NV], cy[NV];     // -dt v_ix / dx and -dt v_iy / dy
    double a;                  // D + I
    double inv_a;              // 1 / (D + I)
    double z;                  // dt / tau
    double dt, tau;
    int32_t nx, ny, bcx, bcy;
    StageParams s;             // the same constants as a stage reads them
};

// The constants of the four-lanes-per-cell kernels (step_quad.hpp).
struct alignas(64) QuadParams {
    // From these each lane forms its own: eep as in KParams, the rows of the
    // axis pairs odd along x (ioe) and along y (ieo), the NND coefficients
    // -dt v / dr of the first stage of velocities towards larger indices
    // (groups a, c along x and along y, groups b, d along x and along y) and
    // the relaxation factors of the first stage (StageParams::cd[0][8 .. 9]: -z / 2
    // of the axis groups, -z / 4 of the diagonal ones).  The rows along y (oy, and
    // ieo below) are those along x with columns 2 and 3 swapped; formed from these
    // in the kernel, 10000 cells in one row took 2.43 us a step against 2.37.
    struct Lane {
        double eep[2][6], ox[2][4], oy[2][4];
        double ax[2], ay[2], dx[2], dy[2], nz[2];
        double pad[2];
    } lane;
    // Those that all lanes use as they are: the rows of the diagonal groups b
    // and d; the speeds (the rows of the momenta, along x and along y the
    // same); the row of the energy (KParams::en, equal for an axis pair).
    struct Shared {
        struct Diag {
            double ees[4], ioe[4], ieo[4], ioo[2];
        } diag[2];
        double jv[4], en_a, en_b, en_c, en_d, a, inv_a;
        double pad[2];
    } s;
};
static_assert(sizeof(QuadParams::Lane) == 5 * 64 && sizeof(QuadParams::Shared) == 5 * 64,
              "quad_const() touches each 64-byte line");

void build_quad(const KParams& k, QuadParams& q);

// Validate p and fill k.  Returns CDBM_OK or an error code with a message.
int build_params(const cdbm_params& p, KParams& k, std::string& err);

// Field values the parameters define but the kernels do not need.
double extra_dof(double gamma);

}  // namespace cdbm
