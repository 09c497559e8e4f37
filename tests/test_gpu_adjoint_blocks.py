"""Stage adjoint at the edges of its blocks (64 cells of a row, x neighbours
through LDS with two halo columns on either side) against the oracle's
reverse-mode derivative.  Tolerance as in the other FP64 adjoint tests: a few
hundred roundings of 1.1e-16 on values of the size of the largest."""
import numpy as np
import pytest
import torch

from oracle import cdbm as C
import workloads as W
from helpers import oracle_f0, rel_max, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bc_x", [W.PERIODIC, W.ZERO_GRADIENT])
@pytest.mark.parametrize("nx,ny", [(1, 3), (2, 2), (62, 3), (63, 1), (64, 2), (65, 5), (66, 4),
                                   (127, 2), (129, 1)])
def test_block_edges_match_oracle(nx, ny, bc_x):
    from paper_2502_16818_amd import Solver
    run = W.random_periodic(nx, ny, seed=nx + ny, dt=1e-4, tau=2e-4)
    run.bc_x, run.bc_y = bc_x, bc_x if ny % 2 else W.ZERO_GRADIENT
    print(f"[case] {nx}x{ny} bc=({run.bc_x},{run.bc_y})", flush=True)
    p, f0 = oracle_f0(run)
    f = C.run(f0, p, 2)
    lam = torch.from_numpy(np.random.default_rng(21).standard_normal(f.shape))
    want_l, want_tau = C.step_vjp(f, lam, p)
    s = Solver.from_run(run, 0)
    got_l, dtau = s.step_adjoint(f.contiguous().cuda(), lam.cuda())
    assert rel_max(to_np(got_l), want_l.numpy()) < 1e-11
    # standard normal lam against f - f^eq: the sum cancels to about the root of its terms
    f1 = f + p.dt * C.rhs(f, p)
    scale = p.dt / p.tau ** 2 * float((lam.abs() * f1.abs()).sum())
    assert abs(float(dtau.item()) - want_tau) < 1e-13 * scale


@pytest.mark.parametrize("precision", [0, 1])
def test_large_grid_repeats_small_grid(precision):
    """More than 2^21 cells (blocks numbered in short bands): a periodic grid made
    of copies of a small one has its adjoint vector copied bit for bit, and the
    sum of its tau terms to rounding (300 equal terms: far fewer than 1000
    roundings of 1.1e-16 on any path, relative to the sum of the magnitudes)."""
    from paper_2502_16818_amd import Solver
    import dataclasses
    small = W.random_periodic(100, 75, seed=5, dt=1e-4, tau=2e-4)
    ny, nx = 20, 15
    tile = lambda a: np.tile(a, (ny, nx))
    big = dataclasses.replace(small, nx=100 * nx, ny=75 * ny, rho=tile(small.rho), ux=tile(small.ux),
                              uy=tile(small.uy), T=tile(small.T))
    print(f"[case] {big.nx}x{big.ny} precision={precision}", flush=True)
    s, b = Solver.from_run(small, precision), Solver.from_run(big, precision)
    f = s.step(s.init(small.rho, small.ux, small.uy, small.T), nsteps=2)
    lam = torch.from_numpy(np.random.default_rng(3).standard_normal((16, 75, 100))).cuda()
    want, tau = s.step_adjoint(f, lam)
    got, tau_big = b.step_adjoint(f.repeat(1, ny, nx), lam.repeat(1, ny, nx))
    assert torch.equal(got, want.repeat(1, ny, nx))
    scale = big.dt / big.tau ** 2 * float((lam.abs() * f.double().abs()).sum()) * nx * ny
    assert abs(tau_big.item() - nx * ny * tau.item()) < 1000 * 1.1e-16 * scale
