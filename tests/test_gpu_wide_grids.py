"""Grids of at least 4096 columns and at most 32 rows, whose blocks of 64 cells
are numbered in bands of columns, and sizes beside that rule: the split step
against the fused step bit for bit, and the step adjoint of a periodic grid
made of copies of a small one."""
import dataclasses

import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

SIZES = [(4096, 32), (4096, 33), (4095, 32), (4160, 1), (5001, 7), (65536, 3)]


@pytest.mark.parametrize("bc_y", [W.PERIODIC, W.ZERO_GRADIENT])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_split_step_equals_fused_step(nx, ny, bc_y):
    from paper_2502_16818_amd import Solver
    from paper_2502_16818_amd.cdbm import STEP_FUSED, STEP_SPLIT
    run = W.random_periodic(nx, ny, seed=nx + ny, dt=1e-6, tau=1e-5)
    run.bc_y = bc_y
    print(f"[case] {nx}x{ny} bc_y={bc_y}", flush=True)
    for precision in (0, 1):
        a, b = (Solver.from_run(run, precision, form) for form in (STEP_FUSED, STEP_SPLIT))
        f = a.init(run.rho, run.ux, run.uy, run.T)
        want = a.step(f, nsteps=1)
        assert torch.equal(b.step(f, nsteps=1), want)
        assert torch.equal(b.step_keep_stage(f)[1], want)


@pytest.mark.parametrize("precision", [0, 1])
def test_adjoint_of_copies(precision):
    """The adjoint vector is copied bit for bit; the sum of the tau terms agrees
    to rounding (82 equal terms: far fewer than 1000 roundings of 1.1e-16 on any
    path, relative to the sum of the magnitudes)."""
    from paper_2502_16818_amd import Solver
    small = W.random_periodic(100, 15, seed=6, dt=1e-4, tau=2e-4)
    ny, nx = 2, 41
    tile = lambda a: np.tile(a, (ny, nx))
    big = dataclasses.replace(small, nx=100 * nx, ny=15 * ny, rho=tile(small.rho), ux=tile(small.ux),
                              uy=tile(small.uy), T=tile(small.T))
    print(f"[case] {big.nx}x{big.ny} precision={precision}", flush=True)
    s, b = Solver.from_run(small, precision), Solver.from_run(big, precision)
    f = s.step(s.init(small.rho, small.ux, small.uy, small.T), nsteps=2)
    lam = torch.from_numpy(np.random.default_rng(4).standard_normal((16, 15, 100))).cuda()
    want, tau = s.step_adjoint(f, lam)
    got, tau_big = b.step_adjoint(f.repeat(1, ny, nx), lam.repeat(1, ny, nx))
    assert torch.equal(got, want.repeat(1, ny, nx))
    scale = big.dt / big.tau ** 2 * float((lam.abs() * f.double().abs()).sum()) * nx * ny
    assert abs(tau_big.item() - nx * ny * tau.item()) < 1000 * 1.1e-16 * scale
