"""The one-launch step on 16 x 16 tiles (grids of more than 2^15 cells and up to
one tile per compute unit) against the single-stage kernels: the same
arithmetic per cell, equal bit for bit.  Whole and partial tiles, a grid
narrower than a tile's surroundings, and sizes on both sides of the rule."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bc_x,bc_y", [(0, 0), (1, 1), (0, 1), (1, 0)])
@pytest.mark.parametrize("nx,ny", [(256, 128), (182, 181), (256, 256), (249, 241), (17, 2000),
                                   (11, 4000), (4000, 9), (257, 256)])
def test_tiles_equal_single_stages(nx, ny, bc_x, bc_y):
    from paper_2502_16818_amd import Solver
    from paper_2502_16818_amd.cdbm import STEP_AUTO, STEP_SPLIT
    run = W.random_periodic(nx, ny, seed=nx + ny, dt=1e-6, tau=1e-5)
    run.bc_x, run.bc_y = bc_x, bc_y
    for precision in (0, 1):
        print(f"[case] {nx}x{ny} bc=({bc_x},{bc_y}) precision={precision}", flush=True)
        a, b = (Solver.from_run(run, precision, form) for form in (STEP_AUTO, STEP_SPLIT))
        f = a.init(run.rho, run.ux, run.uy, run.T)
        for steps in (1, 3, 34):
            assert torch.equal(a.step(f, nsteps=steps), b.step(f, nsteps=steps))
        for x, y in zip(a.step_keep_stage(f), b.step_keep_stage(f)):
            assert torch.equal(x, y)


@pytest.mark.parametrize("bc", [0, 1])
@pytest.mark.parametrize("nx,ny", [(136, 136), (176, 180), (181, 170), (17, 1020), (2000, 15), (5, 2040)])
def test_half_tiles_equal_single_stages(nx, ny, bc):
    """16 x 8 tiles, up to one per compute unit."""
    test_tiles_equal_single_stages(nx, ny, bc, 1 - bc if nx % 2 else bc)
