"""The one-launch step of small grids on tiles of four and of eight rows (four
while 8 x 4 tiles are at most one per compute unit) against the single-stage
kernels: equal bit for bit.  Whole and partial tiles, grids smaller than a tile's
surroundings, and both sides of the rule (88 x 92: 253 tiles; 90 x 88: 264)."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bc_x,bc_y", [(0, 0), (1, 1), (0, 1), (1, 0)])
@pytest.mark.parametrize("nx,ny", [(1, 2), (3, 5), (8, 4), (9, 13), (7, 1000), (2000, 3), (88, 92),
                                   (90, 88)])
def test_tiles_equal_single_stages(nx, ny, bc_x, bc_y):
    from paper_2502_16818_amd import Solver
    from paper_2502_16818_amd.cdbm import STEP_AUTO, STEP_SPLIT
    run = W.random_periodic(nx, ny, seed=nx + ny, dt=1e-6, tau=1e-5)
    run.bc_x, run.bc_y = bc_x, bc_y
    for precision in (0, 1):
        print(f"[case] {nx}x{ny} bc=({bc_x},{bc_y}) precision={precision}", flush=True)
        a, b = (Solver.from_run(run, precision, form) for form in (STEP_AUTO, STEP_SPLIT))
        f = a.init(run.rho, run.ux, run.uy, run.T)
        for steps in (1, 3, 35):
            assert torch.equal(a.step(f, nsteps=steps), b.step(f, nsteps=steps))
        for x, y in zip(a.step_keep_stage(f), b.step_keep_stage(f)):
            assert torch.equal(x, y)
