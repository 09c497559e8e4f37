"""The marching fused FP64 step (grids of 700000 cells and more) against the
single-stage kernels: the same arithmetic per cell, equal bit for bit.  Widths
around a multiple of the 56-column strips, a grid narrower than a strip with its
halo, more strips than resident blocks, and the smallest size of the rule with
one below it."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

SIZES = [(1000, 700), (1000, 699), (728, 1000), (729, 970), (783, 901), (11, 65000),
         (60000, 12), (65536, 11)]


@pytest.mark.parametrize("bc_x,bc_y", [(0, 0), (1, 1), (0, 1), (1, 0)])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_march_equals_single_stages(nx, ny, bc_x, bc_y):
    from paper_2502_16818_amd import Solver
    from paper_2502_16818_amd.cdbm import STEP_FUSED, STEP_SPLIT
    run = W.random_periodic(nx, ny, seed=nx + ny, dt=1e-6, tau=1e-5)
    run.bc_x, run.bc_y = bc_x, bc_y
    print(f"[case] {nx}x{ny} bc=({bc_x},{bc_y})", flush=True)
    a, b = (Solver.from_run(run, 0, form) for form in (STEP_FUSED, STEP_SPLIT))
    f = a.init(run.rho, run.ux, run.uy, run.T)
    for steps in (1, 3):
        assert torch.equal(a.step(f, nsteps=steps), b.step(f, nsteps=steps))
