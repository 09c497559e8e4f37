"""Grids of more than 98304 cells in at most 32 rows, whose single stages take
their blocks of 64 cells in bands of columns, and sizes beside that rule: the
split step against the fused step, bit for bit, and the compensated step
against FP64."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bc_y", [W.PERIODIC, W.ZERO_GRADIENT])
@pytest.mark.parametrize("nx,ny", [(3073, 32), (3072, 32), (3073, 33), (14044, 7), (65536, 2), (65536, 3)])
def test_split_step_equals_fused_step(nx, ny, bc_y):
    from paper_2502_16818_amd import Solver
    from paper_2502_16818_amd.cdbm import STEP_FUSED, STEP_SPLIT
    run = W.random_periodic(nx, ny, seed=nx + ny, dt=1e-6, tau=1e-5)
    run.bc_y = bc_y
    fields = (run.rho, run.ux, run.uy, run.T)
    print(f"[case] {nx}x{ny} bc_y={bc_y}", flush=True)
    for precision in (1, 0):
        a, b = (Solver.from_run(run, precision, form) for form in (STEP_FUSED, STEP_SPLIT))
        f = a.init(*fields)
        want = a.step(f, nsteps=1)
        assert torch.equal(b.step(f, nsteps=1), want)
        assert torch.equal(b.step_keep_stage(f)[1], want)
    # float rounding of the initial state and of two stages, twice that to be safe
    c = Solver.from_run(run, 2)
    got = c.step(c.init(*fields), nsteps=1)[:16].double()
    assert (got - want).abs().max() < 2 * 3 * 2.0 ** -24 * want.abs().max()
