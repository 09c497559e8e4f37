"""Single-stage kernels at the edges of their blocks (64 cells of a row, x
neighbours through LDS) and on both sides of the size from which a block has
one wave instead of two (98304 cells)."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

FP64, MIXED, COMP = 0, 1, 2
SIZES = [(1, 9), (2, 3), (62, 5), (63, 4), (64, 3), (65, 2), (66, 1), (127, 4), (384, 256), (313, 315)]


def _run(nx, ny, bc_x):
    run = W.random_periodic(nx, ny, seed=nx + ny, dt=1e-4, tau=2e-4)
    run.bc_x, run.bc_y = bc_x, bc_x if ny % 2 else W.ZERO_GRADIENT
    print(f"[case] {nx}x{ny} bc=({run.bc_x},{run.bc_y})", flush=True)
    return run


@pytest.mark.parametrize("bc_x", [W.PERIODIC, W.ZERO_GRADIENT])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_split_step_equals_fused_step(nx, ny, bc_x):
    """The same arithmetic per cell: equal bit for bit (FP64 and mixed)."""
    from paper_2502_16818_amd import Solver
    from paper_2502_16818_amd.cdbm import STEP_FUSED, STEP_SPLIT
    run = _run(nx, ny, bc_x)
    for precision in (FP64, MIXED):
        a, b = (Solver.from_run(run, precision, form) for form in (STEP_FUSED, STEP_SPLIT))
        f = a.init(run.rho, run.ux, run.uy, run.T)
        assert torch.equal(a.step(f, nsteps=3), b.step(f, nsteps=3))


@pytest.mark.parametrize("bc_x", [W.PERIODIC, W.ZERO_GRADIENT])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_compensated_step_follows_fp64(nx, ny, bc_x):
    """Arithmetic in double, results rounded to float: after 3 steps of two
    stages the distributions are within one float rounding (2^-24 of the
    largest value) per stage of the FP64 ones, twice that to be safe."""
    from paper_2502_16818_amd import Solver
    run = _run(nx, ny, bc_x)
    a, b = Solver.from_run(run, FP64), Solver.from_run(run, COMP)
    fields = (run.rho, run.ux, run.uy, run.T)
    want = a.step(a.init(*fields), nsteps=3)
    got = b.step(b.init(*fields), nsteps=3)[:16].double()
    err = ((got - want).abs().max() / want.abs().max()).item()
    print(f"  max error {err:.2e}")
    assert err < 2 * 7 * 2.0 ** -24


@pytest.mark.parametrize("nx,ny", [(1500, 1399), (4000, 525), (40000, 53)])
def test_large_grids_in_short_bands(nx, ny):
    """More than 2^21 cells, where the blocks are numbered in bands of eight
    rows, with rows left over: the split step and the kept-stage step against
    the fused step."""
    from paper_2502_16818_amd import Solver
    from paper_2502_16818_amd.cdbm import STEP_FUSED, STEP_SPLIT
    run = W.random_periodic(nx, ny, seed=nx + ny, dt=1e-6, tau=1e-5)
    run.bc_y = W.ZERO_GRADIENT
    print(f"[case] {nx}x{ny}", flush=True)
    a, b = (Solver.from_run(run, MIXED, form) for form in (STEP_FUSED, STEP_SPLIT))
    f = a.init(run.rho, run.ux, run.uy, run.T)
    want = a.step(f, nsteps=1)
    assert torch.equal(b.step(f, nsteps=1), want)
    assert torch.equal(b.step_keep_stage(f)[1], want)
