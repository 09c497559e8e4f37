"""Small grids with CDBM_STEP_AUTO: both stages in one launch (tiles), several
steps in one launch (one-row grids).  Bit for bit the two single-stage
launches of CDBM_STEP_SPLIT, at the edges of the tiles, of the blocks of a row
and of the steps per launch, and on grids smaller than a stencil."""
import dataclasses

import pytest
import torch

import workloads as W
from paper_2502_16818_amd import FP64, MIXED, Solver
from paper_2502_16818_amd.cdbm import STEP_SPLIT

pytestmark = pytest.mark.gpu

# tiles of 8 x 8; the largest is the last to take this form on 256 compute units
TILES = [(1, 2), (3, 2), (7, 9), (8, 8), (17, 16), (130, 70), (128, 128), (2, 300)]
# blocks of 64 cells, of which 64 - 8 k are written for k steps per launch
ROWS = [(1, 1), (2, 1), (8, 1), (9, 1), (63, 1), (64, 1), (65, 1), (500, 1), (10001, 1), (20000, 1)]


def _pair(nx, ny, bc_x, bc_y, precision):
    run = dataclasses.replace(W.random_periodic(nx, ny, seed=nx + ny, dt=1e-4, tau=2e-4),
                              bc_x=bc_x, bc_y=bc_y, dx=1 / 64, dy=1 / 48)
    auto, split = Solver.from_run(run, precision), Solver.from_run(run, precision, STEP_SPLIT)
    return auto, split, auto.init(run.rho, run.ux, run.uy, run.T)


@pytest.mark.parametrize("precision", [FP64, MIXED])
@pytest.mark.parametrize("bc", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("size", TILES + ROWS)
def test_small_grids_equal_split_steps(size, bc, precision):
    auto, split, f = _pair(*size, *bc, precision)
    for n in (1, 2, 3, 7, 8, 16, 131):   # 131: two replays of a 7-step row's graph, one of a tile's
        a, b = auto.step(f, nsteps=n), split.step(f, nsteps=n)
        assert torch.isfinite(b).all()
        assert torch.equal(a, b), n
    a, b = auto.step_keep_stage(f), split.step_keep_stage(f)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
