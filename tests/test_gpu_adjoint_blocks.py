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
