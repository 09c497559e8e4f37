"""Grid totals at the edges of the reduction's passes (262144 cells each)
against sums of the same state on the CPU."""
import pytest
import torch

from oracle import cdbm as C
import workloads as W

pytestmark = pytest.mark.gpu

FP64, MIXED, COMP = 0, 1, 2


@pytest.mark.parametrize("precision", [FP64, MIXED, COMP])
@pytest.mark.parametrize("nx,ny", [(1, 1), (255, 1), (512, 512), (511, 513), (513, 512), (1030, 777)])
def test_totals_match_sums(nx, ny, precision):
    """Both sides add at most 16 * 8e5 terms pairwise or over blocks: far
    fewer than 1000 roundings of 1.1e-16 on any path, relative to sum |term|."""
    from paper_2502_16818_amd import Solver
    run = W.random_periodic(nx, ny, seed=nx + ny, dt=1e-5, tau=1e-4)
    print(f"[case] {nx}x{ny} precision={precision}", flush=True)
    s = Solver.from_run(run, precision)
    f = s.init(run.rho, run.ux, run.uy, run.T)
    got = s.totals(f).cpu()
    p = C.Params.from_run(run)
    vel, eta = C.discrete_velocities(p.v, p.eta)
    d = f.cpu().double().reshape(-1, ny * nx)
    sums, mags = d[:16].sum(1), d[:16].abs().sum(1)
    weight = torch.stack([torch.ones(16, dtype=torch.float64), vel[:, 0], vel[:, 1],
                          (vel ** 2).sum(1) + eta ** 2])
    want = weight @ sums
    if precision == COMP:
        want = want + d[16:].sum(1)
    assert ((got - want).abs() <= 1000 * 1.1e-16 * (weight.abs() @ mags)).all()
