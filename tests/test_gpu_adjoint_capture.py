"""Step adjoints recorded into a caller's graph on a handle that has only run
the form with a given first stage before: no allocation is left for the
recorded call.  Small grids that step on tiles, one row of cells, and a grid of
two launches; the replays against eager calls, with eager work between them."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("nx,ny", [(40, 24), (200, 190), (300, 1), (400, 300)])
def test_step_adjoint_in_a_capture_after_the_stage_form(nx, ny, precision):
    from paper_2502_16818_amd import Solver
    run = W.random_periodic(nx, ny, seed=3, dt=1e-4, tau=2e-4)
    s = Solver.from_run(run, precision)
    f = s.init(run.rho, run.ux, run.uy, run.T)
    f1, _ = s.step_keep_stage(f)
    g = torch.Generator(device="cuda").manual_seed(1)
    lam = torch.randn((16, ny, nx), dtype=torch.float64, device="cuda", generator=g)
    want, _ = s.step_adjoint(f, lam, f1=f1, defer_tau=True)
    tau = s.tau_collect()
    out = s.empty_lam()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        s.step_adjoint(f, lam, out, defer_tau=True)
    for _ in range(3):
        out.fill_(float("nan"))
        s.tau_collect()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        assert torch.equal(s.tau_collect(), tau)
