"""Several steps with kept stages, or their transposes, in one call: the same
as the single calls bit for bit (step forms of one and of two launches)."""
import pytest
import torch

import workloads as W

FP64, MIXED = 0, 1


def test_null_arguments_are_rejected():
    from paper_2502_16818_amd import cdbm
    lib = cdbm.load()
    assert lib.cdbm_steps_keep_stages(None, None, None, 1, None) == -1
    assert lib.cdbm_steps_adjoint_stages(None, None, None, 1, None, None) == -1


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [FP64, MIXED])
@pytest.mark.parametrize("nx,ny", [(40, 24), (200, 150)])
@pytest.mark.parametrize("n", [1, 2, 3])
def test_segment_equals_single_calls(nx, ny, n, precision):
    from paper_2502_16818_amd import Solver
    run = W.random_periodic(nx, ny, seed=n, dt=1e-4, tau=2e-4)
    run.bc_y = W.ZERO_GRADIENT
    print(f"[case] {nx}x{ny} n={n} precision={precision}", flush=True)
    s = Solver.from_run(run, precision)
    f0 = s.init(run.rho, run.ux, run.uy, run.T)
    states, stages = [f0], []
    for _ in range(n):
        f1, f = s.step_keep_stage(states[-1])
        stages.append(f1)
        states.append(f)
    got_f = [f0] + [torch.full_like(f0, float("nan")) for _ in range(n - 1)]
    got_1 = [torch.full_like(f0, float("nan")) for _ in range(n)]
    s.steps_keep_stages(got_f, got_1)
    for a, b in zip(got_f + got_1, states[:n] + stages):
        assert torch.equal(a, b)
    g = torch.Generator(device="cuda").manual_seed(n)
    lam0 = torch.randn((16, ny, nx), dtype=torch.float64, device="cuda", generator=g)
    lam = lam0
    for j in reversed(range(n)):
        lam, _ = s.step_adjoint(states[j], lam, f1=stages[j], defer_tau=True)
    want_tau = s.tau_collect()
    got, other = s.steps_adjoint_stages(got_f, got_1, lam0.clone(), s.empty_lam())
    assert torch.equal(got, lam) and got.data_ptr() != other.data_ptr()
    assert torch.equal(s.tau_collect(), want_tau)
    with pytest.raises(Exception, match="overlap"):
        s.steps_keep_stages([f0], [f0])
