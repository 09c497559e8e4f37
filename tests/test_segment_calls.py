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


@pytest.mark.gpu
@pytest.mark.parametrize("nx,ny", [(40, 24), (200, 150)])
def test_a_refused_segment_writes_nothing(nx, ny):
    """A null or overlapping buffer anywhere in the lists, not only beside its step."""
    import ctypes

    from paper_2502_16818_amd import Solver, cdbm
    run = W.random_periodic(nx, ny, seed=5, dt=1e-4, tau=2e-4)
    s = Solver.from_run(run, MIXED)
    f0 = s.init(run.rho, run.ux, run.uy, run.T)
    n, one = 3, f0.numel()
    pool = torch.full((2 * n - 1, *f0.shape), float("nan"), dtype=f0.dtype, device="cuda")
    f, f1 = [f0, *pool[:n - 1]], list(pool[n - 1:])
    s.steps_keep_stages(f, f1)
    lam = [torch.ones((16, ny, nx), dtype=torch.float64, device="cuda") for _ in range(2)]
    s.steps_adjoint_stages(f, f1, *lam)   # accepted as they are
    s.tau_collect()
    pool.fill_(float("nan"))
    half = pool.view(-1)[one // 2:one // 2 + one].view_as(f0)   # across the first two of the pool

    def ptrs(ts):
        return (ctypes.c_void_p * len(ts))(*[None if t is None else t.data_ptr() for t in ts])

    def keep(f, f1):
        return cdbm.load().cdbm_steps_keep_stages(s._h, ptrs(f), ptrs(f1), n, None)

    for bad_f, bad_1 in [(f, [*f1[:2], None]), ([*f[:2], None], f1), (f, [*f1[:2], f0]),
                         (f, [*f1[:2], f[1]]), ([*f[:2], f1[0]], f1), (f, [*f1[:2], half])]:
        assert keep(bad_f, bad_1) == -1
        assert torch.isnan(pool).all()

    def adjoint(f, f1, lam):
        return cdbm.load().cdbm_steps_adjoint_stages(s._h, ptrs(f), ptrs(f1), n, ptrs(lam), None)

    for t in lam:
        t.fill_(1.0)
    pool.fill_(1.0)
    want = f0.clone()
    for bad_f, bad_1, bad_l in [([None, *f[1:]], f1, lam), (f, [None, *f1[1:]], lam), (f, f1, [lam[0], None]),
                                (f, f1, [lam[0], lam[0]]), (f, f1, [lam[0], f0]), (f, f1, [f0, lam[1]]),
                                (f, f1, [f1[1], lam[1]])]:
        assert adjoint(bad_f, bad_1, bad_l) == -1
        assert (lam[0] == 1).all() and (lam[1] == 1).all() and (pool == 1).all()
        assert torch.equal(f0, want)
