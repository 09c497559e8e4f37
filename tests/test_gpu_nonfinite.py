"""NaN, infinities and cells without mass in the states: every form of a step
treats them as the single-stage kernels do, bit for bit (also the finite
values next to them), and in the reverse pass they reach the cells of the
stencils and no others."""
import dataclasses

import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

# one per form of CDBM_STEP_AUTO: several steps a launch, tiles of 8 x 4, 8 x 8,
# 16 x 8 and 16 x 16 cells, strips and (FP64) marching strips
SIZES = [(300, 1), (9, 1), (40, 24), (3, 5), (128, 100), (150, 140), (256, 200), (900, 780)]
VALUES = {"nan": float("nan"), "inf": float("inf"), "-inf": float("-inf"), "empty": 0.0, "huge": 3e38}


def _same(a, b):
    return torch.equal(a.isnan(), b.isnan()) and torch.equal(a.nan_to_num(nan=0.5, posinf=None, neginf=None),
                                                             b.nan_to_num(nan=0.5, posinf=None, neginf=None))


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("bc", [W.PERIODIC, W.ZERO_GRADIENT])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_step_forms_agree(nx, ny, bc, precision):
    from paper_2502_16818_amd import Solver
    from paper_2502_16818_amd.cdbm import STEP_AUTO, STEP_SPLIT
    run = dataclasses.replace(W.random_periodic(nx, ny, seed=nx, dt=1e-5, tau=1e-4), bc_x=bc, bc_y=bc)
    print(f"[case] {nx}x{ny} bc={bc} precision={precision}", flush=True)
    a, b = (Solver.from_run(run, precision, form) for form in (STEP_AUTO, STEP_SPLIT))
    f0 = a.init(run.rho, run.ux, run.uy, run.T)
    for name, value in VALUES.items():
        f = f0.clone()
        for k, (x, y) in enumerate([(nx // 2, ny // 2), (0, 0), (nx - 1, ny - 1), (min(63, nx - 1), ny // 3)]):
            if name == "empty":
                f[:, y, x] = 0.0
            else:
                f[(5 * k + 1) % 16, y, x] = value
        for steps in (1, 3):
            assert _same(a.step(f, nsteps=steps), b.step(f, nsteps=steps)), (name, steps)
        for x, y in zip(a.step_keep_stage(f), b.step_keep_stage(f)):
            assert _same(x, y), name


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("bc", [W.PERIODIC, W.ZERO_GRADIENT])
@pytest.mark.parametrize("where", ["state", "adjoint"])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_step_adjoint_spreads_by_its_stencils(value, where, bc, precision):
    """Two stages of two cells, recomputed from the state: six cells in x + y at
    most; an adjoint vector reaches four."""
    from paper_2502_16818_amd import Solver
    nx, ny, x0, y0 = 90, 41, 62, 19
    run = dataclasses.replace(W.random_periodic(nx, ny, seed=2, dt=1e-4, tau=2e-4), bc_x=bc, bc_y=bc)
    s = Solver.from_run(run, precision)
    f = s.init(run.rho, run.ux, run.uy, run.T)
    g = torch.Generator(device="cuda").manual_seed(3)
    lam = torch.randn((16, ny, nx), dtype=torch.float64, device="cuda", generator=g)
    want, _ = s.step_adjoint(f, lam)
    f, lam = f.clone(), lam.clone()
    (f if where == "state" else lam)[5, y0, x0] = value
    got, _ = s.step_adjoint(f, lam)
    far = (torch.arange(nx, device="cuda")[None, :] - x0).abs() + (torch.arange(ny, device="cuda")[:, None] - y0).abs()
    outside = far > (6 if where == "state" else 4)
    assert torch.equal(got[:, outside], want[:, outside])
    assert not torch.isfinite(got[:, y0, x0]).any()
