"""Which kernels CDBM_STEP_AUTO runs a step with, by the profiler's names, at
sizes on both sides of each rule (of a GPU with 256 compute units), and that
each form equals the single-stage kernels bit for bit there."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

FP64, MIXED, COMP = 0, 1, 2
LINE, TILE4, TILE8 = ["k_line_steps<{S}>"], ["k_tile_step<{S}, 4>"], ["k_tile_step<{S}, 8>"]
HALF, WHOLE = ["k_cell_tile_step<{S}, 8>"], ["k_cell_tile_step<{S}, 16>"]
SPLIT2, SPLIT1, COLUMNS = ([f"k_stage<{{S}}, {s}, {{C}}, {k}>" for s in ("false", "true")]
                           for k in ("2, false", "1, false", "1, true"))
CASES = [
    # tiles of 8 x 4 and 8 x 8 cells
    (40, 1, None, LINE), (64, 128, None, TILE4), (88, 92, None, TILE4), (90, 88, None, TILE8),
    (128, 128, None, TILE8), (5, 2040, None, TILE8),
    # 16 x 8: more than 256 tiles of 8 x 8, at most 256 of these
    (129, 128, None, HALF), (176, 170, None, HALF), (176, 176, None, HALF), (9, 2040, None, HALF),
    (2000, 15, None, HALF), (17, 1020, None, HALF),
    # 264 tiles of 16 x 8 and no more than 2^15 cells; more
    (177, 177, None, SPLIT2), (181, 170, None, SPLIT2), (181, 181, None, SPLIT2),
    (182, 181, None, WHOLE), (256, 256, None, WHOLE), (11, 4000, None, WHOLE),
    # beyond one tile of 16 x 16 per compute unit
    (257, 256, None, SPLIT2), (384, 256, None, SPLIT2), (385, 256, None, SPLIT1), (4000, 32, None, COLUMNS),
    (600, 583, FP64, SPLIT1), (600, 584, FP64, ["k_step_fused<{S}"]), (1000, 699, FP64, ["k_step_fused<{S}"]),
    (1000, 700, FP64, ["k_step_march"]), (750, 800, MIXED, SPLIT1), (751, 800, MIXED, ["k_step_fused<{S}"]),
    (100, 1, COMP, SPLIT2), (128, 128, COMP, SPLIT2), (385, 256, COMP, SPLIT1), (4000, 32, COMP, COLUMNS),
]


def _kernels(call):
    """(names of the library's kernels that a call runs, its result)"""
    for _ in range(3):   # in case the profiler hands out no events
        torch.cuda.synchronize()
        with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
            out = call()
            torch.cuda.synchronize()
        names = [e.name for e in prof.events() if "cdbm::" in e.name]
        if names:
            break
    return names, out


@pytest.mark.parametrize("nx,ny,precision,kernels", CASES)
def test_step_runs_the_form_of_its_size(nx, ny, precision, kernels):
    from paper_2502_16818_amd import Solver
    from paper_2502_16818_amd.cdbm import STEP_SPLIT
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the sizes are those of 256 compute units")
    run = W.random_periodic(nx, ny, seed=nx + ny, dt=1e-6, tau=1e-5)
    run.bc_x = W.ZERO_GRADIENT
    for p in (FP64, MIXED) if precision is None else (precision,):
        print(f"[case] {nx}x{ny} precision={p}", flush=True)
        a = Solver.from_run(run, p)
        f = a.init(run.rho, run.ux, run.uy, run.T)
        names, got = _kernels(lambda: a.step(f, nsteps=1))
        want = [k.format(S="double" if p == FP64 else "float", C="true" if p == COMP else "false") for k in kernels]
        assert len(names) == len(want) and all(w in n for w, n in zip(want, names)), names
        assert torch.equal(got, Solver.from_run(run, p, STEP_SPLIT).step(f, nsteps=1))


@pytest.mark.parametrize("precision", [FP64, MIXED])
@pytest.mark.parametrize("nx,per_launch", [(500, 7), (6000, 5), (10000, 3), (12000, 5), (16000, 4), (20000, 3), (65536, 2)])
def test_steps_per_launch_of_a_row(nx, per_launch, precision):
    """The number that was fastest when each of 1 to 7 was timed at this length."""
    from paper_2502_16818_amd import Solver
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the lengths are those of 256 compute units")
    run = W.random_periodic(nx, 1, seed=nx, dt=1e-6, tau=1e-5)
    s = Solver.from_run(run, precision)
    f = s.init(run.rho, run.ux, run.uy, run.T)
    for steps, launches in ((per_launch, 1), (per_launch + 1, 2)):
        names, _ = _kernels(lambda: s.step(f, nsteps=steps))
        assert sum("k_line_steps" in n for n in names) == launches
