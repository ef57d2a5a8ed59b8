"""Rows per wave set with automatic steps (needs a GPU): periodic uniform grids
beyond 131072 nodes run wave strips of 8 steps with those rows, and give the
single steps' fields."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# sizes whose automatic shape is a panel of 64 columns (two of them) and the pipeline; rows above and below the grid's
@pytest.mark.parametrize("nx,ny,rows", [(501, 333, 24), (512, 300, 500), (600, 600, 8), (900, 400, 32)])
def test_rows_set_by_the_caller_choose_wave_strips(nx, ny, rows):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_31347_amd import slbm as S
    rng = np.random.default_rng(nx)
    F = 1e-2 * rng.standard_normal((2, ny, nx))
    p = dict(nx=nx, ny=ny, dx=1.0 / nx, E=1.0, nu=0.3, domain=S.PERIODIC, target=1e-3 * F[::-1].copy(),
             control_kind=S.CTRL_FORCE_NODAL, tol=1e-300, check_interval=49, max_steps=150)
    out = []
    for tuning in ((1, 0), (-1, rows)):
        ctx = S.solid_lbm_init(p)
        S.solid_lbm_set_tuning(ctx, *tuning)
        S.solid_lbm_set_launch_timing(ctx, 1)
        rc, J, g, pi, ai = S.objective_and_grad(ctx, F)
        out.append((J, g))
    assert pi.fused_launches > 0 and pi.fused_sweeps == 8 * pi.fused_launches
    assert ai.fused_launches > 0 and ai.fused_sweeps == 8 * ai.fused_launches
    assert out[0][0] == out[1][0] and np.array_equal(out[0][1], out[1][1])
