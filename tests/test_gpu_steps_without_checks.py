"""Runs of a fixed number of steps (needs a GPU): the check interval plays no
part where nothing is checked, so the launches are as long as with the default
interval, and the fields are the single steps'."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("efield", [False, True])
@pytest.mark.parametrize("nx,ny", [(32, 32), (150, 61), (256, 256)])
@pytest.mark.parametrize("K", [1, 5, 9])
def test_launches_without_checks_do_not_depend_on_the_interval(nx, ny, K, efield):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_31347_amd import slbm as S
    rng = np.random.default_rng(nx)
    F = 1e-2 * rng.standard_normal((2, ny, nx))
    p = dict(nx=nx, ny=ny, dx=1.0 / max(nx, ny), E=1.0, nu=0.3, domain=S.PERIODIC, target=1e-3 * F[::-1].copy(),
             control_kind=S.CTRL_E_NODAL if efield else S.CTRL_FORCE_NODAL, fixed_force=F if efield else None, tol=0.0,
             max_steps=280)
    control = 1.0 + 0.3 * np.tanh(rng.standard_normal((ny, nx))) if efield else F
    out = []
    for interval, tuning in ((1000, -1), (K, -1), (K, 1)):
        ctx = S.solid_lbm_init(dict(p, check_interval=interval))
        S.solid_lbm_set_tuning(ctx, tuning, 0)
        S.solid_lbm_set_launch_timing(ctx, 1)
        rc, J, g, pi, ai = S.objective_and_grad(ctx, control)
        out.append((pi.fused_launches, ai.fused_launches, J, g))
    assert 0 < out[0][0] <= 280 // 8 and out[0][:2] == out[1][:2]
    for o in out[1:]:
        assert o[2] == out[0][2] and np.array_equal(o[3], out[0][3])
